// The persistent GEMM for K that is not a multiple of 128: gemm_persistent.hip once more, with its last pair of K tiles
// treated specially (see KTAIL there).
#define LOBRA_GP_KTAIL 1
#define LOBRA_GP_KERNEL gemm_persistent_ktail_kernel
#define LOBRA_GP_HOST gemm_persistent_ktail
#include "gemm_persistent.hip"

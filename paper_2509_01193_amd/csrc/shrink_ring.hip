// The rank-r projection P = s_t Z M_t^T of the bf16 path (Z = x, M = A: s_t A_t x_i; Z = dy, M = B: s_t B_t dy_i; paper section 2.1,
// one pair of factors per task of the fused batch, section 1), written token-major [T][r_pad] and block-transposed [ntb][r_pad][32].
//
// A workgroup of four waves takes G token blocks of one task and walks K through an LDS ring that direct global -> LDS copies
// fill, whole 128-byte lines at a time; its waves share K (G = 1) or own a block each (G = 4).  What bounds it: long batches the
// memory's rate for many row pieces at once, short ones the time a workgroup takes, i.e. what a compute unit can fetch past its first-level
// cache (some 70 GB/s) next to the start and the end (5 us).  Kernels that loaded the operands into registers had two or three
// slabs per wave in flight and fetched lines in halves.  Measured, those / this one, us:
//     4096 columns, rank 16, 32 .. 128 blocks     12.2 .. 12.8 / 9.6 .. 10.2      rank 64, 80 blocks     28.8 / 15.0
//     4096 columns, rank 16, 384 blocks           26.4 / 19.0                     rank 128, 128 blocks   44.3 / 22.9
//     16384 x 4096, rank 16 (K-sliced kernel and its finish)     31.2 / 26.9      65536 x 28672          869 / 651 (5.8 TB/s)
//     32768 x 11008, ranks 8 .. 64    205 / 153                                   49152 x 8192, rank 64  236 / 203 and 224 / 177
// Few blocks go in halves (H = 1), so that twice as many compute units fetch: whole passes 99.3 -> 94.6 us (35 blocks of rank 16, 4096 x 4096,
// a training step), 22.8 -> 22.3 (40 decoding requests); with whole blocks 97.3 and 22.6.  Narrow layers gain nothing there (1088 columns, 31
// blocks, a forward pass: 26.1 and 26.3), but a kernel of their own would sum in another order, and a token's result would depend on the size of
// its batch.
// G = 4 halves the rank rows' way from the L2, which at ranks from 24 is most of what a single block's workgroup fetches (49152 x 8192,
// rank 64, G = 1: 214 and 207 us).  Slots: pieces of 512 bytes per row where blocks are few (3000 x 4096, rank 64: 18.4 us, with pieces of
// 256 22.8), of 128 at G = 4 (256 no better), two workgroups per compute unit where LDS allows.
#include <atomic>

#include "shrink_ring.h"

namespace lobra {

template <int G, int H, int MAXNRB, int KS, int LDS>
__global__ __launch_bounds__(256, LDS > 80 * 1024 ? 1 : 2) void shrink_ring_kernel(PlanDev pd, const uint16_t* __restrict__ Z, const uint16_t* __restrict__ M,
                                                       const float* __restrict__ s, uint16_t* __restrict__ P_tok,
                                                       uint16_t* __restrict__ P_blk, int32_t D, int32_t ldz, int32_t nproj, int32_t proj,
                                                       int32_t rparts)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char ring[];
    ring_item<G, H, MAXNRB, KS, LDS>(pd, Z, M, s, P_tok, P_blk, D, ldz, nproj, proj, rparts, int32_t(blockIdx.z * gridDim.x + blockIdx.x),
                                     int32_t(blockIdx.y), ring);
}

template <int G, int H, int MAXNRB, int KS, int LDS>
static hipError_t launch_ring(const PlanDev& pd, const void* Z, const void* M, const float* s, void* P_tok, void* P_blk, int32_t D,
                              int32_t ldz, int32_t nproj, int32_t proj, int32_t rparts, hipStream_t st)
{
    // the kernel needs more dynamic LDS than the default limit: raise it once per device
    static std::atomic<uint64_t> raised{0};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = uint64_t(1) << (dev & 63);
    if (!(raised.load(std::memory_order_acquire) & bit)) {
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(&shrink_ring_kernel<G, H, MAXNRB, KS, LDS>), hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        if (e != hipSuccess) return e;
        raised.fetch_or(bit, std::memory_order_release);
    }
    // up to 2^23 items in a row of the grid (a dimension of 2^32 threads and more wraps without an error)
    const int32_t items = G == 1 ? pd.ntb : pd.nsb, rows = (items - 1) / (1 << 23) + 1, row = rows > 1 ? 1 << 23 : items;
    shrink_ring_kernel<G, H, MAXNRB, KS, LDS><<<dim3(row, 2 / H * rparts * (proj < 0 ? nproj : 1), rows), 256, LDS, st>>>(
        pd, (const uint16_t*)Z, (const uint16_t*)M, s, (uint16_t*)P_tok, (uint16_t*)P_blk, D, ldz, nproj, proj, rparts);
    return hipGetLastError();
}

hipError_t shrink_ring(const PlanDev& pd, const void* Z, const void* M, const float* s, void* P_tok, void* P_blk, int32_t D,
                       int32_t ldz, int32_t nproj, int32_t proj, hipStream_t st)
{
    const int nrb = (pd.r_max / nproj + 15) / 16;    // rank blocks of the widest window
    constexpr int HALF = 80 * 1024, ALL = 160 * 1024;
#define LOBRA_RING(G, H, MAXNRB, KS, LDS) launch_ring<G, H, MAXNRB, KS, LDS>(pd, Z, M, s, P_tok, P_blk, D, ldz, nproj, proj, (nrb + MAXNRB - 1) / MAXNRB, st)
    if (pd.shrink_group == 4 && nproj == 1) return nrb <= 4 ? LOBRA_RING(4, 2, 4, 64, HALF) : LOBRA_RING(4, 2, 8, 64, HALF);
    // The fewer ranks a workgroup has the sooner it is done, as long as all run at once (us at 4096 columns for 16, 32, 64 and 128 ranks per
    // workgroup: 128 of them 10.2, 12.4, 15.5, 22.9; 256 14.0, 15.4, 17.4, 24.2; 384 19.0, 23.8, 28.5, 41.8)
    const int64_t blocks = int64_t(pd.ntb) * (proj < 0 ? nproj : 1);
    // (whole passes with pieces of 256 bytes and 40 KB of LDS: 24.7 and 98.5 us where these take 22.3 and 94.6)
    if (blocks * nrb <= 128) return LOBRA_RING(1, 1, 1, 256, HALF);
    if (nrb <= 1 || blocks * nrb <= 192) return LOBRA_RING(1, 2, 1, 256, HALF);
    if (nrb <= 2 || blocks * ((nrb + 1) / 2) <= 256) return LOBRA_RING(1, 2, 2, 256, ALL);
    if (nrb <= 4 || blocks * ((nrb + 3) / 4) <= 256) return LOBRA_RING(1, 2, 4, 256, ALL);
    return LOBRA_RING(1, 2, 8, 128, ALL);
#undef LOBRA_RING
}

}  // namespace lobra

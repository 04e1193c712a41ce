// Persistent bf16 MFMA GEMM for gfx950 with the LoRA up projection fused into its epilogue:
//     C[T, N] = Z[T, K] * op(W) + P[T, r] * M_t[r, N]
// forward : Z = x,  op(W) = W   (W stored [K][N], N fastest),  P = s_t A_t x_i,  M = B  -> y
// backward: Z = dy, op(W) = W^T (W stored [N][K], K fastest),  P = s_t B_t dy_i, M = A  -> dx
// (paper section 2.1: X W + X (down)(up); section 1: one shared base product for the fused batch,
// a per-task adapter product on top of it).
//
// One workgroup per compute unit walks a few 256 x 256 output tiles (LOBRA_GP_TPW of them; then the next round of
// workgroups is dispatched, which re-aligns the compute units of an XCD that share panels through its L2):
//   * the K tiles of ALL of a workgroup's output tiles form one stream through the two LDS stages: while the
//     last K tiles of an output tile are multiplied, the first K tiles of the next one are already being
//     copied, so no stage fill is exposed except the very first;
//   * the epilogue keeps its hands off the two stages: the operands of the fused up projection's steps are copied
//     to a third LDS region (the first step's while the tile's last K tile is multiplied, see prefetch_adapter;
//     every other's under the step before), and the result is rounded, passed through the same region
//     (a 64 x 64 block per wave at a time) and stored in whole 128-byte lines; the stores drain under the next
//     tile's first MFMAs.
// One workgroup per output tile instead costs about 15 us per tile (workgroup start, two exposed stage fills,
// the epilogue and its store drain) next to 80 us of MFMAs at K = 4096; of that the stream hides what is not the
// stores and the epilogue's own instructions.
//
// Tile: 256 x 256 x 64, four waves of 128 x 128 (one per SIMD), blocks of v_mfma_f32_16x16x32_bf16 with the
// 64 accumulators of a wave in its 256 AGPRs, which the kernel names itself (gemm_common.h).  The MFMA "A"
// operand is fed from W and the "B" operand from Z, so a lane ends up with four output columns of one token row
// per block; block_col deals the columns of a wave tile to the blocks so that two blocks give a lane 8
// consecutive columns.
// K tiles go global -> LDS with global_load_lds_dwordx4 (no registers, no ds_write); every row segment a copy
// fetches is one 128-byte line.  With one wave per SIMD nothing hides a wave's own latencies, so the loop is
// software-pipelined by hand and its order is pinned (the MFMAs are volatile asm statements, sched_barrier
// between the slots); see kstep for the schedule of a K step.
//
// LDS: stage 0, stage 1 (64 KiB each: Z tile then W tile), up projection's step / result staging (32 KiB).
//   Z tile, and the W tile when K is fastest (backward): [256 rows][64 k], 16-byte chunk c of a row
//       stored at c ^ ((row >> 1) & 7): the 16 rows of one ds_read_b128 pass hit 16 bank groups.
//   W tile when N is fastest (forward), adapter slice: [k][256 n], chunk c of k-row k stored at c ^ kn_swz2(k);
//       the MFMA operand (8 consecutive k of one column) is gathered with two ds_read_b64_tr_b16.
//   A wave-wide direct-to-LDS copy lands in lane order, so the swizzle - and, backward, the dealing of the
//       columns to the MFMA blocks - is applied to the global address each lane fetches from.
#include <atomic>
#include <type_traits>

#include "gemm_common.h"
#include "kernels.h"

#ifndef LOBRA_GP_TPW
#define LOBRA_GP_TPW 4       // output tiles per workgroup
#endif
#ifndef LOBRA_GP_STORES_IN_FLIGHT
#define LOBRA_GP_STORES_IN_FLIGHT 32   // stores of an epilogue (MB x NB / 2 per wave); 0: wait for them at the next barrier
#endif
#ifndef LOBRA_GP_STORE
#define LOBRA_GP_STORE 1     // 1: non-temporal stores of whole lines through LDS (the product); 4: 64-byte pieces straight from the
                             // accumulators; 0 / 2: timing variants (hardly any stores / plain stores)
#endif

// This file is compiled twice: as it is for K that is a multiple of 128, and by gemm_persistent_ktail.hip for any other K,
// as kernels of another name (a flag of one template would do, but the two together cost the first one its last free
// registers).
#ifndef LOBRA_GP_KTAIL
#define LOBRA_GP_KTAIL 0
#define LOBRA_GP_KERNEL gemm_persistent_kernel
#define LOBRA_GP_HOST gemm_persistent
#endif

namespace lobra {

using namespace gemm;

namespace {

constexpr int WM = 2, WN = 2, NW = WM * WN;          // waves
constexpr int TM = BM / WM, TN = BN / WN;            // wave tile 128 x 128
constexpr int MB = TM / 16, NB = TN / 16;            // 16 x 16 blocks per wave
constexpr int ZT_BYTES = BM * BK * 2;                // one operand tile: 32 KiB
constexpr int STAGE_BYTES = 2 * ZT_BYTES;            // Z tile + W tile
constexpr int RSTEP = 32;                            // ranks per step of the up projection
constexpr int MSLICE_OFF = 2 * STAGE_BYTES;          // adapter region: RSTEP rank rows of M_t's 256 columns,
constexpr int P_OFF = RSTEP * BN * 2;                // then RSTEP ranks of the tile's 256 rows of P
constexpr int MSLICE_BYTES = P_OFF + BM * RSTEP * 2;
constexpr int LDS_BYTES = MSLICE_OFF + MSLICE_BYTES; // 160 KiB
constexpr int RCOPIES = 4;                           // 1 KiB copies per wave and step for each of the two
static_assert(RCOPIES * NW * 1024 == P_OFF && 2 * P_OFF == MSLICE_BYTES, "a step's operands fill the adapter region");
constexpr int NBZ = (BK / 2) / NW;                   // 1 KiB copy blocks per wave, for Z and for W each
constexpr int NU = MB + NB;                          // fragments per K step of 32 = sections per K step
static_assert(NW == 4 && MB == 8 && NB == 8 && MB * NB == 4 * NU && 2 * NBZ == NU && BK == 64,
              "four waves of 128 x 128: four MFMAs and at most one copy per section");
static_assert(LDS_BYTES <= 160 * 1024, "LDS budget");
static_assert(BM == kGemmTileRows, "the plan's tile-row table is made for this tile height");

// Column of the wave tile that MFMA block nb produces in its result row i (= row i of its "A" operand).
// Lane (j, kg) of a block holds result rows 4 kg .. 4 kg + 3, so with this dealing the blocks 2 p and
// 2 p + 1 together give it the 8 consecutive columns 32 p + 8 kg .. + 7 of token row j: the low four from block
// 2 p and the high four from block 2 p + 1 when kg is even, the other way round when kg is odd (the alternation
// is what lets the forward kernel's transpose reads use both halves of every 16-byte chunk, see kn_swz2).
__device__ __forceinline__ int block_col(int nb, int i)
{
    return 32 * (nb >> 1) + 8 * (i >> 2) + 4 * ((nb ^ (i >> 2)) & 1) + (i & 3);
}

constexpr int acc_reg(int mb, int nb) { return 4 * (NB * mb + nb); }   // first AGPR of accumulator (mb, nb)

}  // namespace

template <bool W_KN>
__global__ __launch_bounds__(64 * NW)
void LOBRA_GP_KERNEL(PlanDev pd, const uint16_t* __restrict__ Z, const uint16_t* __restrict__ W,
                     const uint16_t* __restrict__ P, const uint16_t* __restrict__ M,
                     uint16_t* __restrict__ C, int32_t K, int32_t N, int32_t ldw, int32_t ldc,
                     int32_t nproj, int32_t proj, int32_t tiles_m, int32_t tiles_n, int32_t GM, int32_t cpx,
                     int32_t TPW, const int32_t* __restrict__ tile_seg, const int32_t* __restrict__ cseg_off,
                     const int32_t* __restrict__ cseg_task, const int32_t* __restrict__ rank_off)
{
    constexpr bool KTAIL = LOBRA_GP_KTAIL;
    // KTAIL: K is not a multiple of 128 (any multiple of 8 from kPersistentMinKTail on).  The last pair of K tiles is then partly,
    // its second tile perhaps wholly, beyond K: their copies repeat the last valid chunk, and both operands' fragments
    // are cleared in registers in front of the K steps that reach beyond K.  A kernel of its own, so that whole K tiles
    // do not pay for it.
    // tile_seg, cseg_off, cseg_task, rank_off: pd's tables of those names once more, as arguments of their own that
    // promise not to alias anything the kernel writes: their entries are the same for every lane, and with the
    // promise the compiler fetches them with scalar loads, which no vector memory operation in flight - copies,
    // stores - has to be waited for first.
    // cpx: workgroups an XCD runs at one time (one per compute unit); TPW: output tiles per workgroup.
    // ldc: row pitch of C.  nproj > 1: this launch is projection `proj` of a fused shared-input
    // call: of every task's rank rows (in M) and rank columns (in P) only the window
    // [proj r, (proj + 1) r) takes part, r = the task's stacked rank / nproj.  proj < 0: the launch
    // covers all projections (N = nproj * pd.dg, pd.dg a multiple of the tile width) and a tile takes
    // the projection its columns lie in; M is then the compact [R_tot][pd.dg] array.
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WN, wn = wave % WN;
    // MFMA 16x16x32 lanes: j = row of the "B" operand (a token) and of the result, kg = group of 8 k
    // (operands) or of 4 result rows of the "A" operand (columns of C)
    const int j = lane & 15, kg = lane >> 4;
    const int32_t T = pd.T;
    // an even number of K tiles (the launcher guarantees K % (2 BK) == 0 unless KTAIL)
    const int32_t KT = KTAIL ? (K + 2 * BK - 1) / (2 * BK) * 2 : K / BK;

    // ---- this workgroup's output tiles.  Consecutive workgroup ids go to different XCDs (each with its own
    //      L2), so every XCD gets a contiguous range of the tile order; inside the order, GM tile-rows share one
    //      sweep over the tile-columns.  The cpx workgroups that an XCD runs at one time walk its range side by
    //      side - at any moment they work on cpx neighbouring tiles and share their panels through the L2 - but
    //      only for TPW tiles each: then the next cpx workgroups are dispatched.  (A workgroup that kept its
    //      place for the whole launch would drift: one that falls behind misses the panels its neighbours have
    //      fetched, which slows it further; at 112 tiles per compute unit that cost 5 % and 44 % more L2 misses.)
    const int32_t ntiles = tiles_m * tiles_n;
    const int32_t wg = blockIdx.x;
    const int32_t xcd = wg & 7, xidx = wg >> 3;
    const int32_t xper = ntiles >> 3, xrem = ntiles & 7;
    const int32_t xstart = xcd * xper + min(xcd, xrem), xcount = xper + (xcd < xrem ? 1 : 0);
    const int32_t xwgs = cpx;                        // stride between a workgroup's tiles
    const int32_t xfirst = (xidx / cpx) * (cpx * TPW) + xidx % cpx;      // its first tile within the XCD's range
    const int32_t my_tiles = xfirst < xcount ? min(TPW, (xcount - xfirst + cpx - 1) / cpx) : 0;
    if (my_tiles == 0) return;                       // uniform over the workgroup
    auto tile_origin = [&](int32_t n, int32_t& row0, int32_t& col0) {   // my n-th tile
        const int32_t id = xstart + xfirst + n * xwgs;
        const int32_t group = id / (GM * tiles_n);
        const int32_t first_m = group * GM;
        const int32_t gsz = min(tiles_m - first_m, GM);
        const int32_t in = id - group * GM * tiles_n;
        // The last tile row / column of a shape that is not a multiple of the tile is moved up / left until it
        // fits (the launcher guarantees T >= BM, N >= BN): it computes some elements of its neighbour once
        // more, bit for bit the same, and no tile needs clamped addresses or masked stores.
        row0 = min((first_m + in % gsz) * BM, T - BM);
        col0 = min((in / gsz) * BN, N - BN);
    };

    // Accumulator (mb, nb) of this wave is a[acc_reg(mb, nb) : + 3] (see gemm_common.h); its register v holds
    // token row mb 16 + j of the wave tile, column block_col(nb, 4 kg + v).  Nothing clears them: the first K
    // step of every output tile starts from zero.

    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    const uint32_t lds0 = uint32_t(uintptr_t((__attribute__((address_space(3))) unsigned char*)lds));
    const uint32_t ldsw = lds0 + wave_u * 1024;      // where this wave's first copy block of stage 0 lands

    // ---- copy side: the stream of K tiles.  Copy block b (1 KiB) of an operand tile holds rows 8 b .. 8 b + 7
    //      of a [rows][64 k] tile or k rows 2 b, 2 b + 1 of a [64 k][256 n] tile; wave w moves blocks w, w + 4, ...
    //      The per-lane source offsets are the same for every tile.
    uint32_t zvo[NBZ], wvo[NBZ];
#pragma unroll
    for (int c = 0; c < NBZ; ++c) {
        const int blk = wave + NW * c;
        const int row = 8 * blk + lane / 8;
        const int ch = (lane % 8) ^ swz_row(row);
        zvo[c] = (uint32_t(row) * uint32_t(K) + 8u * ch) * 2u;
        if (W_KN) {
            const int krow = 2 * blk + (lane >> 5);
            const int chn = (lane & 31) ^ kn_swz2(krow);
            wvo[c] = (uint32_t(krow) * uint32_t(ldw) + 8u * chn) * 2u;
        } else {
            // LDS row `row` of the W tile feeds result row (row & 15) of block (row & 127) >> 4 of wave
            // row >> 7: it holds the column that block_col deals to it
            const int gcol = (row & ~127) + block_col((row & 127) >> 4, row & 15);
            wvo[c] = (uint32_t(gcol) * uint32_t(ldw) + 8u * ch) * 2u;
        }
    }
    const unsigned char *zcur, *wcur;                // K tile the next copies fetch
    const size_t wstep = W_KN ? size_t(BK) * ldw * 2 : size_t(BK) * 2;
    auto set_copy_tile = [&](int32_t n) {
        int32_t r0, c0;
        tile_origin(n, r0, c0);
        zcur = reinterpret_cast<const unsigned char*>(Z + size_t(r0) * K);
        wcur = reinterpret_cast<const unsigned char*>(W_KN ? W + c0 : W + size_t(c0) * ldw);
    };
    int32_t c_n = 0, c_kt = 0;                       // the copy cursor: my c_n-th tile, its K tile c_kt
    auto advance = [&]() __attribute__((always_inline)) {
        if (c_kt + 1 < KT) {
            ++c_kt;
            zcur += BK * 2;
            wcur += wstep;
        } else if (c_n + 1 < my_tiles) {
            ++c_n;
            c_kt = 0;
            set_copy_tile(c_n);
        }
        // else: past the end the last K tile is copied once more into a stage nobody reads any more,
        // which keeps the loop free of branches around the copies
    };
    // where copy c of a K tile lands: Z blocks, then W blocks.  stage_addr = the stage + 1024 x this wave's number
    auto copy_lds_addr = [&](uint32_t stage_addr, int c) {
        return c < NBZ ? stage_addr + NW * c * 1024 : stage_addr + ZT_BYTES + NW * (c - NBZ) * 1024;
    };

    // ---- compute side: operand fragments of K step ks (32 k) of a stage.  Block mb of a [rows][64 k] tile
    //      lies 16 rows = 2048 bytes behind block 0 and (row >> 1) & 7 does not depend on mb, so one per-lane
    //      address per step serves all blocks through the instruction's offset field.
    const int fzj = swz_row(j);
    auto zaddr = [&](int stage, int ks) {
        return lds + stage * STAGE_BYTES + (wm * TM + j) * (BK * 2) + ((4 * ks + kg) ^ fzj) * 16;
    };
    auto waddr = [&](int stage, int ks) {            // backward layout only
        return lds + stage * STAGE_BYTES + ZT_BYTES + (wn * TN + j) * (BK * 2) + ((4 * ks + kg) ^ fzj) * 16;
    };
    auto read_z = [&](const unsigned char* za, int mb, bf16x8 (&zf)[MB]) {
        zf[mb] = *reinterpret_cast<const bf16x8*>(za + mb * 16 * (BK * 2));
    };
    // "A" operand of block nb out of a [k][256 n] tile at `base`: k rows krow0 + 8 kg + (j >> 2) + {0, 4}, the
    // 4-column group (j & 3) of the block - with block_col's dealing that is columns 32 (nb / 2) + 8 (j & 3)
    // + 4 ((nb + j) % 2) .. + 3 of the wave tile
    auto read_kn = [&](const unsigned char* base, int krow0, int nb, int j, int kg) __attribute__((always_inline)) {
        const int krow = krow0 + 8 * kg + (j >> 2);
        const int n = wn * TN + 32 * (nb >> 1) + 8 * (j & 3) + 4 * ((nb ^ j) & 1);
        const int ch = (n >> 3) ^ kn_swz2(krow);
        return tr_pair(base + krow * 512 + ch * 16 + (n & 7) * 2, 512);
    };
    auto read_w = [&](const unsigned char* wa, int stage, int ks, int nb, bf16x8 (&wf)[NB]) __attribute__((always_inline)) {
        if (W_KN) wf[nb] = read_kn(lds + stage * STAGE_BYTES + ZT_BYTES, 32 * ks, nb, j, kg);
        else wf[nb] = *reinterpret_cast<const bf16x8*>(wa + nb * 16 * (BK * 2));
    };
    // One K step of 32: the MB NB = 64 MFMAs in NU = 16 sections of four.  A wave issues one instruction every
    // four cycles and an MFMA of this shape keeps its pipe for 16, so a section has room for 12 other
    // instructions before the matrix pipe runs dry; whatever is not an MFMA is placed behind one.
    // Token-row block mb is done in sections 2 mb and 2 mb + 1, after which its fragment zf[mb] is dead and is
    // re-read for K step rks of stage rstage (the step that follows); the other operand lives through the
    // whole step, so its next fragments go to a second register set (wn_).
    //   STEP_FIRST / STEP_PLAIN (K step 0 of a K tile; FIRST: of an output tile - its MFMAs start from zero):
    //       one fragment read per section; `hook` (the stream's bookkeeping, scalar) runs behind the first MFMA
    //       of section 1 instead of between two K steps, where nothing would cover it.
    //   STEP_COPY (K step 1 of a K tile): the K tile's barrier stands behind the first MFMA of section 1 - the
    //       last fragment read of the stage was issued a section and a half earlier, so the wait in front of
    //       the barrier finds it done (directly behind that read it cost the LDS latency once per K tile).
    //       Sections 2 .. 15 then read the first fragments of the next K tile from the other stage and issue
    //       the 16 copies of the K tile at (zcur, wcur) into the stage at cst, which the barrier has freed
    //       (issued back to back the copies block their wave for as long as the texture unit takes to accept
    //       them): one read and one copy per section, two of each in sections 2 and 3.
    //   STEP_COPY_TAIL: the same with the copies of one of the two K tiles that may reach beyond K.  Their addresses are
    //       taken from a base 128 k earlier, so that the offset of a chunk that is moved back stays positive.
    enum { STEP_FIRST, STEP_PLAIN, STEP_COPY, STEP_COPY_TAIL };
    auto kstep = [&](auto mode_c, int rstage, int rks, bf16x8 (&zf)[MB], bf16x8 (&wc)[NB], bf16x8 (&wn_)[NB], uint32_t cst,
                     auto&& hook) __attribute__((always_inline)) {
        constexpr int mode = decltype(mode_c)::value;
        constexpr bool copies = mode == STEP_COPY || mode == STEP_COPY_TAIL;
        // (opaque to the optimiser, so that the 16 landing addresses of a K tile are sums with a literal here
        //  instead of 16 loop-invariant registers that have to be spilled)
        asm volatile("" : "+s"(cst));
        // (KTAIL: the loop's branches meet here, and where they do the compiler may have moved a fragment by a vector ALU
        //  instruction: an MFMA statement must not read a register in the two wait states after such a write)
        if constexpr (KTAIL) {
            asm volatile("s_nop 1" : "+v"(zf[0]), "+v"(zf[1]), "+v"(zf[2]), "+v"(zf[3]), "+v"(zf[4]), "+v"(zf[5]), "+v"(zf[6]), "+v"(zf[7]),
                                     "+v"(wc[0]), "+v"(wc[1]), "+v"(wc[2]), "+v"(wc[3]), "+v"(wc[4]), "+v"(wc[5]), "+v"(wc[6]), "+v"(wc[7]));
        }
        agpr_fence();
        const unsigned char* za = zaddr(rstage, rks);
        const unsigned char* wa = waddr(rstage, rks);
        // STEP_COPY_TAIL: k left in the K tile at the copy cursor (it may be negative), and how far back this lane's chunk
        // of a [rows][64 k] tile moves (row and chunk of a lane are the same in all of its copies up to a multiple of 16)
        // (lane opaque to the optimiser: worked out here, instead of in registers that live through the main loop)
        int ln = lane;
        if constexpr (mode == STEP_COPY_TAIL) asm volatile("" : "+v"(ln));
        const int32_t left = K - c_kt * BK;
        const uint32_t back = 2u * uint32_t(max(8 * ((ln % 8) ^ swz_row(8 * wave_u + ln / 8)) - (left - 8), 0));
        auto copy_src = [&](int c) __attribute__((always_inline)) {
            if constexpr (mode == STEP_COPY_TAIL) return c < NBZ ? zcur - 256 : wcur - (W_KN ? size_t(128) * ldw * 2 : size_t(256));
            else return c < NBZ ? zcur : wcur;
        };
        auto copy_off = [&](int c) __attribute__((always_inline)) {
            if constexpr (mode == STEP_COPY_TAIL) {
                if (c < NBZ) return zvo[c % NBZ] + 256u - back;
                if (!W_KN) return wvo[c % NBZ] + 256u - back;
                const int krow = 2 * (wave_u + NW * (c % NBZ)) + (ln >> 5);
                return wvo[c % NBZ] + uint32_t(128 - max(krow - (left - 1), 0)) * (uint32_t(ldw) * 2u);
            } else {
                return c < NBZ ? zvo[c % NBZ] : wvo[c % NBZ];
            }
        };
        static_for<0, NU>([&](auto u_c) {
            constexpr int u = decltype(u_c)::value, mb = u / 2, nb0 = (NB / 2) * (u % 2);
            if constexpr (copies && u >= 2) {
                mfma2_dma16<acc_reg(mb, nb0), acc_reg(mb, nb0 + 1)>(wc[nb0], wc[nb0 + 1], zf[mb], copy_lds_addr(cst, u - 2),
                                                                   copy_src(u - 2), copy_off(u - 2));
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (u < 4) {
                    mfma2_dma16<acc_reg(mb, nb0 + 2), acc_reg(mb, nb0 + 3)>(wc[nb0 + 2], wc[nb0 + 3], zf[mb],
                                                                           copy_lds_addr(cst, 12 + u), copy_src(12 + u), copy_off(12 + u));
                } else {
                    mfma_acc<acc_reg(mb, nb0 + 2)>(wc[nb0 + 2], zf[mb]);
                    __builtin_amdgcn_sched_barrier(0);
                    mfma_acc<acc_reg(mb, nb0 + 3)>(wc[nb0 + 3], zf[mb]);
                }
            } else {
                static_for<0, 4>([&](auto q_c) {
                    constexpr int q = decltype(q_c)::value;
                    if constexpr (mode == STEP_FIRST) mfma_first<acc_reg(mb, nb0 + q)>(wc[nb0 + q], zf[mb]);
                    else mfma_acc<acc_reg(mb, nb0 + q)>(wc[nb0 + q], zf[mb]);
                    if constexpr (u == 1 && q == 0) hook();
                    if constexpr (q < 3) __builtin_amdgcn_sched_barrier(0);
                });
            }
            if constexpr (!copies) {
                if constexpr (u % 2 == 0) read_w(wa, rstage, rks, u / 2, wn_);
                else read_z(za, mb, zf);
            } else if constexpr (u == 2) {
                read_w(wa, rstage, rks, 0, wn_);
                read_z(za, 0, zf);
            } else if constexpr (u == 3) {
                read_w(wa, rstage, rks, 1, wn_);
                read_z(za, 1, zf);
            } else if constexpr (u >= 4) {
                if constexpr (u % 2 == 0) read_w(wa, rstage, rks, u / 2, wn_);
                else read_z(za, mb, zf);
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    using step_first = std::integral_constant<int, STEP_FIRST>;
    using step_plain = std::integral_constant<int, STEP_PLAIN>;
    using step_copy = std::integral_constant<int, STEP_COPY>;
    using step_copy_tail = std::integral_constant<int, STEP_COPY_TAIL>;

    // ---- fused up projection: for every segment with an adapter that crosses the tile, its ranks are further K steps of 32:
    //      acc += M_t^T[:, cols] * P[rows, :]^T, rows outside the segment and ranks beyond r_t cleared in registers.  A step has
    //      two halves of 16 ranks: the two of one segment's window of 32, or, where a window has at most 16 ranks left, those
    //      and all of the next segment's, if it has at most 16.  (A window of more is never divided between steps, so a row's
    //      sum does not depend on what else is in its tile.)  Of two segments each is multiplied only with the blocks of 16 rows
    //      that it crosses: zeros in place of a row of P would not keep out what is not finite in another task's adapter.
    //      Both operands are copied into the adapter region, M_t in the [k][256 n] layout (rows beyond a half's last repeat it),
    //      P 64 bytes a row (chunks beyond repeat the half's first): the first step's while the tile's last K tile is multiplied,
    //      and every other's behind the reads of the one before, under its MFMAs.  What a step costs beyond its 64 MFMAs per wave
    //      is what is left of one round trip to memory.  (With each segment's slice passing through registers behind its own
    //      chain of table reads, five round trips at rank 64, a step of 49152 x 8192 x 8192, 32 tasks of rank 64, took 9837 us, with
    //      this 9764; 8190 x 1376 x 4096, rank 16, 236.4 -> 232.4; 16384 x 2048 x 4096 in segments of 40 tokens 508 -> 487; the forward
    //      product of 47000 x 600 x 7232 at rank 128 804 -> 625, of 12000 x 584 x 1000 in segments of four tokens 151 -> 85.)
    //      tile_seg's record of the tile row, read when the tile's main loop begins: scalar registers.
    auto rfl = [](int32_t v) { return __builtin_amdgcn_readfirstlane(v); };
    int32_t rec[kGemmTileSegRec];
    struct Half { int32_t lo, hi, m, n, pc; };       // rows, first row of M, ranks (0: none), first column of P
    struct Walk {                                    // over a tile's segments:
        int32_t e, sg, lo, hi, m, r, k, pc;          // entry, next segment to look at, the segment, its window, next rank of it
        int32_t pj, mcol0, mpitch;                   // the tile's projection, its first column, the row pitch of M
        Half a, b;                                   // the step that is in the region, or on its way
    };
    auto window = [&](Walk& w, int32_t lo, int32_t hi, int32_t r0, int32_t stacked) __attribute__((always_inline)) {
        w.lo = lo;
        w.hi = hi;
        w.r = nproj == 1 ? stacked : rfl(stacked / nproj);
        w.pc = w.pj * w.r;
        w.m = r0 + w.pc;
        w.k = 0;
    };
    auto next_segment = [&](Walk& w, int32_t row_end) __attribute__((always_inline)) {     // w.r = 0: there is none
        ++w.e;
        if (w.e < kGemmTileSegs) {
            const bool one = w.e == 1;
            window(w, one ? rec[4] : rec[8], one ? rec[5] : rec[9], one ? rec[6] : rec[10], one ? rec[7] : rec[11]);
            return;
        }
        w.r = 0;
        for (; w.sg < pd.nseg; ++w.sg) {
            const int32_t lo = rfl(cseg_off[w.sg]);
            if (lo >= row_end) return;
            const int32_t t = rfl(cseg_task[w.sg]);
            if (t < 0) continue;
            const int32_t r0 = rfl(rank_off[t]);
            window(w, lo, rfl(cseg_off[w.sg + 1]), r0, rfl(rank_off[t + 1]) - r0);
            ++w.sg;
            return;
        }
    };
    auto load_table = [&](int32_t row0) __attribute__((always_inline)) {
        if (!P) return;
        // (the last tile row may start above a multiple of the tile height)
        const int32_t* src = tile_seg + size_t((row0 + BM - 1) / BM) * kGemmTileSegRec;
#pragma unroll
        for (int i = 0; i < 4 * kGemmTileSegs + 1; ++i) rec[i] = src[i];
    };
    // the next step into (w.a, w.b); false: there is none
    auto next_step = [&](Walk& w, int32_t row_end) __attribute__((always_inline)) {
        if (w.r == 0) return false;
        const int32_t left = w.r - w.k;
        w.a = Half{w.lo, w.hi, w.m + w.k, min(left, 16), w.pc + w.k};
        w.b = Half{w.lo, w.hi, w.a.m, 0, w.a.pc};
        if (left > 16) {
            w.b.m += 16;
            w.b.n = min(left - 16, 16);
            w.b.pc += 16;
        }
        w.k += 32;
        if (w.k >= w.r) {
            next_segment(w, row_end);
            if (left <= 16 && w.r > 0 && w.r <= 16) {
                w.b = Half{w.lo, w.hi, w.m, w.r, w.pc};
                next_segment(w, row_end);
            }
        }
        return true;
    };
    // the first step.  (Worked out where its operands are copied and once more in the epilogue: carried through the main loop, a walk's
    // numbers take the scalar registers of the loop's own counts, whose way back from vector registers it then waits for: 1 % of
    // 16384 x 4096 x 4096.)
    auto first_step = [&](Walk& w, int32_t row0, int32_t col0) __attribute__((always_inline)) {
        w.e = 0;
        w.sg = rec[4 * kGemmTileSegs];
        w.pj = proj >= 0 ? proj : rfl(col0 / pd.dg);
        w.mcol0 = proj >= 0 ? 0 : w.pj * pd.dg;
        w.mpitch = proj >= 0 ? N : pd.dg;
        window(w, rec[0], rec[1], rec[2], rec[3]);
        return next_step(w, min(row0 + BM, T));
    };
    // copies a step's operands for the tile at (row0, col0): 2 RCOPIES copies per wave
    auto copy_step = [&](const Walk& w, int32_t row0, int32_t col0) __attribute__((always_inline)) {
        // (opaque to the optimiser: the per-lane offsets are worked out here instead of living in loop-invariant registers
        //  through the main loop)
        int ln = lane;
        asm volatile("" : "+v"(ln));
#pragma unroll
        for (int c = 0; c < RCOPIES; ++c) {
            const int krow = 2 * (wave_u + NW * c) + (ln >> 5);      // half c / 2
            const int32_t m = c < RCOPIES / 2 ? w.a.m : w.b.m, n = c < RCOPIES / 2 ? w.a.n : w.b.n;
            dma16(lds0 + MSLICE_OFF + (wave_u + NW * c) * 1024,
                  reinterpret_cast<const unsigned char*>(M + size_t(m) * w.mpitch + (col0 - w.mcol0)),
                  (uint32_t(min(krow & 15, max(n - 1, 0))) * uint32_t(w.mpitch) + 8u * ((ln & 31) ^ kn_swz2(krow))) * 2u);
        }
        const int ch = ln & 3, k = 8 * (ch & 1);
        const int32_t pcol = ch < 2 ? w.a.pc + (k < w.a.n ? k : 0) : w.b.pc + (k < w.b.n ? k : 0);
#pragma unroll
        for (int c = 0; c < RCOPIES; ++c)
            dma16(lds0 + MSLICE_OFF + P_OFF + (wave_u + NW * c) * 1024, reinterpret_cast<const unsigned char*>(P + size_t(row0) * pd.r_pad),
                  (uint32_t(16 * (wave_u + NW * c) + (ln >> 2)) * uint32_t(pd.r_pad) + uint32_t(pcol)) * 2u);
    };
    auto prefetch_adapter = [&](int32_t row0, int32_t col0) __attribute__((always_inline)) {
        if (!P) return;                              // uniform
        Walk w;
        if (first_step(w, row0, col0)) copy_step(w, row0, col0);
    };
    // ---- epilogue of the tile at (row0, col0): fused up projection, then fp32 -> bf16 and the stores.
    const u32x4 zero4 = {0u, 0u, 0u, 0u};
    const int main_lane = lane, main_j = j, main_kg = kg;
    auto epilogue = [&](int32_t row0, int32_t col0) __attribute__((always_inline)) {
        // (KTAIL: counted anew and opaque to the optimiser, so that the epilogue's addresses are worked out here, once per
        //  output tile: kept through the main loop they would be spilled, and every reload waits for the copies in flight)
        int lane = main_lane;
        if constexpr (KTAIL) {
            lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
            asm volatile("" : "+v"(lane));
        }
        const int j = KTAIL ? lane & 15 : main_j, kg = KTAIL ? lane >> 4 : main_kg;
        // the loop's MFMAs are asm statements, so the compiler does not know that the accumulators come out of
        // the matrix pipeline: keep the first read of them the documented number of wait states away
        asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
        const int32_t row_end = min(row0 + BM, T);
        const int32_t wrow0 = row0 + wm * TM;        // the wave's rows are wrow0 .. wrow0 + TM - 1
        // ---- the up projection's steps (uniform over the workgroup, the barriers too)
        Walk walk;
        bool up = P && rec[3] > 0;
        for (bool first = true; up; first = false) {
            const unsigned char* ml = lds + MSLICE_OFF;
            if (!first) {                            // (the first step was waited for at the last K tile's barrier)
                wait_vmcnt<0>();
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            }
            const unsigned char* pl = ml + P_OFF + (wm * TM + j) * (RSTEP * 2) + kg * 16;
            u32x4 pv[MB];
            bf16x8 mf[NB];
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) pv[mb] = *reinterpret_cast<const u32x4*>(pl + mb * 16 * (RSTEP * 2));
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) mf[nb] = read_kn(ml, 0, nb, j, kg);
            __builtin_amdgcn_sched_barrier(0);       // (the scalar work of the step, and of the next one, under the reads)
            if (first) first_step(walk, row0, col0);
            // lane (j, kg) holds ranks 8 (kg % 2) .. + 7 of half kg / 2 in both operands
            const Half ha = walk.a, hb = walk.b;
            const int32_t srow0 = row0 + wave_u / WN * TM;           // (wrow0, in a scalar register)
            const bool two = hb.lo != ha.lo;         // the second half is another (later) segment's
            int32_t lo = ha.lo, hi = ha.hi, n = kg < 2 ? ha.n : two ? 0 : hb.n;
            const int32_t lo2 = hb.lo, hi2 = hb.hi, n2 = kg < 2 ? 0 : hb.n;
            const bool mine = (hi > srow0 && lo < srow0 + TM) || (two && hi2 > srow0 && lo2 < srow0 + TM);
            up = next_step(walk, row_end);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();            // everybody has read the step: the region is free
            asm volatile("" ::: "memory");
            if (up) copy_step(walk, row0, col0);
            if (!mine) continue;
            // once per segment, with the ranks of the other cleared in both operands
            for (int again = rfl(two);;) {
                const int nv = min(max(n - 8 * (kg & 1), 0), 8);
                u32x4 km;
#pragma unroll
                for (int w = 0; w < 4; ++w) km[w] = (2 * w < nv ? 0xffffu : 0u) | (2 * w + 1 < nv ? 0xffff0000u : 0u);
                bf16x8 m[NB];
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    union { bf16x8 b; u32x4 u; } cv;
                    cv.b = mf[nb];
                    cv.u &= km;
                    m[nb] = cv.b;
                }
                // The MFMAs are asm statements, which the compiler's hazard pass does not look into: an MFMA must not read a
                // register in the two wait states after a vector ALU instruction has written it, and the masking above is such a
                // write (operands that come straight from a load need nothing).  The statements below order the masking before the
                // wait states and the MFMAs behind them.
                asm volatile("s_nop 1" : "+v"(m[0]), "+v"(m[1]), "+v"(m[2]), "+v"(m[3]), "+v"(m[4]), "+v"(m[5]), "+v"(m[6]), "+v"(m[7]));
                static_for<0, MB>([&](auto mb_c) {
                    constexpr int mb = decltype(mb_c)::value;
                    const int32_t rb = srow0 + mb * 16, row = rb + j;
                    if (hi <= rb || lo >= rb + 16) return;           // wave-uniform
                    bf16x8 pf = as_bf16x8((row >= lo && row < hi) ? (pv[mb] & km) : zero4);
                    asm volatile("s_nop 1" : "+v"(pf));
                    static_for<0, NB>([&](auto nb_c) { mfma_acc<acc_reg(mb, decltype(nb_c)::value)>(m[decltype(nb_c)::value], pf); });
                });
                if (!again) break;
                again = 0;
                lo = lo2;
                hi = hi2;
                n = n2;
                asm volatile("" : "+s"(again), "+s"(lo), "+s"(hi), "+v"(n));      // (opaque to the optimiser, which would make two copies of the loop's body)
            }
        }
        if (P) asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
        // (block_col: a lane with odd kg holds its high four columns in block 2 p and its low four in block 2 p + 1)
        auto pair_order = [&](bf16x8 o) {
            union { bf16x8 b; uint64_t h[2]; } u, v;
            u.b = o;
            v.h[0] = (kg & 1) ? u.h[1] : u.h[0];
            v.h[1] = (kg & 1) ? u.h[0] : u.h[1];
            return v.b;
        };
        // ---- fp32 -> bf16 (one rounding, to nearest even) and the stores.  Blocks 2 p and 2 p + 1 hold this lane's
        //      columns 32 p + 8 kg .. + 7 of token row j.  Non-temporal, so that y / dx do not evict x / dy from the
        //      caches before the rank-r passes read them.
#if LOBRA_GP_STORE == 4
        //      Straight from the accumulators: 16 bytes per lane, 64 contiguous bytes per row and instruction.
        const int32_t orow = wrow0 + j, ocol = col0 + wn * TN + 8 * kg;
        uint16_t* cp = C + size_t(orow) * ldc + ocol;
        static_for<0, MB>([&](auto mb_c) {
            constexpr int mb = decltype(mb_c)::value;
            static_for<0, NB / 2>([&](auto p_c) {
                constexpr int p = decltype(p_c)::value;
                bf16x8 o;
                static_for<0, 8>([&](auto q_c) {     // accumulators (mb, 2 p) and (mb, 2 p + 1) are neighbours
                    constexpr int q = decltype(q_c)::value;
                    o[q] = (__bf16)acc_read<acc_reg(mb, 2 * p) + q>();
                });
                o = pair_order(o);
                __builtin_nontemporal_store(o, reinterpret_cast<bf16x8*>(cp + size_t(16 * mb) * ldc + 32 * p));
            });
        });
#else
        //      Through the wave's quarter of the adapter-slice region (8 KiB, free now), a 64 x 64 block at a time,
        //      so that every store instruction writes whole 128-byte lines (8 rows of them): written 64 bytes at a
        //      time the result costs 40 % more write requests between L2 and memory.  Rows of a block are 128 bytes
        //      apart in LDS, 16-byte chunk c of row r stored at c ^ ((r >> 1) & 7); a wave's LDS operations are
        //      carried out in order, so the reads of a block need no wait for its writes.
        //      (Nobody reads the adapter region any more: the last step's reads are behind a barrier.)
        unsigned char* cs = lds + MSLICE_OFF + wave * 8192;
        static_for<0, 4>([&](auto b_c) {
            constexpr int hm = decltype(b_c)::value / 2, hn = decltype(b_c)::value % 2;
            static_for<0, 4>([&](auto m_c) {
                constexpr int mb = 4 * hm + decltype(m_c)::value;
                static_for<0, 2>([&](auto p_c) {
                    constexpr int p = 2 * hn + decltype(p_c)::value;
                    bf16x8 o;
                    static_for<0, 8>([&](auto q_c) {     // accumulators (mb, 2 p) and (mb, 2 p + 1) are neighbours
                        constexpr int q = decltype(q_c)::value;
                        o[q] = (__bf16)acc_read<acc_reg(mb, 2 * p) + q>();
                    });
                    o = pair_order(o);
                    const int r = 16 * (mb % 4) + j, c = 4 * (p % 2) + kg;
                    *reinterpret_cast<bf16x8*>(cs + r * 128 + ((c ^ swz_row(r)) << 4)) = o;
                });
            });
            static_for<0, 8>([&](auto i_c) {
                const int r = 8 * decltype(i_c)::value + (lane >> 3), pos = lane & 7;
                const bf16x8 o = *reinterpret_cast<const bf16x8*>(cs + r * 128 + (pos << 4));
                uint16_t* dst = C + size_t(wrow0 + 64 * hm + r) * ldc + (col0 + wn * TN + 64 * hn + 8 * (pos ^ swz_row(r)));
#if LOBRA_GP_STORE == 0     // timing variant: only a token store, so that the result is not dead code
                if (decltype(b_c)::value == 0 && decltype(i_c)::value == 0) __builtin_nontemporal_store(o, reinterpret_cast<bf16x8*>(dst));
                else asm volatile("" : : "v"(o));
#elif LOBRA_GP_STORE == 2
                *reinterpret_cast<bf16x8*>(dst) = o;
#else
                __builtin_nontemporal_store(o, reinterpret_cast<bf16x8*>(dst));
#endif
            });
        });
#endif
        // (the accumulators are not cleared here: the first K step of the next tile starts from zero)
    };

    // ---- the stream: K tile g of it sits in stage g & 1 and is copied two K tiles ahead of its use.  The loop
    //      body handles two K tiles, so that the stages are compile-time constants.
    bf16x8 zf[MB], wf[2][NB];
    set_copy_tile(0);
#pragma unroll
    for (int c = 0; c < 2 * NBZ; ++c) dma16(copy_lds_addr(ldsw, c), c < NBZ ? zcur : wcur, c < NBZ ? zvo[c] : wvo[c - NBZ]);
    advance();
#pragma unroll
    for (int c = 0; c < 2 * NBZ; ++c)
        dma16(copy_lds_addr(ldsw + STAGE_BYTES, c), c < NBZ ? zcur : wcur, c < NBZ ? zvo[c] : wvo[c - NBZ]);
    int32_t t_n = 0, t_kt = 0, t_row0, t_col0;       // the compute cursor
    tile_origin(0, t_row0, t_col0);
    load_table(t_row0);
    wait_vmcnt<0>();                                 // the first two K tiles have landed
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int u = 0; u < MB; ++u) read_z(zaddr(0, 0), u, zf);
#pragma unroll
    for (int u = 0; u < NB; ++u) read_w(waddr(0, 0), 0, 0, u, wf[0]);
    // every wave has read the last fragments of this stage, and the copies of the next K tile have landed
    auto tile_barrier = []() __attribute__((always_inline)) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        wait_vmcnt<0>();
        __builtin_amdgcn_s_barrier();
    };
    // The same in the first K tile of an output tile: the 32 stores of the previous tile's epilogue were
    // issued after the copies this barrier is about, and vector memory operations complete in the order they
    // were issued, so the barrier does not have to wait for the stores: they drain under the MFMAs that follow.
    // (The workgroup's very first tile has no stores behind its copies: the prologue waits for them itself.)
    auto tile_barrier_after_stores = []() __attribute__((always_inline)) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        wait_vmcnt<LOBRA_GP_STORES_IN_FLIGHT>();
        __builtin_amdgcn_s_barrier();
    };
    // KTAIL: in front of K step q (0 .. 3) of a pair of K tiles, the fragments' lanes whose 8 k lie beyond K are
    // cleared - in both operands, since what they hold instead is another k's value, perhaps no finite one.
    auto clear_beyond = [&](int q, bf16x8 (&z)[MB], bf16x8 (&w)[NB]) __attribute__((always_inline)) {
        const int32_t rem = K - t_kt * BK;           // 8 .. 120 in the last pair, more before
        if (32 * q + 32 <= rem) return;              // uniform
        const bool in = 32 * q + 8 * kg < rem;
        const bf16x8 zero = as_bf16x8(zero4);
#pragma unroll
        for (int i = 0; i < MB; ++i) z[i] = in ? z[i] : zero;
#pragma unroll
        for (int i = 0; i < NB; ++i) w[i] = in ? w[i] : zero;
    };
    // One K tile in stage STG: K step 0 (fragments in registers) reads the fragments of K step 1 and moves the
    // copy cursor on to the K tile after next; K step 1, once the barrier in its second section is passed,
    // reads the first fragments of the next K tile from the other stage and copies the K tile after next
    // into this one.
    // (copy_c: how the K tile after next is copied; MASK: this K tile may be one of the last pair, see clear_beyond)
    auto ktile = [&](auto stg_c, auto mode_c, auto copy_c, auto mask_c) __attribute__((always_inline)) {
        constexpr int STG = decltype(stg_c)::value;
        constexpr bool MASK = decltype(mask_c)::value;
        if constexpr (MASK) clear_beyond(2 * STG, zf, wf[0]);
        kstep(mode_c, STG, 1, zf, wf[0], wf[1], 0, advance);
        if constexpr (MASK) clear_beyond(2 * STG + 1, zf, wf[1]);
        if constexpr (decltype(mode_c)::value == STEP_FIRST)
            kstep(copy_c, STG ^ 1, 0, zf, wf[1], wf[0], ldsw + uint32_t(STG) * STAGE_BYTES, tile_barrier_after_stores);
        else
            kstep(copy_c, STG ^ 1, 0, zf, wf[1], wf[0], ldsw + uint32_t(STG) * STAGE_BYTES, tile_barrier);
    };
    using yes = std::true_type;
    using no = std::false_type;
    using stage0 = std::integral_constant<int, 0>;
    using stage1 = std::integral_constant<int, 1>;
    for (;;) {
        if (KTAIL && t_kt + 4 >= KT) {               // (uniform) the last pair of K tiles is copied, or multiplied, here
            ktile(stage0{}, step_plain{}, step_copy_tail{}, yes{});
            if (t_kt + 2 == KT) prefetch_adapter(t_row0, t_col0);
            ktile(stage1{}, step_plain{}, step_copy_tail{}, yes{});
        } else {
            if (t_kt == 0) ktile(stage0{}, step_first{}, step_copy{}, no{});
            else ktile(stage0{}, step_plain{}, step_copy{}, no{});
            if (!KTAIL && t_kt + 2 == KT) prefetch_adapter(t_row0, t_col0);   // waited for at the tile barrier that follows
            ktile(stage1{}, step_plain{}, step_copy{}, no{});
        }
        t_kt += 2;
        if (t_kt == KT) {                            // uniform: an output tile is complete
            epilogue(t_row0, t_col0);
            t_kt = 0;
            if (++t_n == my_tiles) break;
            tile_origin(t_n, t_row0, t_col0);
            load_table(t_row0);
            // the first fragments of the next output tile once more: holding 64 registers of them through
            // the epilogue costs more (spills) than these sixteen reads
#pragma unroll
            for (int u = 0; u < MB; ++u) read_z(zaddr(0, 0), u, zf);
#pragma unroll
            for (int u = 0; u < NB; ++u) read_w(waddr(0, 0), 0, 0, u, wf[0]);
        }
    }
    // copies past the end are still in flight: they must have landed before the LDS is given back
    wait_vmcnt<0>();
}

namespace {
template <bool W_KN>
hipError_t launch_persistent(const PlanDev& pd, const void* Z, const void* W, const void* P, const void* M, void* C,
                             int32_t K, int32_t N, int32_t ldw, int32_t ldc, int32_t nproj, int32_t proj,
                             int32_t tiles_m, int32_t tiles_n, int32_t gm, hipStream_t st)
{
    // once per device: the kernel needs more dynamic LDS than the default limit; one workgroup per compute unit
    static std::atomic<int32_t> cus[64];
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    int32_t ncu = cus[dev].load(std::memory_order_acquire);
    if (ncu == 0) {
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(&LOBRA_GP_KERNEL<W_KN>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
        if (e != hipSuccess) return e;
        int n = 0;
        e = hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess) return e;
        ncu = n > 0 ? n : 1;
        cus[dev].store(ncu, std::memory_order_release);
    }
    const int64_t ntiles = int64_t(tiles_m) * tiles_n;
    const int32_t cpx = ncu >= 8 ? ncu / 8 : 1;
    const int32_t tpw = LOBRA_GP_TPW;
    const int64_t xmax = (ntiles + 7) / 8;                                    // tiles of the fullest XCD
    const int64_t rounds = (xmax + int64_t(cpx) * tpw - 1) / (int64_t(cpx) * tpw);
    const int64_t wgs = ntiles <= 8 * int64_t(cpx) ? ntiles : 8 * rounds * cpx;   // few tiles: one workgroup each
    LOBRA_GP_KERNEL<W_KN><<<dim3(uint32_t(wgs)), 64 * NW, LDS_BYTES, st>>>(
        pd, (const uint16_t*)Z, (const uint16_t*)W, (const uint16_t*)P, (const uint16_t*)M, (uint16_t*)C,
        K, N, ldw, ldc, nproj, proj, tiles_m, tiles_n, gm, cpx, tpw, pd.gemm_tile_seg, pd.cseg_off, pd.cseg_task, pd.rank_off);
    return hipGetLastError();
}
}  // namespace

hipError_t LOBRA_GP_HOST(const PlanDev& pd, bool transW, const void* Z, const void* W, const void* P,
                           const void* M, void* C, int32_t K, int32_t N, int32_t ldw, int32_t ldc, int32_t nproj,
                           int32_t proj, int32_t tiles_m, int32_t tiles_n, int32_t gm, hipStream_t st)
{
#if !LOBRA_GP_KTAIL
    if (K % (2 * BK) != 0)
        return gemm_persistent_ktail(pd, transW, Z, W, P, M, C, K, N, ldw, ldc, nproj, proj, tiles_m, tiles_n, gm, st);
#endif
    if (transW) return launch_persistent<false>(pd, Z, W, P, M, C, K, N, ldw, ldc, nproj, proj, tiles_m, tiles_n, gm, st);
    return launch_persistent<true>(pd, Z, W, P, M, C, K, N, ldw, ldc, nproj, proj, tiles_m, tiles_n, gm, st);
}

}  // namespace lobra

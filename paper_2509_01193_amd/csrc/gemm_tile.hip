// Tiled bf16 MFMA GEMM for gfx950 with the LoRA up projection fused into its epilogue, for products of few output tiles and,
// where K is no multiple of 128, batches of short segments; the others run on the persistent kernel (gemm_persistent.hip) and
// the register-staged one (gemm_staged.hip), see choose_gemm.
//     C[T, N] = Z[T, K] * op(W) + P[T, r] * M_t[r, N]
// forward : Z = x,  op(W) = W   (W stored [K][N], N fastest),  P = s_t A_t x_i,  M = B  -> y
// backward: Z = dy, op(W) = W^T (W stored [N][K], K fastest),  P = s_t B_t dy_i, M = A  -> dx
// (paper section 2.1: X W + X (down)(up); section 1: one shared base product for the fused batch,
// a per-task adapter product on top of it).
//
// One workgroup per TM x TN output tile, WM x WN waves, K in steps of 64 through a ring of STAGES LDS slots that
// direct global -> LDS copies fill (no registers, no ds_write).  Blocks of v_mfma_f32_16x16x32_bf16 with fp32
// accumulators; the MFMA "A" operand is fed from W and the "B" operand from Z, so a lane ends up with four
// consecutive output columns of one row.  Sums run over ascending k in steps of 32 like the other kernels',
// so all give the same bits.
//
// What bounds it: inside a compute unit, the copies (64 bytes a cycle) and the LDS reads of a 128 x 128 tile take as
// long as its MFMAs (512 cycles per K tile each), so nothing may wait for anything else.  The order of a K step is
// pinned (sched_barrier): every fragment read and every copy goes out behind an MFMA, a K tile's copies are dealt over
// two K steps, and the only waits are one counted vmcnt and one barrier per K tile.  Left to the compiler, which put the
// copies and the reads in front of the MFMAs, the same kernel took 61 instead of 39 us (x [1000, 4096] times W [4096, 4096],
// 256 tiles of 128 x 128; without MFMAs 31 us, without fragment reads 34, without copies 36).
//
// K may be any multiple of 8 and T, N anything from 8 columns up: rows and columns beyond the edge repeat the last
// valid one (what they produce is never stored), chunks beyond K repeat the last valid chunk and both operands'
// fragments are cleared in registers, in the last K tile only.
//
// LDS layouts
//   Z tile, and the W tile when K is fastest (backward): [rows][64 k], 128 bytes per row, 16-byte chunk c of a row
//       stored at c ^ swz_row(row).
//   W tile when N is fastest (forward), adapter slice: [k][TN n], chunk c of k-row k stored at c ^ swz_kn<TN>(k); the
//       MFMA operand (8 consecutive k of one column) is gathered with two ds_read_b64_tr_b16.
//   C staging in the epilogue: per wave [rows][cols + 8] bf16, written back with non-temporal stores.
#include <algorithm>
#include <atomic>
#include <cstddef>

#include "gemm_common.h"
#include "kernels.h"
#include "shrink_ring.h"

namespace lobra {

using namespace gemm;

static_assert(kGemmKTile == BK && kGemmTiles[0].tm == BM && kGemmTiles[0].tn == BN, "the plan's choice is about these kernels");

namespace {

// Swizzle of a [k][TN n] tile.  A transpose read's two 16-lane groups of a pass touch 32 bytes in each of the k rows
// k0 .. k0 + 3 and k0 + 8 .. k0 + 11: eight rows, whose pieces have to fall into the eight 32-byte parts of the 256
// bytes that the banks span.  Rows of 256 bytes and more all start at bank 0, so three bits of k pick the part; rows
// of 128 bytes start at bank 0 or 32 by their lowest bit, so two bits of k pick one of four.
template <int TN> __device__ __forceinline__ int swz_kn(int k)
{
    if constexpr (TN >= 128) return kn_swz(k);
    else return (((k >> 1) & 1) << 2) | (((k >> 3) & 1) << 1);
}

// What a tile's rows belong to, in LDS behind the ring: the segments that cross the tile (at most one per row), each with
// its first token, task and rank window; which of them are the first of their task; and per row the first segment of its
// task (-1: no adapter).
template <int TM> struct alignas(16) TileTable {
    int32_t lo[TM], task[TM], r0[TM], r[TM], row[TM];
    uint64_t firsts[(TM + 63) / 64];
};

// A set of segments of a tile, in scalar registers.
template <int TM> struct TaskSet {
    static_assert(TM <= 128, "two words");
    uint64_t a, b;
    static __device__ __forceinline__ uint64_t uniform(uint64_t v)
    {
        const uint32_t lo = __builtin_amdgcn_readfirstlane(uint32_t(v)), hi = __builtin_amdgcn_readfirstlane(uint32_t(v >> 32));
        return (uint64_t(hi) << 32) | lo;
    }
    __device__ __forceinline__ void load(const uint64_t* w)
    {
        a = uniform(w[0]);
        b = TM > 64 ? uniform(w[TM > 64 ? 1 : 0]) : 0;
    }
    __device__ __forceinline__ bool empty() const { return (a | b) == 0; }
    __device__ __forceinline__ int32_t lowest() const       // -1: empty
    {
        return a ? __builtin_ctzll(a) : (b ? 64 + __builtin_ctzll(b) : -1);
    }
    __device__ __forceinline__ void remove_lowest()
    {
        if (a) a &= a - 1;
        else b &= b - 1;
    }
    __device__ __forceinline__ void remove(const TaskSet& o) { a &= ~o.a, b &= ~o.b; }
};

template <int TM, int TN, int WN, int STAGES> constexpr int ring_bytes()
{
    constexpr int loop = STAGES * (TM + TN) * BK * 2;
    static_assert(loop >= TM * (TN + 8 * WN) * 2, "all waves' C staging fits the ring");
    static_assert(loop >= LOBRA_MAX_RANK * TN * 2, "an adapter slice of any rank fits the ring");
    return loop;
}

// Rank rows (whole groups of eight) of adapter slices that fit behind ring and table, with OCC workgroups on a compute unit: up to 96.
template <int TM, int TN, int WN, int STAGES, int OCC> constexpr int ahead_rows()
{
    const int left = 160 * 1024 / OCC - ring_bytes<TM, TN, WN, STAGES>() - int(sizeof(TileTable<TM>));
    return std::min(left / (TN * 2) / 8 * 8, 96);
}

template <bool W_KN, int TM, int TN, int WM, int WN, int STAGES, int AHEAD>
__device__ __forceinline__
void tile_body(const PlanDev& pd, const uint16_t* __restrict__ Z, const uint16_t* __restrict__ W,
               const uint16_t* __restrict__ P, const uint16_t* __restrict__ M,
               uint16_t* __restrict__ C, int32_t K, int32_t N, int32_t ldw, int32_t ldc,
               int32_t nproj, int32_t proj, int32_t tiles_m, int32_t tiles_n, int32_t GM, int32_t splits,
               float* __restrict__ part, int32_t wg, unsigned char* lds)
{
    // splits > 1: that many workgroups per tile share the K tiles, and one more has the adapter term (if P): in the time
    // that its chain of table reads, copies and products takes, the others are done with theirs.  Their fp32 sums go to
    // part [splits (+ 1)][T][N]; gemm_add_kernel adds them and writes C.  (C = NULL: also with one split.)
    // ldc: row pitch of C.  nproj > 1: this launch is projection `proj` of a fused shared-input
    // call: of every task's rank rows (in M) and rank columns (in P) only the window
    // [proj r, (proj + 1) r) takes part, r = the task's stacked rank / nproj.  proj < 0: the launch
    // covers all projections (N = nproj * pd.dg, pd.dg a multiple of the tile width) and a tile takes
    // the projection its columns lie in; M is then the compact [R_tot][pd.dg] array.
    constexpr int NW = WM * WN;
    constexpr int WTM = TM / WM, WTN = TN / WN;     // wave tile
    constexpr int MB = WTM / 16, NB = WTN / 16;     // 16 x 16 blocks per wave
    constexpr int ZT = TM * BK * 2, STAGE = (TM + TN) * BK * 2;
    constexpr int ZC = TM / 8 / NW, WC = TN / 8 / NW, CPW = ZC + WC;   // 1 KiB copies per wave and K tile
    constexpr int CR = TN / 8, RPC = 64 / CR;       // [k][n] tile: 16-byte chunks per k row, k rows per copy
    constexpr int CS_PITCH = WTN + 8;
    static_assert(ZC * 8 * NW == TM && WC * 8 * NW == TN && RPC * CR == 64, "whole copies");
    static_assert(STAGES > 2, "a K tile's copies are dealt over two K steps");

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    // MFMA 16x16x32 lanes: j = row of the "B" operand (a token) and of the result, kg = group of 8 k
    // (operands) or of 4 result columns
    const int j = lane & 15, kg = lane >> 4;
    const int32_t T = pd.T;

    // ---- workgroup -> tile: consecutive ids go to different XCDs, so give each XCD a contiguous
    //      range of the tile order; inside it, GM tile-rows share one sweep over the tile-columns.
    int32_t row0, col0, split;
    {
        const int32_t per = splits + (splits > 1 && P ? 1 : 0);
        const int32_t wid = xcd_contiguous(wg, tiles_m * tiles_n * per);
        const int32_t id = wid / per;
        split = wid - id * per;
        const int32_t group = id / (GM * tiles_n);
        const int32_t first_m = group * GM;
        const int32_t gsz = min(tiles_m - first_m, GM);
        const int32_t in = id - group * GM * tiles_n;
        row0 = (first_m + in % gsz) * TM;
        col0 = in / gsz * TN;
    }

    // ---- copies.  Block b (1 KiB) of a [rows][64 k] tile holds rows 8 b .. 8 b + 7, of a [k][n] tile the k rows
    //      RPC b ..; wave w moves blocks w, w + NW, ...; the swizzle is applied to the address a lane fetches from.
    const int32_t sg0 = P ? pd.rowblk_seg[row0 / kRowBlock] : 0;     // (in front of the copies: a scalar load)
    const uint32_t lds0 = uint32_t(uintptr_t((__attribute__((address_space(3))) unsigned char*)lds));
    const unsigned char* zbase = reinterpret_cast<const unsigned char*>(Z + size_t(row0) * K);
    const unsigned char* wbase = reinterpret_cast<const unsigned char*>(W_KN ? W + col0 : W + size_t(col0) * ldw);
    const size_t wstep = W_KN ? size_t(BK) * ldw * 2 : size_t(BK) * 2;
    uint32_t zvo[ZC], wvo[WC];
#pragma unroll
    for (int c = 0; c < ZC; ++c) {
        const int row = 8 * (wave + NW * c) + lane / 8;
        zvo[c] = (uint32_t(min(row, T - 1 - row0)) * uint32_t(K) + 8u * ((lane % 8) ^ swz_row(row))) * 2u;
    }
#pragma unroll
    for (int c = 0; c < WC; ++c) {
        if (W_KN) {
            const int krow = RPC * (wave + NW * c) + lane / CR;
            wvo[c] = (uint32_t(krow) * uint32_t(ldw) + uint32_t(min(8 * ((lane % CR) ^ swz_kn<TN>(krow)), N - 8 - col0))) * 2u;
        } else {
            const int row = 8 * (wave + NW * c) + lane / 8;
            wvo[c] = (uint32_t(min(row, N - 1 - col0)) * uint32_t(ldw) + 8u * ((lane % 8) ^ swz_row(row))) * 2u;
        }
    }
    // this workgroup's K tiles, and the k of a partial last one (0: none)
    const int32_t KA = (K + BK - 1) / BK, kt0 = KA * split / splits;
    const int32_t KT = split < splits ? KA * (split + 1) / splits - kt0 : 0;
    const int32_t ktail = split + 1 == splits ? K % BK : 0;
    const unsigned char *zcur = zbase + size_t(kt0) * (BK * 2), *wcur = wbase + size_t(kt0) * wstep;   // K tile the next copies fetch
    if (splits > 1 && split < splits) P = nullptr;
    auto copy = [&](auto c_c, uint32_t la) __attribute__((always_inline)) {      // copy c of a whole K tile
        constexpr int c = decltype(c_c)::value;
        if constexpr (c < ZC) dma16(la + NW * c * 1024, zcur, zvo[c]);
        else dma16(la + ZT + NW * (c - ZC) * 1024, wcur, wvo[c - ZC]);
    };
    auto next_copy_tile = [&]() __attribute__((always_inline)) {
        zcur += BK * 2;
        wcur += wstep;
    };
    auto copy_tail = [&](uint32_t la) {             // the partial last K tile: chunks beyond K repeat the last one
#pragma unroll
        for (int c = 0; c < ZC; ++c) {
            const int ch = (lane % 8) ^ swz_row(8 * (wave + NW * c) + lane / 8);
            dma16(la + NW * c * 1024, zcur, zvo[c] - 2u * uint32_t(max(8 * ch - (ktail - 8), 0)));
        }
#pragma unroll
        for (int c = 0; c < WC; ++c) {
            uint32_t vo;
            if (W_KN) {
                const int krow = RPC * (wave + NW * c) + lane / CR;
                vo = wvo[c] - 2u * uint32_t(max(krow - (ktail - 1), 0)) * uint32_t(ldw);
            } else {
                const int ch = (lane % 8) ^ swz_row(8 * (wave + NW * c) + lane / 8);
                vo = wvo[c] - 2u * uint32_t(max(8 * ch - (ktail - 8), 0));
            }
            dma16(la + ZT + NW * c * 1024, wcur, vo);
        }
    };

    // ---- operand fragments of K step ks (32 k) of a slot
    auto read_z = [&](const unsigned char* st, int ks, int mb) __attribute__((always_inline)) {
        const int row = wm * WTM + mb * 16 + j;
        return *reinterpret_cast<const bf16x8*>(st + row * (BK * 2) + (((4 * ks + kg) ^ swz_row(j)) << 4));
    };
    auto read_kn = [&](const unsigned char* base, int krow0, int nb, int kg) __attribute__((always_inline)) {
        const int krow = krow0 + 8 * kg + (j >> 2);
        const int n = wn * WTN + nb * 16 + 4 * (j & 3);
        return tr_pair(base + krow * (TN * 2) + (((n >> 3) ^ swz_kn<TN>(krow)) << 4) + (n & 7) * 2, TN * 2);
    };
    auto read_w = [&](const unsigned char* st, int ks, int nb) __attribute__((always_inline)) {
        if (W_KN) return read_kn(st + ZT, 32 * ks, nb, kg);
        const int row = wn * WTN + nb * 16 + j;
        return *reinterpret_cast<const bf16x8*>(st + ZT + row * (BK * 2) + (((4 * ks + kg) ^ swz_row(j)) << 4));
    };
    const bf16x8 zero8 = as_bf16x8(u32x4{0u, 0u, 0u, 0u});
    // lane group kg holds k 32 ks + 8 kg .. + 7 of the tile in both operands
    auto clear_tail = [&](int ks, bf16x8 (&zf)[MB], bf16x8 (&wf)[NB]) __attribute__((always_inline)) {
        const bool in = 32 * ks + 8 * kg < ktail;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) zf[mb] = in ? zf[mb] : zero8;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) wf[nb] = in ? wf[nb] : zero8;
    };

    // acc[mb][nb][v]: token row mb 16 + j of the wave tile, column nb 16 + 4 kg + v
    f32x4 acc[MB][NB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int jj = 0; jj < NB; ++jj) acc[i][jj] = f32x4{0.f, 0.f, 0.f, 0.f};
    // One K step: MB NB MFMAs on (zf, wf) with the reads of the fragments (zn, wn_) of K step rks of the slot at rst
    // and (COPY) the CPW copies of a K tile into the slot at la dealt evenly behind them, in this order.
    auto kstep = [&](auto read_c, auto copy_c, const bf16x8 (&zf)[MB], const bf16x8 (&wf)[NB], const unsigned char* rst, int rks,
                     bf16x8 (&zn)[MB], bf16x8 (&wn_)[NB], uint32_t la) __attribute__((always_inline)) {
        constexpr bool READ = decltype(read_c)::value;
        constexpr int C0 = decltype(copy_c)::value >> 8, NC = (decltype(copy_c)::value & 255) - C0;
        constexpr int NM = MB * NB, NR = READ ? MB + NB : 0;
        static_for<0, NM>([&](auto q_c) {
            constexpr int q = decltype(q_c)::value, mb = q / NB, nb = q % NB;
            acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[nb], zf[mb], acc[mb][nb], 0, 0, 0);
            static_for<q * NR / NM, (q + 1) * NR / NM>([&](auto i_c) {
                constexpr int i = decltype(i_c)::value;
                if constexpr (i < NB) wn_[i] = read_w(rst, rks, i);
                else zn[i - NB] = read_z(rst, rks, i - NB);
            });
            static_for<q * NC / NM, (q + 1) * NC / NM>([&](auto i_c) { copy(std::integral_constant<int, C0 + decltype(i_c)::value>{}, la); });
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    using yes = std::true_type;
    using no = std::false_type;
    // copies [c0, c1) of a K tile, as kstep's argument
    constexpr int CH = CPW / 2;
    using none = std::integral_constant<int, 0>;
    using half0 = std::integral_constant<int, CH>;
    using half1 = std::integral_constant<int, (CH << 8) | CPW>;

    const int32_t pj = proj >= 0 ? proj : col0 / pd.dg;          // this tile's projection
    const int32_t mcol0 = proj >= 0 ? 0 : pj * pd.dg;            // first column of that projection
    const int32_t mpitch = proj >= 0 ? N : pd.dg;                // row pitch of M
    TileTable<TM>& tab = *reinterpret_cast<TileTable<TM>*>(lds + STAGES * STAGE);
    auto lds_barrier = []() __attribute__((always_inline)) {     // (bare: a fence would wait for the copies in flight)
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    // ---- main loop.  A K tile's second K step is multiplied behind the barrier that hands its slot back: by then
    //      its fragments are in registers, so the slot can be refilled and the next tile's first fragments are read
    //      while the matrix cores work.
    const uint32_t la0 = lds0 + wave * 1024;
    const int32_t KF = ktail ? KT - 1 : KT;          // whole K tiles
    for (int s = 0; s < STAGES; ++s) {
        if (s < KF) static_for<0, CPW>([&](auto c_c) { copy(c_c, la0 + s * STAGE); });
        else if (s < KT) copy_tail(la0 + s * STAGE);
        next_copy_tile();
        // the segments from the tile's first row on, one a lane, behind the first K tile's copies: the chain of reads through
        // registers in front of them or behind all of them kept the main loop waiting for one or the other
        if (s == 0 && P && wave < TM / 64) {
            const uint32_t to = lds0 + STAGES * STAGE + wave * 256, at = 4u * uint32_t(min(sg0 + wave * 64 + lane, pd.nseg - 1));
            dma4(to + offsetof(TileTable<TM>, lo), pd.cseg_off, at);
            dma4(to + offsetof(TileTable<TM>, task), pd.cseg_task, at);
            dma4(to + offsetof(TileTable<TM>, r0), cseg_rank(pd), at);
            dma4(to + offsetof(TileTable<TM>, r), cseg_rank(pd) + pd.nseg, at);
        }
    }
    bf16x8 za[MB], wa[NB], zb[MB], wb[NB];
    if (KT >= STAGES) wait_vmcnt<(STAGES - 1) * CPW>();
    else wait_vmcnt<0>();
    lds_barrier();
    // What this tile's rows belong to, worked out while further K tiles are on their way.  (A batch of decoding requests has a
    // segment per token; one chain of table reads and one staging of adapter rows per segment, behind the main loop, took
    // longer than the product: 39 us where this takes 24, 40 one-token segments of eight tasks, K = N = 4096.)
    if (P) {
        const int32_t sg = sg0 + tid;
        int32_t t = -1;
        if (tid < TM) {
            const int32_t lo = tab.lo[tid];
            const bool in = sg < pd.nseg && lo < min(row0 + TM, T);
            t = in ? tab.task[tid] : -1;
            const int32_t r = t >= 0 ? (nproj == 1 ? tab.r[tid] : tab.r[tid] / nproj) : 0;
            if (!in) tab.lo[tid] = 0x7fffffff;
            tab.task[tid] = t;
            tab.r0[tid] += pj * r;
            tab.r[tid] = r;
        }
        lds_barrier();
        // the task of thread's row, then the first segment of that task, and whether the thread's own segment is such a first (the
        // table is read eight segments at a time, all threads the same; what lies beyond the last segment has task -1)
        int32_t row_task = -1, row_first = TM, first = TM;
        auto segments = [&](auto&& f) __attribute__((always_inline)) {
            for (int32_t i = 0; i < TM && tab.lo[i] != 0x7fffffff; i += 8) {         // (uniform)
                const int4 a = *reinterpret_cast<const int4*>(&tab.task[i]), b = *reinterpret_cast<const int4*>(&tab.task[i + 4]);
                const int32_t e[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
                f(i, e);
            }
        };
        if (tid < TM) {
            segments([&](int32_t i, const int32_t (&e)[8]) {
                const int4 a = *reinterpret_cast<const int4*>(&tab.lo[i]), b = *reinterpret_cast<const int4*>(&tab.lo[i + 4]);
                const int32_t lo[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (lo[u] <= row0 + tid) row_task = e[u];
            });
            segments([&](int32_t i, const int32_t (&e)[8]) {
#pragma unroll
                for (int u = 7; u >= 0; --u) {
                    if (e[u] == t) first = min(first, i + u);
                    if (e[u] == row_task) row_first = min(row_first, i + u);
                }
            });
            tab.row[tid] = (row0 + tid < T && row_task >= 0) ? row_first : -1;
        }
        const uint64_t firsts = __ballot(t >= 0 && first == tid);
        if (wave < (TM + 63) / 64 && lane == 0) tab.firsts[wave] = firsts;
        lds_barrier();
    }
    // ---- fused up projection: for every task with rows in this tile, ceil(r_t / 32) extra K steps
    //      acc += M_t^T[:, cols] * P[rows, :]^T with the rows of other tasks masked to zero.  The M_t slices [r_t][TN cols] are
    //      copied to LDS in the [k][n] layout and gathered with the transpose read; rows of a slice from r_t up to the next
    //      multiple of 8 repeat row r_t - 1, and what lies beyond r_t is cleared in registers.  P comes straight from global
    //      memory, 16 bytes per lane and rank step.  The first step's P and the slices of as many tasks as fit AHEAD rank rows
    //      behind the table are fetched some K tiles before the main loop ends (prepare_up); further slices go into the ring
    //      behind it, as many at a time as fit.
    //      The loops over tasks and their barriers are uniform over the workgroup.
    //      (With the table's chain of reads waiting for all of the first copies, and slices and P fetched behind the main loop,
    //      x [1000, 4096] times W [4096, 4096] with four tasks of rank 16 took 41.4 us, 5 more than without adapters, like this
    //      39.0; x [1108, 1088] W [1088, 6400] with its projection 26.2 -> 25.2.)
    constexpr int ROWS = STAGES * STAGE / (TN * 2);
    constexpr int AHEAD_TILES = AHEAD ? 4 : 0;       // (with the ring's: so many K tiles in front of the end)
    unsigned char* const ahead = lds + STAGES * STAGE + int(sizeof(TileTable<TM>));
    const u32x4 zero4 = {0u, 0u, 0u, 0u};
    int32_t of[MB], rw[MB];                          // first segment and rank of the row's task
    u32x4 pv[MB], pn[MB];                            // this rank step's P fragments and the next one's
    // the P fragments of rank step s: lane (j, kg) holds the ranks 32 s + 8 kg .. + 7 of token row j of each 16-row
    // block; groups that start beyond r_t hold padding, or another projection's ranks, and are not read
    auto load_p = [&](int32_t s) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const int32_t row = min(row0 + wm * WTM + mb * 16 + j, T - 1), k = 32 * s + 8 * kg;
            pn[mb] = k < rw[mb] ? *reinterpret_cast<const u32x4*>(P + size_t(row) * pd.r_pad + pj * rw[mb] + k) : zero4;
        }
    };
    // rank and first rank row of segment i, out of the lanes' registers
    constexpr int SEGW = (TM + 63) / 64;
    int32_t lane_r[SEGW], lane_r0[SEGW];
    auto of_segment = [&](const int32_t (&v)[SEGW], int32_t i) __attribute__((always_inline)) {
        return __builtin_amdgcn_readlane(v[SEGW > 1 && i >= 64 ? SEGW - 1 : 0], i & 63);
    };
    TaskSet<TM> left, batch;                         // the tasks whose slices are still to be copied; those copied last
    auto copy_slices = [&](uint32_t to, int32_t room) {              // of as many of those left as fit
        batch = left;
        int32_t rows = 0;
        for (int32_t i = left.lowest(); i >= 0; i = left.lowest()) {
            const int32_t r = of_segment(lane_r, i), rp = (r + 7) & ~7;
            if (rows + rp > room) break;
            const unsigned char* mbase = reinterpret_cast<const unsigned char*>(M + size_t(of_segment(lane_r0, i)) * mpitch + (col0 - mcol0));
            for (int32_t c = wave; c < rp / RPC; c += NW) {
                const int krow = RPC * c + lane / CR;
                dma16(to + rows * (TN * 2) + c * 1024, mbase,
                      (uint32_t(min(krow, r - 1)) * uint32_t(mpitch) + uint32_t(min(8 * ((lane % CR) ^ swz_kn<TN>(krow)), N - 8 - col0))) * 2u);
            }
            rows += rp;
            left.remove_lowest();
        }
        batch.remove(left);
    };
    auto prepare_up = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            of[mb] = tab.row[wm * WTM + mb * 16 + j];
            rw[mb] = of[mb] >= 0 ? tab.r[of[mb]] : 0;
        }
        load_p(0);
#pragma unroll
        for (int w = 0; w < SEGW; ++w) lane_r[w] = tab.r[64 * w + lane % TM], lane_r0[w] = tab.r0[64 * w + lane % TM];
        left.load(tab.firsts);
        // (vector memory operations complete in order, so the main loop's counted waits, which are about copies issued before
        //  or after these, wait for no less than they did)
        copy_slices(lds0 + STAGES * STAGE + int(sizeof(TileTable<TM>)), AHEAD);
    };
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) wa[nb] = read_w(lds, 0, nb);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) za[mb] = read_z(lds, 0, mb);
    int32_t kt = 0, slot = 0;
    const int32_t steady = KF - STAGES;              // K tiles behind which a whole K tile is still to be copied
    uint32_t pla = 0;
    auto body = [&](auto h_c) __attribute__((always_inline)) {
        kstep(yes{}, h_c, za, wa, lds + slot * STAGE, 1, zb, wb, pla);
        if constexpr (decltype(h_c)::value != 0) next_copy_tile();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        wait_vmcnt<(STAGES - 2) * CPW>();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        const int32_t ns = slot + 1 == STAGES ? 0 : slot + 1;
        pla = la0 + slot * STAGE;
        kstep(yes{}, half0{}, zb, wb, lds + ns * STAGE, 0, za, wa, pla);
        slot = ns;
    };
    if (steady > 0) {
        body(none{});
        for (kt = 1; kt < steady - AHEAD_TILES; ++kt) body(half1{});
    }
    if (P) prepare_up();
    if constexpr (AHEAD > 0)
        for (; kt < steady; ++kt) body(half1{});
    for (; kt < KT; ++kt) {                          // the last STAGES K tiles, and the partial one
        const bool tail = ktail != 0 && kt + 1 == KT;           // uniform
        if (tail) clear_tail(0, za, wa);
        if (steady > 0 && kt == steady) {
            kstep(yes{}, half1{}, za, wa, lds + slot * STAGE, 1, zb, wb, pla);
            next_copy_tile();
        } else {
            kstep(yes{}, none{}, za, wa, lds + slot * STAGE, 1, zb, wb, 0);
        }
        if (tail) clear_tail(1, zb, wb);
        const int32_t ns = slot + 1 == STAGES ? 0 : slot + 1;
        if (kt + 1 < KT) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            wait_vmcnt<0>();
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            if (kt + STAGES < KT) copy_tail(la0 + slot * STAGE);
            kstep(yes{}, none{}, zb, wb, lds + ns * STAGE, 0, za, wa, 0);
        } else {
            kstep(no{}, none{}, zb, wb, lds, 0, za, wa, 0);
        }
        slot = ns;
    }

    // ---- the up projection's steps
    if (P) {
        const int32_t nks = (pd.r_max / nproj + 31) >> 5;            // rank steps of the widest window (uniform)
        const unsigned char* at = ahead;
        // (with two K tiles and more the last barrier is behind a wait for all that was copied ahead)
        if (KT < 2) {
            wait_vmcnt<0>();
            lds_barrier();
        }
        for (;;) {
            if (!batch.empty())
                for (int32_t s = 0; s < nks; ++s) {
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb) pv[mb] = pn[mb];
                    if (nks > 1) load_p(s + 1 < nks ? s + 1 : 0);
                    const unsigned char* slice = at;
                    TaskSet<TM> todo = batch;
                    for (int32_t i = todo.lowest(); i >= 0; i = todo.lowest()) {
                        todo.remove_lowest();
                        const int32_t r = of_segment(lane_r, i);
                        bool mine[MB], some = false; // wave-uniform: a row of this block is the task's
#pragma unroll
                        for (int mb = 0; mb < MB; ++mb) {
                            mine[mb] = __ballot(of[mb] == i) != 0;
                            some |= mine[mb];
                        }
                        if (some && 32 * s < r) {
                            const int nv = min(max(r - 32 * s - 8 * kg, 0), 8);
                            const int kgs = min(kg, ((r - 32 * s + 7) >> 3) - 1);      // (groups beyond the slice read its last one)
                            u32x4 km;
#pragma unroll
                            for (int w = 0; w < 4; ++w) km[w] = (2 * w < nv ? 0xffffu : 0u) | (2 * w + 1 < nv ? 0xffff0000u : 0u);
                            bf16x8 wf[NB];
#pragma unroll
                            for (int nb = 0; nb < NB; ++nb) {
                                union { bf16x8 b; u32x4 u; } cv;
                                cv.b = read_kn(slice, 32 * s, nb, kgs);
                                cv.u &= km;
                                wf[nb] = cv.b;
                            }
#pragma unroll
                            for (int mb = 0; mb < MB; ++mb) {
                                if (!mine[mb]) continue;
                                const bf16x8 pf = as_bf16x8(of[mb] == i ? pv[mb] : zero4);
#pragma unroll
                                for (int nb = 0; nb < NB; ++nb)
                                    acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[nb], pf, acc[mb][nb], 0, 0, 0);
                            }
                        }
                        slice += ((r + 7) & ~7) * (TN * 2);
                    }
                }
            if (left.empty()) break;
            lds_barrier();                           // everybody is done with what the ring held before
            copy_slices(lds0, ROWS);
            at = lds;
            wait_vmcnt<0>();
            lds_barrier();
        }
    }
    if (splits > 1 || !C) {                         // the sums as they are, 16 bytes per lane
        float* dst = part + size_t(split) * T * N;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const int32_t row = row0 + wm * WTM + mb * 16 + j;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const int32_t col = col0 + wn * WTN + nb * 16 + 4 * kg;
                if (row < T && col < N) *reinterpret_cast<f32x4*>(dst + size_t(row) * N + col) = acc[mb][nb];
            }
        }
        return;
    }
    __syncthreads();                                // the C staging below reuses the same LDS

    // ---- epilogue: fp32 -> bf16, stage the wave's block in LDS, store 16 bytes per lane
    {
        unsigned char* cs = lds + wave * (WTM * CS_PITCH * 2);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                bf16x4 o;
#pragma unroll
                for (int q = 0; q < 4; ++q) o[q] = (__bf16)acc[mb][nb][q];
                const int m = mb * 16 + j, n = nb * 16 + 4 * kg;
                *reinterpret_cast<bf16x4*>(cs + (m * CS_PITCH + n) * 2) = o;
            }
        // (the wave's own block: its LDS operations are carried out in order)
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        constexpr int CPR = WTN / 8;                 // 16-byte chunks per row of the wave tile
        constexpr int RPI = 64 / CPR;                // rows per store instruction
        const int cchunk = lane % CPR, rsub = lane / CPR;
        const int32_t col = col0 + wn * WTN + cchunk * 8;
#pragma unroll 4
        for (int i = 0; i < WTM / RPI; ++i) {
            const int m = i * RPI + rsub;
            const int32_t row = row0 + wm * WTM + m;
            const u32x4 v = *reinterpret_cast<const u32x4*>(cs + (m * CS_PITCH + cchunk * 8) * 2);
            if (row < T && col < N) __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(C + size_t(row) * ldc + col));
        }
    }
}

}  // namespace

template <bool W_KN, int TM, int TN, int WM, int WN, int STAGES, int OCC>
__global__ __launch_bounds__(64 * WM * WN, OCC * WM * WN / 4)
void gemm_tile_kernel(PlanDev pd, const uint16_t* __restrict__ Z, const uint16_t* __restrict__ W,
                      const uint16_t* __restrict__ P, const uint16_t* __restrict__ M,
                      uint16_t* __restrict__ C, int32_t K, int32_t N, int32_t ldw, int32_t ldc,
                      int32_t nproj, int32_t proj, int32_t tiles_m, int32_t tiles_n, int32_t GM, int32_t splits,
                      float* __restrict__ part)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    tile_body<W_KN, TM, TN, WM, WN, STAGES, ahead_rows<TM, TN, WN, STAGES, OCC>()>(pd, Z, W, P, M, C, K, N, ldw, ldc, nproj, proj, tiles_m, tiles_n, GM, splits, part,
                                            int32_t(blockIdx.x), lds);
}

// A split product and the rank-r projection of the same Z in one launch: the first pwgs workgroups (a multiple of eight, so that the
// others keep their XCDs) project, rparts * 2 columns of items as in shrink_ring_kernel<1, 1, 1, 256>, the others multiply.
// Neither needs the other; gemm_add_up_kernel brings them together.  Small batches are bound by launches and memory round trips: 40
// one-token requests to 8 adapters, 4096 x 4096, took 9.5 us for the projection, 12.5 for the product, whose adapter workgroups waited for
// it, and 3.5 for the sum; together 22.3, now 15.0.
constexpr int kBesideLds = 80 * 1024;
template <bool W_KN, int TM, int TN, int WM, int WN, int STAGES>
__global__ __launch_bounds__(256, 2)
void gemm_tile_beside_kernel(PlanDev pd, const uint16_t* __restrict__ Z, const uint16_t* __restrict__ W, int32_t K, int32_t N,
                             int32_t ldw, int32_t tiles_m, int32_t tiles_n, int32_t GM, int32_t splits, float* __restrict__ part,
                             const uint16_t* __restrict__ D, const float* __restrict__ s, uint16_t* __restrict__ P_tok,
                             uint16_t* __restrict__ P_blk, int32_t rparts, int32_t pwgs)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int32_t wg = int32_t(blockIdx.x);
    if (wg < pwgs) {
        if (wg < pd.ntb * 2 * rparts)
            ring_item<1, 1, 1, 256, kBesideLds>(pd, Z, D, s, P_tok, P_blk, K, K, 1, 0, rparts, wg % pd.ntb, wg / pd.ntb, lds);
        return;
    }
    tile_body<W_KN, TM, TN, WM, WN, STAGES, 0>(pd, Z, W, nullptr, nullptr, nullptr, K, N, ldw, N, 1, 0, tiles_m, tiles_n, GM, splits, part,
                                            wg - pwgs, lds);
}

// C = the splits' partial products, in split order, plus the adapter term P M_t, rounded once.  A wave has 256 columns of a row, so the
// row's task and its projected activations are the same for all lanes; the rank rows go straight from memory into fp32 products, 16 of
// them in flight.  (S splits as a template argument: under a condition of its own every load waited for the one before.)  What bounds it:
// the chain of reads, each a round trip.  With the table of rows (ROWS: batches of up to kRowTableTokens) it is the row's
// entry, beside the sums and the first projected activations, then the rank rows; through the segments' tables it was
// row block, segments, task, ranks, rank rows: 40 requests x 4096 x 4096 15.2 us in all, with it 14.5.
template <int S, bool ROWS>
__global__ __launch_bounds__(256) void gemm_add_up_kernel(PlanDev pd, const float* __restrict__ part, const uint16_t* __restrict__ P,
                                                          const uint16_t* __restrict__ M, uint16_t* __restrict__ C, int32_t N)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    const int32_t row = int32_t(blockIdx.x) * 4 + wave, col = int32_t(blockIdx.y) * 256 + 4 * lane;
    if (row >= pd.T) return;
    const int32_t c = min(col, N - 4);
    f32x4 v[S];
    const int64_t n = int64_t(pd.T) * N;
#pragma unroll
    for (int i = 0; i < S; ++i) v[i] = *reinterpret_cast<const f32x4*>(part + i * n + int64_t(row) * N + c);
    const uint16_t first = P[size_t(row) * pd.r_pad + (lane & 15)];      // (a row has 16 ranks at least; not all of them its task's)
    int32_t r0 = 0, r = 0;                           // the row's first rank row, and how many; 0: no adapter
    if constexpr (ROWS) {
        const int32_t* e = row_rank(pd) + 2 * row;
        r0 = e[0], r = e[1];
    } else {
        // the row's segment: at most 32 begin in its block of 32 rows, and the table has the one of the block's first row
        const int32_t k0 = pd.rowblk_seg[row / kRowBlock], k = k0 + 1 + lane;
        const bool before = lane < kRowBlock && k < pd.nseg && pd.cseg_off[min(k, pd.nseg - 1)] <= row;
        const int32_t t = pd.cseg_task[k0 + __builtin_popcountll(__ballot(before))];
        if (t >= 0) {                                // (uniform)
            r0 = __builtin_amdgcn_readfirstlane(pd.rank_off[t]);
            r = __builtin_amdgcn_readfirstlane(pd.rank_off[t + 1]) - r0;
        }
    }
    f32x4 a = v[0];
#pragma unroll
    for (int i = 1; i < S; ++i) a = a + v[i];
    if (r > 0) {                                     // (uniform)
        f32x4 up = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int32_t p0 = 0; p0 < r; p0 += 16) {
            const int32_t left = r - p0;             // ranks beyond r: zero times zero
            const float pv = bf16_bits_to_float(p0 == 0 ? first : P[size_t(row) * pd.r_pad + min(p0 + (lane & 15), r - 1)]);
            uint64_t b[16];
#pragma unroll
            for (int q = 0; q < 16; ++q) b[q] = *reinterpret_cast<const uint64_t*>(M + size_t(r0 + min(p0 + q, r - 1)) * N + uint32_t(c));
            const float p = (lane & 15) < left ? pv : 0.f;
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                const float pq = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(p), q));
                const uint64_t m = b[q] & (q < left ? ~uint64_t(0) : uint64_t(0));
                const uint32_t lo = uint32_t(m), hi = uint32_t(m >> 32);
                up[0] += pq * __uint_as_float(lo << 16);
                up[1] += pq * __uint_as_float(lo & 0xffff0000u);
                up[2] += pq * __uint_as_float(hi << 16);
                up[3] += pq * __uint_as_float(hi & 0xffff0000u);
            }
        }
        a = a + up;
    }
    bf16x4 o;
#pragma unroll
    for (int u = 0; u < 4; ++u) o[u] = (__bf16)a[u];
    if (col < N) *reinterpret_cast<bf16x4*>(C + size_t(row) * N + col) = o;
}

// C = the sum of the splits' partial products, in split order, rounded once: 8 columns per thread.
template <int S>
__global__ __launch_bounds__(256) void gemm_add_kernel(const float* __restrict__ part, uint16_t* __restrict__ C, int64_t n, int32_t N,
                                                       int32_t ldc)
{
    const int64_t i = (int64_t(blockIdx.x) * 256 + threadIdx.x) * 8;
    if (i >= n) return;
    f32x4 v[S][2];
#pragma unroll
    for (int k = 0; k < S; ++k) {
        v[k][0] = *reinterpret_cast<const f32x4*>(part + k * n + i);
        v[k][1] = *reinterpret_cast<const f32x4*>(part + k * n + i + 4);
    }
    f32x4 a = v[0][0], b = v[0][1];
#pragma unroll
    for (int k = 1; k < S; ++k) a = a + v[k][0], b = b + v[k][1];
    bf16x8 o;
#pragma unroll
    for (int q = 0; q < 4; ++q) o[q] = (__bf16)a[q], o[4 + q] = (__bf16)b[q];
    *reinterpret_cast<bf16x8*>(C + size_t(i / N) * ldc + size_t(i % N)) = o;
}

// f(S) with S = n as a constant, S .. LAST
template <int S, int LAST, typename F> static void with_splits(int32_t n, F&& f)
{
    if constexpr (S <= LAST) {
        if (n == S) f(std::integral_constant<int, S>{});
        else with_splits<S + 1, LAST>(n, f);
    }
}

template <bool W_KN, int TM, int TN, int WM, int WN, int STAGES, int OCC>
static hipError_t launch_tile(const PlanDev& pd, const void* Z, const void* W, const void* P,
                              const void* M, void* C, int32_t K, int32_t N, int32_t ldw, int32_t ldc,
                              int32_t nproj, int32_t proj, hipStream_t st, int32_t splits, float* part)
{
    constexpr int bytes = ring_bytes<TM, TN, WN, STAGES>() + int(sizeof(TileTable<TM>)) + ahead_rows<TM, TN, WN, STAGES, OCC>() * TN * 2;
    static_assert(bytes * OCC <= 160 * 1024 && ahead_rows<TM, TN, WN, STAGES, OCC>() >= 16, "LDS budget");
    // the kernel needs more dynamic LDS than the default limit: raise it once per device
    static std::atomic<uint64_t> raised{0};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = uint64_t(1) << (dev & 63);
    if (!(raised.load(std::memory_order_acquire) & bit)) {
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_tile_kernel<W_KN, TM, TN, WM, WN, STAGES, OCC>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        if (e != hipSuccess) return e;
        raised.fetch_or(bit, std::memory_order_release);
    }
    const int32_t tiles_m = (pd.T + TM - 1) / TM, tiles_n = (N + TN - 1) / TN;
    const int32_t per = splits + (splits > 1 && P ? 1 : 0);          // workgroups per tile
    gemm_tile_kernel<W_KN, TM, TN, WM, WN, STAGES, OCC><<<dim3(uint32_t(tiles_m) * uint32_t(tiles_n) * uint32_t(per)), 64 * WM * WN, bytes, st>>>(
        pd, (const uint16_t*)Z, (const uint16_t*)W, (const uint16_t*)P, (const uint16_t*)M, (uint16_t*)C,
        K, N, ldw, ldc, nproj, proj, tiles_m, tiles_n, 1024 / TM, splits, part);
    e = hipGetLastError();
    if (e != hipSuccess || splits == 1) return e;
    const int64_t n = int64_t(pd.T) * N;             // (N is a multiple of 8)
    with_splits<2, kMaxSplits + 1>(per, [&](auto s_c) {
        gemm_add_kernel<decltype(s_c)::value><<<dim3(uint32_t((n + 2047) / 2048)), 256, 0, st>>>(part, (uint16_t*)C, n, N, ldc);
    });
    return hipGetLastError();
}

template <bool W_KN, int TM, int TN, int WM, int WN, int STAGES>
static hipError_t launch_beside(const PlanDev& pd, const void* Z, const void* W, const void* D, const float* s, void* P_tok, void* P_blk,
                                const void* M, void* C, int32_t K, int32_t N, int32_t ldw, hipStream_t st, int32_t splits, float* part)
{
    static_assert(WM * WN == 4 && ring_bytes<TM, TN, WN, STAGES>() + int(sizeof(TileTable<TM>)) <= kBesideLds, "two workgroups per compute unit");
    // the kernel needs more dynamic LDS than the default limit: raise it once per device
    static std::atomic<uint64_t> raised{0};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = uint64_t(1) << (dev & 63);
    if (!(raised.load(std::memory_order_acquire) & bit)) {
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_tile_beside_kernel<W_KN, TM, TN, WM, WN, STAGES>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, kBesideLds);
        if (e != hipSuccess) return e;
        raised.fetch_or(bit, std::memory_order_release);
    }
    const int32_t tiles_m = (pd.T + TM - 1) / TM, tiles_n = (N + TN - 1) / TN, rparts = (pd.r_max + 15) / 16;
    const int32_t pwgs = (pd.ntb * 2 * rparts + 7) / 8 * 8;
    gemm_tile_beside_kernel<W_KN, TM, TN, WM, WN, STAGES><<<dim3(uint32_t(pwgs + tiles_m * tiles_n * splits)), 256, kBesideLds, st>>>(
        pd, (const uint16_t*)Z, (const uint16_t*)W, K, N, ldw, tiles_m, tiles_n, 1024 / TM, splits, part, (const uint16_t*)D, s,
        (uint16_t*)P_tok, (uint16_t*)P_blk, rparts, pwgs);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    with_splits<1, kMaxSplits>(splits, [&](auto s_c) {
        const dim3 grid(uint32_t((pd.T + 3) / 4), uint32_t((N + 255) / 256));
        (pd.T <= kRowTableTokens ? gemm_add_up_kernel<decltype(s_c)::value, true> : gemm_add_up_kernel<decltype(s_c)::value, false>)<<<grid, 256, 0, st>>>(
            pd, part, (const uint16_t*)P_tok, (const uint16_t*)M, (uint16_t*)C, N);
    });
    return hipGetLastError();
}

hipError_t gemm_mfma_beside(const PlanDev& pd, const GemmChoice& choice, bool transW, const void* Z, const void* W, const void* D,
                            const float* s, void* P_tok, void* P_blk, const void* M, void* C, int32_t K, int32_t N, int32_t ldw,
                            hipStream_t st, float* part, size_t part_bytes)
{
    if (choice.tile < 0 || pd.T == 0 || pd.n_proj != 1 || !part || size_t(choice.splits) * size_t(pd.T) * size_t(N) * 4 > part_bytes ||
        !gemm_mfma_shape_ok(pd.T, K, N, ldw))
        return hipErrorInvalidValue;
#define LOBRA_BESIDE(...)                                                                                          \
    (transW ? launch_beside<false, __VA_ARGS__>(pd, Z, W, D, s, P_tok, P_blk, M, C, K, N, ldw, st, choice.splits, part)   \
            : launch_beside<true, __VA_ARGS__>(pd, Z, W, D, s, P_tok, P_blk, M, C, K, N, ldw, st, choice.splits, part))
    return choice.tile == 3 ? LOBRA_BESIDE(128, 64, 2, 2, 3) : LOBRA_BESIDE(64, 64, 2, 2, 4);
#undef LOBRA_BESIDE
}

bool gemm_mfma_shape_ok(int64_t T, int32_t K, int32_t N, int32_t ldw)
{
    if ((T + BM - 1) / BM * ((int64_t(N) + BN - 1) / BN) > 0x7fffffff) return false;
    // 32-bit byte offsets inside a tile: 256 rows of K (or ldw) elements, 64 rows of ldw elements
    if (int64_t(K) * 512 >= (int64_t(1) << 32) || int64_t(ldw) * 512 >= (int64_t(1) << 32)) return false;
    return N >= 8 && K >= 8;
}

hipError_t gemm_mfma(const PlanDev& pd, bool transW, const void* Z, const void* W, const void* P,
                     const void* M, void* C, int32_t K, int32_t N, int32_t ldw, hipStream_t st,
                     int32_t ldc, int32_t nproj, int32_t proj, float* part, size_t part_bytes)
{
    if (pd.T == 0) return hipSuccess;
    if (ldc == 0) ldc = N;
    if (!gemm_mfma_shape_ok(pd.T, K, N, ldw)) return hipErrorInvalidValue;   // (plan creation has checked already)
    const GemmChoice choice = choose_gemm(pd.T, K, N, proj < 0 ? pd.dg : 0, P ? pd.nseg : 0, pd.r_max / nproj,
                                          part ? std::min(part_bytes, kMaxPartBytes) : 0);
#define LOBRA_TILE(...)                                                                                          \
    (transW ? launch_tile<false, __VA_ARGS__>(pd, Z, W, P, M, C, K, N, ldw, ldc, nproj, proj, st, choice.splits, part)                 \
            : launch_tile<true, __VA_ARGS__>(pd, Z, W, P, M, C, K, N, ldw, ldc, nproj, proj, st, choice.splits, part))
    switch (choice.tile) {
    case kPersistentTile:
    case kStagedTile: {
        const int32_t tiles_m = (pd.T + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
        // tile rows per sweep of the tile order: the workgroups that run on an XCD at one time share their
        // Z and W panels through its L2 only while they walk K nearly in step, and the row bands that the 8
        // XCDs sweep at one time (8 x rows x 256 x K x 2 bytes) should stay in the 256 MB infinity cache for
        // their re-reads; measured on the five workloads, long K wants shorter sweeps (K = 8192 .. 28672:
        // 4 rows up to 7 % faster than 8; K = 4096: 5 .. 8 alike)
        return (choice.tile == kStagedTile ? gemm_staged : gemm_persistent)(pd, transW, Z, W, P, M, C, K, N, ldw, ldc, nproj, proj, tiles_m,
                                                                           tiles_n, K > 4096 ? 4 : 6, st);
    }
    case 1: return LOBRA_TILE(128, 256, 2, 4, 3, 1);
    case 2: return LOBRA_TILE(128, 128, 2, 2, 4, 1);
    case 3: return LOBRA_TILE(128, 64, 2, 2, 3, 2);
    case 4: return LOBRA_TILE(64, 64, 2, 2, 4, 2);
    default: return hipErrorInvalidValue;
    }
#undef LOBRA_TILE
}

}  // namespace lobra

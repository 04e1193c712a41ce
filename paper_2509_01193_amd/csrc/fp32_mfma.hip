// The fp32 path on the matrix cores (gfx950 v_mfma_f32_16x16x4_f32: fp32 operands, fp32 sums - twice the rate of the
// vector ALUs, same precision):
//   gemm        C = Z op(W) + P M_t        (y = x W + P B_t;  dx = dy W^T + P A_t)
//   shrink      P = s_t Z M_t^T            (Z = x, M = A: s_t A_t x_i;  Z = dy, M = B: s_t B_t dy_i)
//   gradreduce  dM_t = sum_i P_i^T Z_i     (dB_t from P = s h, Z = dy;  dA_t from P = s g, Z = x), stage 1
// (paper section 2.1: X W + X (down)(up), applied per task to a fused batch, section 1, and its derivatives).
//
// Operands of the MFMA: lane (i, kg), i = lane % 16, kg = lane / 16, supplies element k = kg of row i of "A" and of
// column i of "B"; a lane gets the results (4 kg .. 4 kg + 3, i).  A lane fetches four consecutive k of its row at a time
// and uses them in four MFMAs, MFMA q taking the k {q, 4 + q, 8 + q, 12 + q} of a group of 16: any dealing of the k
// will do as long as both operands follow it.
//
// VEC: rows start on 16-byte boundaries and end on them (widths that are multiples of 4).  Other widths take the same
// kernels with loads at any element and guards at the rows' ends.
#include "gemm_common.h"
#include "kernels.h"

namespace lobra {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));     // at any element

// elements i .. i + 3 of the row at p; elements from n on read as 0
template <bool VEC> __device__ __forceinline__ f32x4 load4(const float* __restrict__ p, int32_t i, int32_t n)
{
    if constexpr (VEC) {
        return i < n ? *reinterpret_cast<const f32x4*>(p + i) : f32x4{0.f, 0.f, 0.f, 0.f};
    } else {
        // (one load all the same - global memory takes 16 bytes at any address that is a multiple of 4 - except at the
        //  row's end; four loads of 4 bytes, 16 bytes apart from lane to lane, cost the address unit four times as much)
        if (i + 4 <= n) return *reinterpret_cast<const f32x4_any*>(p + i);
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = i + e < n ? p[i + e] : 0.f;
        return v;
    }
}

// K tiles of 32 to a range of a projection's sums, at most eight of them
__device__ __forceinline__ int32_t f32_range(int32_t ktiles) { return (ktiles + 7) / 8; }

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

}  // namespace

// -------------------------------------------------------------------------------------------
// gemm: TM x TN per workgroup of 2 x 2 waves; K tiles of 32 come through a ring of STAGES LDS slots that direct global -> LDS copies
// fill (16 bytes a lane, or 4 where rows start anywhere), one counted wait and one barrier each; the fragments of 16 k are read
// while the ones before are multiplied, every read and copy behind an MFMA (pinned by sched_barrier).  Bound by the matrix cores (a K tile
// of 64 x 64 is 1024 cycles of MFMAs, its copies 16 KiB and its fragment reads 20), tiles of 32 by the barriers.  Through registers, with the
// wait for all loads and a barrier around their way to LDS, the products of 3000 x 1024 x 1024 took 76 us, like this 61 and 63 (with
// neither reads nor copies in the loop 52: the rate of the MFMAs at the clock the chip keeps), of 8192 x 2048 x 2048 627 and 600, like
// this 559 and 563, of 1500 x 700 x 333 25 and 21, like this 18 and 19; the step of the first 162.8 -> 134.
//
// LDS: [rows][32 k], 128 bytes per row, 16-byte chunk c of a row at c ^ swz_row(row), for Z and, where K is fastest, W; else W as
// [32 k][TN n], and the MFMA columns are dealt so that a lane reads the NB columns of its NB blocks at once: column NB i of the
// wave tile and the ones behind it, for row i of the "A" operand.  (TN = 64 and 32: the chunks of odd lane groups' k rows are
// exchanged half a row apart, so that two groups' reads fall into different banks.)
// -------------------------------------------------------------------------------------------
template <bool TRANSW, int TM, int TN, int STAGES, int OCC, bool VEC, int NI = 0>
__global__ __launch_bounds__(256, OCC) void gemm_f32_kernel(PlanDev pd, const float* __restrict__ Z, const float* __restrict__ W,
                                                               const float* __restrict__ P, const float* __restrict__ M,
                                                               float* __restrict__ C, int32_t K, int32_t N, int32_t ldw, int32_t ldc,
                                                               int32_t nproj, int32_t proj, int32_t tiles_n,
                                                               const float* __restrict__ D, const float* __restrict__ s,
                                                               float* __restrict__ Pout)
{
    // NI > 0 (P = NULL): the tile projects its own rows.  The up to NI blocks of 16 ranks that its row block meets (F32Item) are further
    // rows of the ring, their products with the tile's rows of Z further MFMAs of the waves, and the workgroups of the first
    // column tile store the projected activations.
    using gemm::static_for;
    using gemm::swz_row;
    using gemm::wait_vmcnt;
    constexpr int FK = 32, WTM = TM / 2, WTN = TN / 2, MB = WTM / 16, NB = WTN / 16;
    constexpr int ZT = TM * FK * 4, AOFF = ZT + TN * FK * 4, SLOT = AOFF + NI * 16 * FK * 4;
    constexpr int E = VEC ? 4 : 1, LB = 64 * E * 4;              // elements per lane and bytes of a copy
    constexpr int ZC = ZT / LB / 4, WC = TN * FK * 4 / LB / 4, AC = NI * 16 * FK * 4 / LB / 4;
    constexpr int CPW = ZC + WC + AC;                            // copies per wave and K tile
    constexpr int ZL = FK / E, CR = TN / E;                      // lanes of a copy per row of 32 k, per k row of n
    constexpr int FPITCH = 20, NPITCH = TN + 4;                  // adapter step of 16 ranks: [rows][k] and [k][n] in front of the ring
    constexpr int ROW_TASK = (TM * FPITCH + 16 * NPITCH) * 4;    // behind it: the rows' tasks, and which rows are the first of one
    static_assert(ROW_TASK + TM * 4 + 16 <= STAGES * SLOT && ROW_TASK % 16 == 0, "the adapter term fits the ring");
    static_assert(TM <= 128 && NB <= 4 && (STAGES - 1) * CPW < 64, "two words of firsts; reads of up to 16 bytes; what vmcnt can count");
    static_assert(NI == 0 || (TM == 32 && TN == 32 && NI % 2 == 0), "a wave has every second block of ranks for its half of the rows");
    __shared__ __attribute__((aligned(16))) unsigned char lds[STAGES * SLOT];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1, j = lane & 15, kg = lane >> 4;
    const int32_t id = xcd_contiguous(blockIdx.x, gridDim.x);
    const int32_t row0 = id / tiles_n * TM, col0 = id % tiles_n * TN;
    const int32_t T = pd.T, row_end = min(row0 + TM, T);

    const F32BlockRec rec = P ? f32_block_rec(pd, row0 / kRowBlock) : F32BlockRec{};       // (in front of the copies: a scalar load)
    const int32_t first_sg = rec.own + (rec.lo > 0);
    const bool many = P && rec.fifth < row_end - row0;           // more than kFewSegments segments in the tile
    F32Item item[NI > 0 ? NI : 1];
    if constexpr (NI > 0) {
#pragma unroll
        for (int i = 0; i < NI; ++i) item[i] = f32_items(pd)[size_t(row0 / kRowBlock) * NI + i];
    }

    // ---- copies: rows beyond T and columns beyond N repeat the last one (what they produce is not stored), chunks beyond K too (the
    //      fragments are cleared)
    const uint32_t lds0 = uint32_t(uintptr_t((__attribute__((address_space(3))) unsigned char*)lds)), la0 = lds0 + wave * LB;
    const unsigned char* zcur = reinterpret_cast<const unsigned char*>(Z + size_t(row0) * K);
    const unsigned char* wcur = reinterpret_cast<const unsigned char*>(TRANSW ? W + size_t(col0) * ldw : W + col0);
    const size_t wstep = TRANSW ? size_t(FK) * 4 : size_t(FK) * ldw * 4;
    auto dma = [](uint32_t to, const unsigned char* from, uint32_t off) __attribute__((always_inline)) {
        if constexpr (VEC) gemm::dma16(to, from, off);
        else gemm::dma4(to, from, off);
    };
    auto swz_k = [](int k) { return TN == 128 ? 0 : ((k >> 2) & 1) << (TN == 64 ? 3 : 2); };
    // (element e of a row lies at swizzled(e, s): its chunk of 16 bytes exchanged)
    auto swizzled = [](int e, int s) { return (((e >> 2) ^ s) << 2) | (e & 3); };
    auto z_off = [&](int c, int32_t left, int lane) {          // of copy c, with `left` k in the K tile
        const int row = 64 / ZL * (wave + 4 * c) + lane / ZL;
        return (uint32_t(min(row, T - 1 - row0)) * uint32_t(K) + uint32_t(min(swizzled(E * (lane % ZL), swz_row(row)), left - E))) * 4u;
    };
    auto w_off = [&](int c, int32_t left, int lane) {
        if (TRANSW) {
            const int row = 64 / ZL * (wave + 4 * c) + lane / ZL;
            return (uint32_t(min(row, N - 1 - col0)) * uint32_t(ldw) + uint32_t(min(swizzled(E * (lane % ZL), swz_row(row)), left - E))) * 4u;
        }
        // (a copy has several k rows, or half of one: TN = 128, four bytes a lane)
        const int at = 64 * (wave + 4 * c) + lane, k = at / CR;
        return (uint32_t(min(k, left - 1)) * uint32_t(ldw) + uint32_t(min(swizzled(E * (at % CR), swz_k(k)), N - E - col0))) * 4u;
    };
    uint32_t zvo[ZC], wvo[WC];
#pragma unroll
    for (int c = 0; c < ZC; ++c) zvo[c] = z_off(c, FK, lane);
#pragma unroll
    for (int c = 0; c < WC; ++c) wvo[c] = w_off(c, FK, lane);
    // (rank rows: a copy has rows of one block; those beyond its last repeat it)
    const unsigned char* abase[AC > 0 ? AC : 1];
    int32_t an[AC > 0 ? AC : 1];
    uint32_t avo[AC > 0 ? AC : 1];
    size_t aat = 0;
    auto a_off = [&](int c, int32_t left, int lane) {
        const int row = 64 / ZL * (wave + 4 * c) + lane / ZL;
        return (uint32_t(min(row & 15, max(an[c] - 1, 0))) * uint32_t(K) + uint32_t(min(swizzled(E * (lane % ZL), swz_row(row)), left - E))) * 4u;
    };
    if constexpr (NI > 0) {
#pragma unroll
        for (int c = 0; c < AC; ++c) {
            int32_t row = item[0].row;
            an[c] = item[0].n;
#pragma unroll
            for (int i = 1; i < NI; ++i)
                if ((64 / ZL * (wave + 4 * c)) >> 4 == i) row = item[i].row, an[c] = item[i].n;
            abase[c] = reinterpret_cast<const unsigned char*>(D + size_t(row) * K);
            avo[c] = a_off(c, FK, lane);
        }
    }
    auto copy = [&](auto c_c, uint32_t la) __attribute__((always_inline)) {
        constexpr int c = decltype(c_c)::value;
        if constexpr (c < ZC) dma(la + 4 * c * LB, zcur, zvo[c]);
        else if constexpr (c < ZC + WC) dma(la + ZT + 4 * (c - ZC) * LB, wcur, wvo[c - ZC]);
        else dma(la + AOFF + 4 * (c - ZC - WC) * LB, abase[c - ZC - WC] + aat, avo[c - ZC - WC]);
    };
    auto next_copy_tile = [&]() __attribute__((always_inline)) { zcur += FK * 4, wcur += wstep, aat += FK * 4; };
    const int32_t KT = (K + FK - 1) / FK, ktail = K % FK, KF = K / FK;
    auto copy_tail = [&](uint32_t la) {
        int ln = lane;
        if constexpr (TM == 128) asm volatile("" : "+v"(ln));        // (its addresses are worked out here: no registers are left for them in the main loop)
#pragma unroll
        for (int c = 0; c < ZC; ++c) dma(la + 4 * c * LB, zcur, z_off(c, ktail, ln));
#pragma unroll
        for (int c = 0; c < WC; ++c) dma(la + ZT + 4 * c * LB, wcur, w_off(c, ktail, ln));
#pragma unroll
        for (int c = 0; c < AC; ++c) dma(la + AOFF + 4 * c * LB, abase[c] + aat, a_off(c, ktail, ln));
    };
    for (int s = 0; s < STAGES; ++s) {
        if (s < KF) static_for<0, CPW>([&](auto c_c) { copy(c_c, la0 + s * SLOT); });
        else if (s < KT) copy_tail(la0 + s * SLOT);
        next_copy_tile();
    }

    // ---- the adapter term's first step - the first segment's first 16 ranks - is fetched in front of the main loop, behind its first
    //      copies, with what the row block's record says (through the segments' tables, a chain of four reads: 4 us of 62 at 3000 x
    //      1024 x 1024)
    constexpr int ZA = TM * 16 / 256, WA = TN * 16 / 256;
    float pa[ZA], ma[WA];
    // (mine(u, row): whether the row of piece u is the segment's, or the task's)
    auto load_adapter_of = [&](auto mine, int32_t r, int32_t pofs, int32_t r0, int32_t c0) {
#pragma unroll
        for (int u = 0; u < ZA; ++u) {
            const int e = tid + 256 * u, kk = e & 15, row = row0 + (e >> 4);
            pa[u] = (mine(u, row) && c0 + kk < r) ? P[size_t(row) * pd.r_max + pofs + c0 + kk] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < WA; ++u) {
            const int e = tid + 256 * u, n = col0 + e % TN, kk = e / TN;
            ma[u] = (c0 + kk < r && n < N) ? M[size_t(r0 + c0 + kk) * N + n] : 0.f;
        }
    };
    auto load_adapter = [&](int32_t lo, int32_t hi, int32_t r, int32_t pofs, int32_t r0, int32_t c0) {
        load_adapter_of([&](int, int32_t row) { return row >= lo && row < hi; }, r, pofs, r0, c0);
    };
    const bool some = P && !many && rec.lo < row_end - row0;
    if (some) {
        const int32_t r = rec.rank / nproj;
        load_adapter(row0 + rec.lo, min(row0 + rec.hi, row_end), r, proj * r, rec.rank0 + proj * r, 0);
    }

    float mi[NI > 0 ? NI : 1][WA], scale[NI > 0 ? NI / 2 : 1];       // the up factors' rows of the blocks; the scales of this wave's
    if constexpr (NI > 0) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int u = 0; u < WA; ++u) {
                const int e = tid + 256 * u, n = col0 + e % TN, kk = e / TN;
                mi[i][u] = kk < item[i].n && n < N ? M[size_t(item[i].row + kk) * N + n] : 0.f;
            }
#pragma unroll
        for (int b = 0; b < NI / 2; ++b) scale[b] = s[wn ? item[2 * b + 1].task : item[2 * b].task];
    }

    // ---- fragments and the steps of 16 k
    constexpr int HB = NI / 2;                       // this wave's blocks of ranks: wn, wn + 2, ...
    struct Frags {
        f32x4 z[MB];
        float w[NB][4];                              // [block][q]
        f32x4 a[HB > 0 ? HB : 1];
    };
    constexpr int NR = MB + (TRANSW ? NB : 4) + HB;  // reads of a step
    auto read = [&](auto i_c, Frags& f, const unsigned char* slot, int ks) __attribute__((always_inline)) {
        constexpr int i = decltype(i_c)::value;
        constexpr int NW = TRANSW ? NB : 4;
        const int ch = (4 * ks + kg) ^ swz_row(j);
        if constexpr (i >= NW + MB) {
            f.a[i - NW - MB] = *reinterpret_cast<const f32x4*>(slot + AOFF + ((wn + 2 * (i - NW - MB)) * 16 + j) * 128 + ch * 16);
        } else if constexpr (i >= NW) {
            f.z[i - NW] = *reinterpret_cast<const f32x4*>(slot + (wm * WTM + (i - NW) * 16 + j) * 128 + ch * 16);
        } else if constexpr (TRANSW) {
            const f32x4 v = *reinterpret_cast<const f32x4*>(slot + ZT + (wn * WTN + i * 16 + j) * 128 + ch * 16);
#pragma unroll
            for (int q = 0; q < 4; ++q) f.w[i][q] = v[q];
        } else {
            const int k = 16 * ks + 4 * kg + i, n = wn * WTN + NB * j;
            const unsigned char* at = slot + ZT + k * (TN * 4) + swizzled(n, swz_k(k)) * 4;
            if constexpr (NB == 1) {
                f.w[0][i] = *reinterpret_cast<const float*>(at);
            } else {
                typedef float row_t __attribute__((ext_vector_type(NB)));
                const row_t v = *reinterpret_cast<const row_t*>(at);
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) f.w[nb][i] = v[nb];
            }
        }
    };
    f32x4 acc[MB][NB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    // The projections: a chain of sums over an eighth of the K tiles, first and second K steps of a K tile apart, and the sum of those before,
    // so that as few products follow each other as in the 16 waves of shrink_f32_kernel.  (Two chains over all of K, 1000 x 2500 x 64:
    // gradients 6.7e-7 from 64 bits, like this 2.6e-7, with a projection of its own 2.7e-7.)
    struct Chain { f32x4 run, all; };
    Chain h[HB > 0 ? HB : 1][2];
#pragma unroll
    for (int b = 0; b < HB; ++b)
#pragma unroll
        for (int k = 0; k < 2; ++k) h[b][k].run = h[b][k].all = f32x4{0.f, 0.f, 0.f, 0.f};
    const int32_t range = NI > 0 ? f32_range(KT) : 0;
    int32_t range_end = range;
    auto fold = [&](int k) {                         // in front of the K step k that begins a range, half a K tile behind the chain's last MFMA
#pragma unroll
        for (int b = 0; b < HB; ++b) {
            h[b][k].all = h[b][k].all + h[b][k].run;
            h[b][k].run = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    };
    // the MFMAs on `f`, fragments of K step ks ^ 1, with the reads of the next step's fragments (ks) and (COPY) a K tile's copies dealt
    // evenly behind them
    auto kstep = [&](auto read_c, auto copy_c, const Frags& f, Frags& next, const unsigned char* slot, auto ks_c, uint32_t la) __attribute__((always_inline)) {
        constexpr int ks = decltype(ks_c)::value, PQ = MB * NB + HB;
        constexpr int NM = 4 * PQ, R = decltype(read_c)::value ? NR : 0, CC = decltype(copy_c)::value ? CPW : 0;
        static_for<0, NM>([&](auto m_c) {
            constexpr int m = decltype(m_c)::value, q = m / PQ, mb = m % PQ / NB, nb = m % PQ % NB;
            if constexpr (m % PQ < MB * NB) {
                acc[mb][nb] = mfma4(f.w[nb][q], f.z[mb][q], acc[mb][nb]);
            } else {
                f32x4& run = h[m % PQ - MB * NB][ks ^ 1].run;
                run = mfma4(f.a[m % PQ - MB * NB][q], f.z[0][q], run);
            }
            static_for<m * R / NM, (m + 1) * R / NM>([&](auto i_c) { read(i_c, next, slot, ks); });
            static_for<m * CC / NM, (m + 1) * CC / NM>([&](auto c_c) { copy(c_c, la); });
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    auto clear_tail = [&](Frags& f, int ks) __attribute__((always_inline)) {       // lane group kg holds k 16 ks + 4 kg .. + 3
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const bool in = 16 * ks + 4 * kg + q < ktail;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) f.z[mb][q] = in ? f.z[mb][q] : 0.f;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) f.w[nb][q] = in ? f.w[nb][q] : 0.f;
#pragma unroll
            for (int b = 0; b < HB; ++b) f.a[b][q] = in ? f.a[b][q] : 0.f;
        }
    };
    using step0 = std::integral_constant<int, 0>;
    using step1 = std::integral_constant<int, 1>;
    using yes = std::true_type;
    using no = std::false_type;
    auto barrier = []() __attribute__((always_inline)) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    if (KT >= STAGES) wait_vmcnt<(STAGES - 1) * CPW>();
    else wait_vmcnt<0>();
    barrier();
    Frags fa, fb;
    static_for<0, NR>([&](auto i_c) { read(i_c, fa, lds, 0); });
    int32_t kt = 0, slot = 0;
    auto ktile = [&](auto fold_c) __attribute__((always_inline)) {   // a whole K tile is still to be copied
        const unsigned char* cur = lds + slot * SLOT;
        if constexpr (decltype(fold_c)::value) fold(0);
        kstep(yes{}, no{}, fa, fb, cur, step1{}, 0);
        if constexpr (decltype(fold_c)::value) fold(1);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        wait_vmcnt<(STAGES - 2) * CPW>();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        const uint32_t la = la0 + slot * SLOT;
        slot = slot + 1 == STAGES ? 0 : slot + 1;
        kstep(yes{}, yes{}, fb, fa, lds + slot * SLOT, step0{}, la);
        next_copy_tile();
    };
    if constexpr (NI > 0) {
        while (kt < KF - STAGES) {
            if (kt == range_end) {
                ktile(yes{});
                ++kt;
                range_end += range;
            }
            const int32_t end = min(range_end, KF - STAGES);
            for (; kt < end; ++kt) ktile(no{});
        }
    } else {
        for (; kt < KF - STAGES; ++kt) ktile(no{});
    }
    for (; kt < KT; ++kt) {                          // the last STAGES K tiles, and the partial one
        const bool tail = ktail != 0 && kt + 1 == KT;            // uniform
        const bool begins = NI > 0 && kt == range_end;
        if (begins) fold(0);
        if (tail) clear_tail(fa, 0);
        kstep(yes{}, no{}, fa, fb, lds + slot * SLOT, step1{}, 0);
        if (begins) {
            fold(1);
            range_end += range;
        }
        if (tail) clear_tail(fb, 1);
        if (kt + 1 < KT) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            wait_vmcnt<0>();
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            if (kt + STAGES < KT) copy_tail(la0 + slot * SLOT);
            slot = slot + 1 == STAGES ? 0 : slot + 1;
            kstep(yes{}, no{}, fb, fa, lds + slot * SLOT, step0{}, 0);
        } else {
            kstep(no{}, no{}, fb, fa, lds, step0{}, 0);
        }
    }

    // ---- adapter term: 16 ranks at a time are further k of the same tile product, rows outside the segment and ranks beyond r_t zero (the
    //      loops are uniform over the workgroup).  Where more than kFewSegments segments cross the tile, per task that has rows in it
    //      (8000 one-token segments of 8 tasks of rank 128, 10 x 1373: 4820 -> 290 us; 10119 tokens in segments of 3, rank 8, 64 x 1920:
    //      390 -> 112).
    float *const zs = reinterpret_cast<float*>(lds), *const ws = zs + TM * FPITCH;
    auto stash_adapter = [&]() {
#pragma unroll
        for (int u = 0; u < ZA; ++u) zs[((tid + 256 * u) >> 4) * FPITCH + (tid & 15)] = pa[u];
#pragma unroll
        for (int u = 0; u < WA; ++u) ws[(tid + 256 * u) / TN * NPITCH + (tid + 256 * u) % TN] = ma[u];
    };
    auto col_of = [&](int nb, int i) { return wn * WTN + (TRANSW ? nb * 16 + i : NB * i + nb); };    // of result row i of block nb
    // (crosses(mb): whether the segment, or the task, has rows in block mb of the wave, uniform.  The others are left alone: zeros in place of a
    //  row of P would not keep out what is not finite in another task's adapter)
    auto mac = [&](const float* zs, const float* ws, auto crosses) {
        float w[NB][4];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int q = 0; q < 4; ++q) w[nb][q] = ws[(4 * kg + q) * NPITCH + col_of(nb, j)];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            if (!crosses(mb)) continue;
            const f32x4 z = *reinterpret_cast<const f32x4*>(zs + (wm * WTM + mb * 16 + j) * FPITCH + 4 * kg);
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = mfma4(w[nb][q], z[q], acc[mb][nb]);
        }
    };
    auto crosses_rows = [&](int32_t lo, int32_t hi) {
        return [=](int mb) { return hi > row0 + wm * WTM + mb * 16 && lo < row0 + wm * WTM + mb * 16 + 16; };
    };
    if constexpr (NI > 0) {
        constexpr int HZ = TM * FPITCH, HW = 16 * NPITCH;
        static_assert(NI * (HZ + HW) * 4 <= STAGES * SLOT, "all blocks fit the ring");
        __syncthreads();                             // everybody is done with the ring
#pragma unroll
        for (int b = 0; b < HB; ++b) {               // lane (j, kg): ranks 4 kg .. + 3 of token row j of the wave's half
            const F32Item u = item[2 * b], w = item[2 * b + 1];          // (member by member: a choice of whole ones goes through memory)
            const F32Item t = {wn ? w.lo : u.lo, wn ? w.hi : u.hi, 0, wn ? w.n : u.n, 0, wn ? w.c0 : u.c0, wn ? w.r : u.r, 0};
            const int32_t row = row0 + wm * 16 + j;
            const bool in = row >= t.lo && row < t.hi;
            const f32x4 sum = (h[b][0].all + h[b][0].run) + (h[b][1].all + h[b][1].run);
            f32x4 p;
#pragma unroll
            for (int v = 0; v < 4; ++v) p[v] = in && 4 * kg + v < t.n ? scale[b] * sum[v] : 0.f;
            *reinterpret_cast<f32x4*>(zs + (wn + 2 * b) * HZ + (wm * 16 + j) * FPITCH + 4 * kg) = p;
            if (col0 == 0 && in) {
                // (and zeros behind the task's last block, as far as a row goes)
                float* dst = Pout + size_t(row) * pd.r_max;
                for (int32_t k = t.c0 + 4 * kg; k < (t.c0 + 16 < t.r ? t.c0 + 16 : pd.r_max); k += 16) {
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (k + v < pd.r_max) dst[k + v] = p[v];
                    p = f32x4{0.f, 0.f, 0.f, 0.f};
                }
            }
        }
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int u = 0; u < WA; ++u) zs[NI * HZ + i * HW + (tid + 256 * u) / TN * NPITCH + (tid + 256 * u) % TN] = mi[i][u];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NI; ++i)
            if (item[i].n > 0) mac(zs + i * HZ, zs + NI * HZ + i * HW, crosses_rows(item[i].lo, item[i].hi));        // (uniform)
    }
    if (some || many) __syncthreads();               // everybody is done with the ring
    if (some) {
        for (int32_t sg = first_sg; sg < pd.nseg; ++sg) {
            const int32_t seg_lo = pd.cseg_off[sg];
            if (seg_lo >= row_end) break;
            const int32_t t = pd.cseg_task[sg];
            if (t < 0) continue;
            const int32_t lo = max(seg_lo, row0), hi = min(pd.cseg_off[sg + 1], row_end);
            const int32_t r = (pd.rank_off[t + 1] - pd.rank_off[t]) / nproj, pofs = proj * r;
            const int32_t r0 = pd.rank_off[t] + pofs;
            for (int32_t c0 = 0; c0 < r; c0 += 16) {
                if (sg != first_sg || c0 > 0) load_adapter(lo, hi, r, pofs, r0, c0);
                stash_adapter();
                __syncthreads();
                mac(zs, ws, crosses_rows(lo, hi));
                __syncthreads();
            }
        }
    }
    if (many) {
        int32_t* const row_task = reinterpret_cast<int32_t*>(lds + ROW_TASK);
        uint64_t* const firsts = reinterpret_cast<uint64_t*>(lds + ROW_TASK + TM * 4);
        if (tid < TM) {
            const int32_t sg = rec.own + tid;        // (at most one segment per row)
            if (sg < pd.nseg && pd.cseg_off[sg] < row_end) {
                const int32_t t = pd.cseg_task[sg], hi = min(pd.cseg_off[sg + 1], row_end) - row0;
                for (int32_t i = max(pd.cseg_off[sg], row0) - row0; i < hi; ++i) row_task[i] = t;
            }
            if (row0 + tid >= row_end) row_task[tid] = -1;
        }
        __syncthreads();
        const int32_t own = tid < TM ? row_task[tid] : -1;
        bool first = own >= 0;
        for (int i = 0; i < TM; i += 4) {
            const int4 a = *reinterpret_cast<const int4*>(&row_task[i]);
            first &= !((a.x == own && i < tid) || (a.y == own && i + 1 < tid) || (a.z == own && i + 2 < tid) || (a.w == own && i + 3 < tid));
        }
        const uint64_t word = __ballot(first);
        if (wave < 2 && lane == 0) firsts[wave] = word;
        int32_t rt[ZA];                              // tasks of this thread's rows
#pragma unroll
        for (int u = 0; u < ZA; ++u) rt[u] = row_task[(tid + 256 * u) >> 4];
        __syncthreads();
        auto uniform = [](uint64_t v) {
            return (uint64_t(uint32_t(__builtin_amdgcn_readfirstlane(uint32_t(v >> 32)))) << 32) |
                   uint32_t(__builtin_amdgcn_readfirstlane(uint32_t(v)));
        };
        uint64_t left[2] = {uniform(firsts[0]), uniform(firsts[1])};
        int32_t t = -1, r = 0, c0 = 0;
        auto next = [&]() {                          // moves to the next 16 ranks, of the next task at a task's end
            c0 += 16;
            if (c0 < r) return true;
            const int w = left[0] ? 0 : 1;
            if (!left[w]) return false;
            t = __builtin_amdgcn_readfirstlane(row_task[64 * w + __builtin_ctzll(left[w])]);
            left[w] &= left[w] - 1;
            r = (pd.rank_off[t + 1] - pd.rank_off[t]) / nproj;
            c0 = 0;
            return true;
        };
        auto load = [&]() { load_adapter_of([&](int u, int32_t) { return rt[u] == t; }, r, proj * r, pd.rank_off[t] + proj * r, c0); };
        bool more = next();
        if (more) load();
        while (more) {
            stash_adapter();
            __syncthreads();
            const int32_t now = t;
            more = next();
            if (more) load();
            mac(zs, ws, [&](int mb) { return __ballot(row_task[wm * WTM + mb * 16 + j] == now) != 0; });
            __syncthreads();
        }
    }
    // acc[mb][nb][v]: token row mb 16 + j of the wave tile, column col_of(nb, 4 kg + v)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        const int32_t row = row0 + wm * WTM + mb * 16 + j;
        if (row >= T) continue;
#pragma unroll
        for (int u = 0; u < NB; ++u) {               // 16 bytes at a time
            const int32_t col = col0 + wn * WTN + (TRANSW ? 16 * u + 4 * kg : 4 * NB * kg + 4 * u);
            f32x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = TRANSW ? acc[mb][u][e] : acc[mb][(4 * u + e) % NB][(4 * u + e) / NB];
            float* c = C + size_t(row) * ldc + col;
            if (VEC && col < N) {
                *reinterpret_cast<f32x4*>(c) = v;
            } else if (!VEC && col + 4 <= N) {
                *reinterpret_cast<f32x4_any*>(c) = v;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (col + e < N) c[e] = v[e];
            }
        }
    }
}

hipError_t gemm_f32(const PlanDev& pd, bool transW, const float* Z, const float* W, const float* P, const float* M, float* C,
                    int32_t K, int32_t N, int32_t ldw, int32_t ldc, int32_t nproj, int32_t proj, hipStream_t st)
{
    // The larger the tile the fewer loads per MFMA, as long as every compute unit has work: by an estimate of rounds of workgroups
    // (us; four of 32, three of 64, two of 128 to a compute unit; the rounds of a short K overlap).  Tiles of 32 / 64 / 128:
    //     600 x 1024 x 1024  23 / 25 / 70      1000 x 1024 x 1024  30 / 27 / 74     4000 x 1024 x 1024  104 / 89 / 77
    //     2000 x 512 x 512  17 / 16 / 43       4000 x 96 x 512  16 / 12 / 20        8000 x 128 x 1024  50 / 33 / 36
    //     3000 x 256 x 256  11.0 / 11.5        1500 x 512 x 512  15.1 / 16.2        8000 x 512 x 96  15.1 / 17.3
    //     3000 x 128 x 512  13.1 / 12.5        2000 x 256 x 384  10.6 / 11.2        8000 x 64 x 64  6.3 / 8.6
    //     8000 x 256 x 256  21.5 / 17.3        8000 x 512 x 512  - / 49 / 45        8000 x 2048 x 2048  - / 587 / 549
    //     3000 x 2048 x 2048  - / 205 / 245    4000 x 2048 x 2048  - / 268 / 255    5000 x 384 x 768  - / 34.3 / 37.2
    // (W read along K, in backward passes: tiles of 64 take 620 for 8000 x 2048 x 2048, of 128 548), and at rows on no 16-byte boundaries
    //     600 x 1357 x 1676  40 / 51 / 149     2000 x 1357 x 1676  130 / 104 / 157  4000 x 1357 x 1676  262 / 187 / 262
    // (128 four bytes a lane: behind the others everywhere, the addresses of 32 copies a K tile do not fit the registers)
    const bool vec = ((K | N | ldw | ldc) & 3) == 0;
    auto tiles = [&](int32_t t) { return int64_t((pd.T + t - 1) / t) * ((N + t - 1) / t); };
    auto estimate = [&](int32_t t) {
        const float k = float(K) / 1024.f;
        const int64_t n = tiles(t), per = t == 64 ? 768 : 512, full = n / per, rest = n % per;
        if (t == 32) return 4.5f + 3.f * k + float(n) * (0.0205f * k + 0.003f);
        if (t == 64)
            return (transW ? 1.04f : 1.f) * (float(full) * (2.f + 48.f * k) +
                                             (rest == 0 ? 4.f : rest <= 256 ? (full ? 5.f + 24.f * k : 7.f + 18.5f * k) : rest <= 512 ? 8.5f + 34.f * k : 10.f + 47.f * k));
        return float(full) * (20.f + 120.f * k) + (rest == 0 ? 0.f : rest <= 256 ? 11.f + (full ? 48.f : 63.f) * k : 22.f + 118.f * k);
    };
    int32_t tm = estimate(64) < estimate(32) ? 64 : 32;
    if (vec && estimate(128) < estimate(tm)) tm = 128;
    const int32_t tiles_n = (N + tm - 1) / tm;
    const dim3 grid(uint32_t((pd.T + tm - 1) / tm) * uint32_t(tiles_n));
#define LOBRA_F32_GEMM(TR, TILE, STAGES, OCC) \
    (vec ? gemm_f32_kernel<TR, TILE, TILE, STAGES, OCC, true> : gemm_f32_kernel<TR, TILE, TILE, STAGES, OCC, false>)<<<grid, 256, 0, st>>>(pd, Z, W, P, M, C, K, N, ldw, ldc, nproj, proj, tiles_n, nullptr, nullptr, nullptr)
#define LOBRA_F32_GEMM2(TR) \
    do { \
        if (tm == 32) LOBRA_F32_GEMM(TR, 32, 5, 4); \
        else if (tm == 64) LOBRA_F32_GEMM(TR, 64, 3, 3); \
        else gemm_f32_kernel<TR, 128, 128, 2, 2, true><<<grid, 256, 0, st>>>(pd, Z, W, P, M, C, K, N, ldw, ldc, nproj, proj, tiles_n, nullptr, nullptr, nullptr); \
    } while (0)
    if (transW) LOBRA_F32_GEMM2(true);
    else LOBRA_F32_GEMM2(false);
#undef LOBRA_F32_GEMM
#undef LOBRA_F32_GEMM2
    return hipGetLastError();
}

// The same with the projection of Z's rows in the product's launch (pd's plan has ni items per 32-row block, see f32_fused): what a
// short batch is bound by is launches and round trips to memory.  618 x 256 x 256, two tasks of rank 8, projection and product 4.6 + 7.1
// us, like this 7.7 (the step 26.7 -> 22.3).
hipError_t gemm_f32_fused(const PlanDev& pd, int32_t ni, bool transW, const float* Z, const float* W, const float* D, const float* s, float* P,
                          const float* M, float* C, int32_t K, int32_t N, int32_t ldw, hipStream_t st)
{
    const int32_t tiles_n = (N + 31) / 32;
    const dim3 grid(uint32_t((pd.T + 31) / 32) * uint32_t(tiles_n));
    const bool vec = ((K | N | ldw) & 3) == 0;
#define LOBRA_F32_FUSED(TR, NI, OCC) \
    (vec ? gemm_f32_kernel<TR, 32, 32, 4, OCC, true, NI> : gemm_f32_kernel<TR, 32, 32, 4, OCC, false, NI>)<<<grid, 256, 0, st>>>(pd, Z, W, nullptr, M, C, K, N, ldw, N, 1, 0, tiles_n, D, s, P)
    if (ni == 2) {
        if (transW) LOBRA_F32_FUSED(true, 2, 3);
        else LOBRA_F32_FUSED(false, 2, 3);
    } else if (ni == 4) {
        if (transW) LOBRA_F32_FUSED(true, 4, 2);
        else LOBRA_F32_FUSED(false, 4, 2);
    } else {
        return hipErrorInvalidValue;
    }
#undef LOBRA_F32_FUSED
    return hipGetLastError();
}

// -------------------------------------------------------------------------------------------
// shrink: one workgroup per half of a token block (16 tokens of one task), NW waves (16, or 4 for longer batches) split K in
// groups of 16; both operands go straight from global memory into registers, "A" = 16 rank rows, "B" = 16 token rows, four
// rank blocks at a time.
// Latency and memory bound: a wave has the loads of four groups in flight (two at large ranks).
// RANGES: the groups and the order of the sums are those of the projection inside its product, so that it gives the same bits: wave
// 2 i + k has the K steps k of the K tiles of range i.  (Through the product's kernel without the product, one K tile after another:
// backward passes without dx, 32 x 2048 x 2048, 27.0 us, like this 12.9, without the saved activations, 1000 x 2500 x 64, 64 and 34.)
// -------------------------------------------------------------------------------------------
template <int NRB, int NW, bool VEC, bool RANGES>
__global__ __launch_bounds__(64 * NW) void shrink_f32_kernel(PlanDev pd, const float* __restrict__ Z, const float* __restrict__ M,
                                                         const float* __restrict__ s, float* __restrict__ P, int32_t D,
                                                         int32_t ldz, int32_t nproj, int32_t proj)
{
    // nproj > 1 (fused shared-input projections): projection `proj` only - Z is its column block of
    // dy (row pitch ldz), M its rows of the compact up factors, and of the task's ranks the window
    // [proj r, (proj + 1) r) is read and written
    constexpr int DEPTH = NRB == 4 ? 2 : 4;          // (128 registers per wave)
    static_assert(NW >= NRB, "a wave per rank block adds the sums");
    static_assert(!RANGES || NW == 16, "two waves for each of eight ranges");
    __shared__ f32x4 red[NW][NRB][64];
    const TokenBlock b = pd.tb[blockIdx.x >> 1];
    const int half = blockIdx.x & 1;
    if (16 * half >= b.nrows) return;
    const int32_t r = (pd.rank_off[b.task + 1] - pd.rank_off[b.task]) / nproj;
    const int32_t pofs = proj * r;
    const int32_t plim = proj == nproj - 1 ? pd.r_max - pofs : r;   // ranks (and zero padding) stored here
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, j = lane & 15, kg = lane >> 4;
    const int32_t tok = 16 * half + j;
    const float* zrow = Z + size_t(b.row0 + min(tok, b.nrows - 1)) * ldz;    // rows beyond the block repeat its last one
    const float st = s[b.task];
    for (int32_t p0 = 0; p0 < plim; p0 += 16 * NRB) {
        f32x4 acc[NRB];
        const float* mrow[NRB];          // ranks beyond r_t repeat the last rank row; their sums are not stored
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) {
            acc[rb] = f32x4{0.f, 0.f, 0.f, 0.f};
            mrow[rb] = M + size_t(b.rank_row0 + pofs + min(p0 + 16 * rb + j, r - 1)) * D;
        }
        const int32_t nrb = min(NRB, (r - p0 + 15) >> 4);           // rank blocks with ranks of the task (uniform)
        f32x4 z[DEPTH], m[DEPTH][NRB];
        const int32_t range = 2 * f32_range((D + 31) >> 5), STRIDE = RANGES ? 2 : NW;
        const int32_t g0 = RANGES ? (wave >> 1) * range + (wave & 1) : wave, ng = RANGES ? (wave >> 1) * range + range : (D + 15) >> 4;
        for (int32_t g = g0; nrb > 0 && g < ng; g += DEPTH * STRIDE) {          // (groups beyond D, or the range, read as zero)
#pragma unroll
            for (int u = 0; u < DEPTH; ++u) {
                const int32_t gu = g + u * STRIDE, k = RANGES && gu >= ng ? D : 16 * gu + 4 * kg;
                z[u] = load4<VEC>(zrow, k, D);
#pragma unroll
                for (int rb = 0; rb < NRB; ++rb)
                    if (rb < nrb) m[u][rb] = load4<VEC>(mrow[rb], k, D);
            }
#pragma unroll
            for (int u = 0; u < DEPTH; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int rb = 0; rb < NRB; ++rb)
                        if (rb < nrb) acc[rb] = mfma4(m[u][rb][q], z[u][q], acc[rb]);
        }
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) red[wave][rb][lane] = acc[rb];
        __syncthreads();
        // rank block rb is summed by wave rb, in wave order: lane (j, kg) stores ranks 4 kg .. 4 kg + 3 of token j
        if (wave < NRB) {
            f32x4 sum;
            if constexpr (RANGES) {
                f32x4 all[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
                for (int w = 0; w < NW; ++w) all[w & 1] = all[w & 1] + red[w][wave][lane];
                sum = all[0] + all[1];
            } else {
                sum = red[0][wave][lane];
#pragma unroll
                for (int w = 1; w < NW; ++w) sum = sum + red[w][wave][lane];
            }
            if (tok < b.nrows)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int32_t p = p0 + 16 * wave + 4 * kg + v;
                    if (p < plim) P[size_t(b.row0 + tok) * pd.r_max + pofs + p] = p < r ? st * sum[v] : 0.f;
                }
        }
        __syncthreads();
    }
}

hipError_t shrink_f32(const PlanDev& pd, const float* Z, const float* M, const float* s, float* P, int32_t D, int32_t ldz,
                      int32_t nproj, int32_t proj, hipStream_t st, bool as_fused)
{
    const bool vec = ((D | ldz) & 3) == 0;
    const int nrb = (pd.r_max / nproj + 15) / 16;
    // 16 waves where every compute unit has at most one workgroup, so that what counts is how long one takes; else 4: a
    // workgroup's waves are then as many fewer to start (us, 4 / 16 waves, blocks of 32 tokens: 128 blocks x 1024, rank 64 23.6 /
    // 16.7, 192 27.9 / 27.4, 4096 340 / 379; 128 x 256, rank 16 6.1 / 6.4, 4096 36 / 62; blocks of one token, 4096 x 256, rank 16:
    // 26 / 59).  It also keeps the launch below 2^32 threads, beyond which the grid wraps silently, at any number of
    // blocks: 512 threads each, and no more blocks than tokens (kPlainMaxTokens).
    static_assert(kPlainMaxTokens * 2 * 256 < (int64_t(1) << 32), "the grid of four waves per half block");
    const bool few = pd.ntb <= 128;
#define LOBRA_F32_SHRINK2(NRB, NW, RANGES)                                                                                 \
    do {                                                                                                                   \
        if (vec) shrink_f32_kernel<NRB, NW, true, RANGES><<<2 * pd.ntb, 64 * NW, 0, st>>>(pd, Z, M, s, P, D, ldz, nproj, proj);     \
        else shrink_f32_kernel<NRB, NW, false, RANGES><<<2 * pd.ntb, 64 * NW, 0, st>>>(pd, Z, M, s, P, D, ldz, nproj, proj);        \
    } while (0)
#define LOBRA_F32_SHRINK(NRB)                                  \
    do {                                                       \
        if (as_fused) LOBRA_F32_SHRINK2(NRB, 16, true);        \
        else if (few) LOBRA_F32_SHRINK2(NRB, 16, false);       \
        else LOBRA_F32_SHRINK2(NRB, 4, false);                 \
    } while (0)
    if (nrb <= 1) LOBRA_F32_SHRINK(1);
    else if (nrb <= 2) LOBRA_F32_SHRINK(2);
    else LOBRA_F32_SHRINK(4);
    return hipGetLastError();
}

// -------------------------------------------------------------------------------------------
// gradreduce stage 1: one workgroup per (chunk, 256 columns), wave w owns 64 columns for all tokens of the chunk.  Lane (i, kg)
// loads the four columns 4 i .. of token kg of a group of four tokens: element e feeds MFMA e, whose result columns are
// {4 i + e}, so a lane ends up with four consecutive columns.  "A" = the projected activations, rank i of token kg.
// -------------------------------------------------------------------------------------------
template <int NRB, bool VEC>
__global__ __launch_bounds__(256) void grad_f32_kernel(PlanDev pd, const float* __restrict__ P, const float* __restrict__ Z,
                                                       float* __restrict__ part, int32_t D, int32_t ldz, int32_t nproj,
                                                       int32_t proj, int32_t tiles_a, const float* __restrict__ P2,
                                                       const float* __restrict__ Z2, float* __restrict__ part2, int32_t D2)
{
    // nproj > 1: projection `proj` of a fused call - Z is its column block (row pitch ldz), and of the
    // task's ranks only the window [proj r, (proj + 1) r) is reduced (columns of P, rows of part).
    // One launch can serve two gradients (nproj = 1): column tiles from tiles_a on belong to (P2, Z2, part2, D2).
    int32_t coltile = blockIdx.y;
    if (coltile >= tiles_a) {
        coltile -= tiles_a;
        P = P2;
        Z = Z2;
        part = part2;
        D = ldz = D2;
    }
    const GradChunk c = pd.chunks[blockIdx.x];
    const int32_t r = (pd.rank_off[c.task + 1] - pd.rank_off[c.task]) / nproj;
    const int32_t pofs = proj * r;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i = lane & 15, kg = lane >> 4;
    const int32_t col = coltile * 256 + wave * 64 + 4 * i;
    if (coltile * 256 + wave * 64 >= D) return;          // the wave has no column (it meets no barrier)
    for (int32_t p0 = 0; p0 < r; p0 += 16 * NRB) {
        f32x4 acc[NRB][4];
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[rb][e] = f32x4{0.f, 0.f, 0.f, 0.f};
        const int32_t nrb = min(NRB, (r - p0 + 15) >> 4);           // uniform
        for (int32_t bi = c.tb_begin; bi < c.tb_end; ++bi) {
            const TokenBlock b = pd.tb[bi];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (16 * h >= b.nrows) break;            // uniform
                f32x4 z[4];
                float p[NRB][4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {            // tokens beyond the block: zero in both operands
                    const int32_t tok = 16 * h + 4 * q + kg;
                    const size_t row = size_t(b.row0 + min(tok, b.nrows - 1));
                    z[q] = load4<VEC>(Z + row * ldz, tok < b.nrows ? col : D, D);
#pragma unroll
                    for (int rb = 0; rb < NRB; ++rb) {
                        const int32_t k = p0 + 16 * rb + i;
                        p[rb][q] = (rb < nrb && tok < b.nrows && k < r) ? P[row * pd.r_max + pofs + k] : 0.f;
                    }
                }
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int rb = 0; rb < NRB; ++rb)
                        if (rb < nrb)
#pragma unroll
                            for (int e = 0; e < 4; ++e) acc[rb][e] = mfma4(p[rb][q], z[q][e], acc[rb][e]);
            }
        }
        // acc[rb][e][v]: rank p0 + 16 rb + 4 kg + v, column col + e
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int32_t k = p0 + 16 * rb + 4 * kg + v;
                if (k >= r || col >= D) continue;
                float* dst = part + size_t(c.part_row0 + pofs + k) * D + col;
                if constexpr (VEC) {
                    *reinterpret_cast<f32x4*>(dst) = f32x4{acc[rb][0][v], acc[rb][1][v], acc[rb][2][v], acc[rb][3][v]};
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (col + e < D) dst[e] = acc[rb][e][v];
                }
            }
    }
}

// -------------------------------------------------------------------------------------------
// Both gradients of a batch whose tasks are short in one launch: one workgroup per (task, 64 columns), its NW waves take half blocks
// of tokens in turn and add their sums through LDS in order.  What bounds it: a memory round trip per 16 tokens and wave, next to the
// launch; the second stage that it saves was another launch and the partial sums' way to memory and back (618 tokens of 256 x 256,
// two tasks of rank 8: 4.4 + 6.3 us; the step 29.4 -> 26.7).
// -------------------------------------------------------------------------------------------
template <int NRB, int NW, bool VEC>
__global__ __launch_bounds__(64 * NW) void grad_f32_one_kernel(PlanDev pd, const float* __restrict__ P, const float* __restrict__ Z,
                                                               float* __restrict__ out, int32_t D, int32_t tiles_a,
                                                               const float* __restrict__ P2, const float* __restrict__ Z2,
                                                               float* __restrict__ out2, int32_t D2, int accumulate)
{
    __shared__ __attribute__((aligned(16))) float red[NW][16][64];       // [wave][rank][column]
    // (column tile fastest: workgroups are dealt to the XCDs in turn, and with the task fastest all of one task's would share an XCD where
    //  their number is a multiple of eight: 1316 x 348 x 780, one of 16 tasks with tokens, gradients 24 us, like this 15)
    int32_t coltile = blockIdx.x;
    if (coltile >= tiles_a) {
        coltile -= tiles_a;
        P = P2;
        Z = Z2;
        out = out2;
        D = D2;
    }
    const int32_t t = blockIdx.y, tb0 = pd.task_tb_off[t], nb = pd.task_tb_off[t + 1] - tb0;
    const int32_t r0 = pd.rank_off[t], r = pd.rank_off[t + 1] - r0;
    if (nb == 0 && accumulate) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6)), i = lane & 15, kg = lane >> 4;
    const int32_t col = coltile * 64 + 4 * i;
    for (int32_t p0 = 0; p0 < r; p0 += 16 * NRB) {
        f32x4 acc[NRB][4];
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[rb][e] = f32x4{0.f, 0.f, 0.f, 0.f};
        const int32_t nrb = min(NRB, (r - p0 + 15) >> 4);           // uniform
        for (int32_t it = wave; it < 2 * nb; it += NW) {            // the first halves of all blocks, then the second ones
            const int32_t h = it >= nb ? 16 : 0;
            const TokenBlock b = pd.tb[tb0 + (it >= nb ? it - nb : it)];
            if (h >= b.nrows) continue;              // uniform
            f32x4 z[4];
            float p[NRB][4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {            // tokens beyond the block: zero in both operands
                const int32_t tok = h + 4 * q + kg;
                const size_t row = size_t(b.row0 + min(tok, b.nrows - 1));
                z[q] = load4<VEC>(Z + row * D, tok < b.nrows ? col : D, D);
#pragma unroll
                for (int rb = 0; rb < NRB; ++rb) {
                    const int32_t k = p0 + 16 * rb + i;
                    p[rb][q] = (rb < nrb && tok < b.nrows && k < r) ? P[row * pd.r_max + k] : 0.f;
                }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int rb = 0; rb < NRB; ++rb)
                    if (rb < nrb)
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[rb][e] = mfma4(p[rb][q], z[q][e], acc[rb][e]);
        }
        // acc[rb][e][v]: rank p0 + 16 rb + 4 kg + v, column col + e
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) {
            if (rb >= nrb) break;                    // uniform
            __syncthreads();
#pragma unroll
            for (int v = 0; v < 4; ++v)
                *reinterpret_cast<f32x4*>(&red[wave][4 * kg + v][4 * i]) = f32x4{acc[rb][0][v], acc[rb][1][v], acc[rb][2][v], acc[rb][3][v]};
            __syncthreads();
            for (int e = threadIdx.x; e < 16 * 64; e += 64 * NW) {
                const int32_t k = p0 + 16 * rb + e / 64, c = coltile * 64 + e % 64;
                float sum = red[0][e / 64][e % 64];
#pragma unroll
                for (int w = 1; w < NW; ++w) sum += red[w][e / 64][e % 64];
                if (k >= r || c >= D) continue;
                float* dst = out + size_t(r0 + k) * D + c;
                *dst = accumulate ? *dst + sum : sum;
            }
        }
    }
}

hipError_t grad_f32_one(const PlanDev& pd, const GradJob& ja, const GradJob& jb, bool accumulate, hipStream_t st)
{
    const int32_t tiles_a = (ja.D + 63) / 64, tiles_b = (jb.D + 63) / 64;
    const dim3 grid(tiles_a + tiles_b, pd.n_tasks);
    if (grid.y > 65535u) return hipErrorInvalidValue;
    const bool vec = ((ja.D | jb.D) & 3) == 0;
    const int nrb = (pd.r_max + 15) / 16;
#define LOBRA_F32_ONE2(NRB, NW, VEC)                                                                                         \
    grad_f32_one_kernel<NRB, NW, VEC><<<grid, 64 * NW, 0, st>>>(pd, (const float*)ja.P, (const float*)ja.Z, ja.out, ja.D, tiles_a, \
                                                                (const float*)jb.P, (const float*)jb.Z, jb.out, jb.D, accumulate ? 1 : 0)
#define LOBRA_F32_ONE(NRB, NW) do { if (vec) LOBRA_F32_ONE2(NRB, NW, true); else LOBRA_F32_ONE2(NRB, NW, false); } while (0)
    if (nrb <= 1) LOBRA_F32_ONE(1, 16);
    else if (nrb <= 2) LOBRA_F32_ONE(2, 16);
    else LOBRA_F32_ONE(4, 8);
    return hipGetLastError();
}

hipError_t grad_f32_stage1(const PlanDev& pd, const float* P, const float* Z, float* part, int32_t D, int32_t ldz, int32_t nproj,
                           int32_t proj, const float* P2, const float* Z2, float* part2, int32_t D2, hipStream_t st)
{
    const int32_t tiles_a = (D + 255) / 256, tiles_b = P2 ? (D2 + 255) / 256 : 0;
    const dim3 grid(pd.nchunks, tiles_a + tiles_b);
    if (grid.y > 65535u) return hipErrorInvalidValue;
    const bool vec = ((D | ldz | (P2 ? D2 : 0)) & 3) == 0;
    const int nrb = (pd.r_max / nproj + 15) / 16;
#define LOBRA_F32_GRAD(NRB)                                                                                                  \
    do {                                                                                                                     \
        if (vec) grad_f32_kernel<NRB, true><<<grid, 256, 0, st>>>(pd, P, Z, part, D, ldz, nproj, proj, tiles_a, P2, Z2, part2, D2); \
        else grad_f32_kernel<NRB, false><<<grid, 256, 0, st>>>(pd, P, Z, part, D, ldz, nproj, proj, tiles_a, P2, Z2, part2, D2);    \
    } while (0)
    if (nrb <= 1) LOBRA_F32_GRAD(1);
    else if (nrb <= 2) LOBRA_F32_GRAD(2);
    else LOBRA_F32_GRAD(4);
    return hipGetLastError();
}

}  // namespace lobra

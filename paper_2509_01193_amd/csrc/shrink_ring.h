// The rank-r projection through an LDS ring, as a device function: a kernel of its own (shrink_ring.hip, which says what bounds it)
// and a part of the split product's launch (gemm_tile.hip).
#pragma once
#include "gemm_common.h"
#include "kernels.h"

namespace lobra {

using namespace gemm;

namespace {

// G token blocks of one task, or (H = 1) a half of one, per workgroup of four waves, which share K where G < 4.  A slot of the ring holds KS
// k as K tiles of 64: [KS / 64][16 H G token rows, then 16 NRB rank rows][64 k], 128 bytes per row, swizzled as in the GEMMs.
// the ranks p0 .. plim - 1 of halves h0 .. h1 - 1 of a block, where there is nothing but padding; one wave
__device__ __forceinline__ void store_zeros(const PlanDev& pd, uint16_t* __restrict__ P_tok, uint16_t* __restrict__ P_blk, const TokenBlock& b,
                                            int32_t bi, int32_t h0, int32_t h1, int32_t pofs, int32_t p0, int32_t plim, int lane)
{
    for (int32_t p = p0 + 4 * (lane >> 4); p < plim; p += 16)
        for (int h = h0; h < h1; ++h) {
            const int32_t tok = 16 * h + (lane & 15);
            if (tok < b.nrows) *reinterpret_cast<uint64_t*>(P_tok + size_t(b.row0 + tok) * pd.r_pad + pofs + p) = 0;
            for (int v = 0; v < 4; ++v) P_blk[(size_t(bi) * pd.r_pad + pofs + p + v) * kTokenBlock + tok] = 0;
        }
}

template <int G, int H, int NRB, int KS, int LDS>
__device__ __forceinline__ void ring_body(const PlanDev& pd, const uint16_t* __restrict__ Z, const uint16_t* __restrict__ M,
                                          const float* __restrict__ s, uint16_t* __restrict__ P_tok, uint16_t* __restrict__ P_blk,
                                          int32_t D, int32_t ldz, int32_t pofs, int32_t r, int32_t plim, int32_t tb0, int32_t cnt,
                                          const TokenBlock& b, int32_t half0, unsigned char* lds)
{
    constexpr int WK = 4 / G;                        // waves per token block
    constexpr int SUB = KS / 64, ROWS = 16 * H * G, KTILE = (ROWS + 16 * NRB) * 128, SLOT = SUB * KTILE;
    constexpr int STAGES = LDS / SLOT < 8 ? LDS / SLOT : 8;
    static_assert(STAGES >= 2, "a ring");
    constexpr int ZC = SUB * G * H / 2;              // copies of 8 rows per wave and slot: token rows
    constexpr int AP = 2 * NRB * SUB, AC = (AP + 3) / 4;     // pieces of the rank rows; copies of them per wave
    static_assert((AP % 4 == 0 || AP == 2) && ZC * 2 == SUB * G * H && (G == 1 || (H == 2 && SUB == 1)), "whole copies");
    constexpr int CPW = ZC + AC, STEPS = KS / 32 / WK;       // copies, K steps of 32 per wave and slot
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    const int blk = wave % G, wk = wave / G;
    const int j = lane & 15, kg = lane >> 4;
    const uint32_t lds0 = uint32_t(uintptr_t((__attribute__((address_space(3))) unsigned char*)lds));

    // ---- copies: rows beyond a block repeat its last one, rank rows beyond r_t the last one (what they produce is dropped)
    const unsigned char* zcur = reinterpret_cast<const unsigned char*>(Z + size_t(b.row0) * ldz);
    const unsigned char* mcur = reinterpret_cast<const unsigned char*>(M + size_t(b.rank_row0 + pofs) * D);
    uint32_t zvo[ZC], avo[AC], zat[ZC], aat[AC];
    int32_t zk[ZC], ak[AC];                          // first k of the lane's chunk within the slot
#pragma unroll
    for (int c = 0; c < ZC; ++c) {
        // (copy c of a wave: 8 rows that are the same for all c where G = 1, K tile sub of the slot)
        const int sub = G == 1 ? (wk + 4 * c) / (2 * H) : 0, q = G == 1 ? wk % (2 * H) : c, row = 8 * q + lane / 8;
        zk[c] = 64 * sub + 8 * ((lane % 8) ^ swz_row(row));
        zvo[c] = (uint32_t(min(16 * half0 + row, b.nrows - 1)) * uint32_t(ldz) + uint32_t(zk[c])) * 2u;
        zat[c] = lds0 + sub * KTILE + (16 * H * blk + 8 * q) * 128;
    }
#pragma unroll
    for (int c = 0; c < AC; ++c) {
        const int q = (wave + 4 * c) % AP, sub = q / (2 * NRB), row = 8 * (q % (2 * NRB)) + lane / 8;
        ak[c] = 64 * sub + 8 * ((lane % 8) ^ swz_row(row));
        avo[c] = (uint32_t(min(row, r - 1)) * uint32_t(D) + uint32_t(ak[c])) * 2u;
        aat[c] = lds0 + sub * KTILE + (ROWS + 8 * (q % (2 * NRB))) * 128;
    }
    const int32_t n = (D + KS - 1) / KS, ktail = D % KS;
    // G = 1: a wave copies 8 of the token rows, and none if the block ends before them (one-token blocks of a decoding batch)
    const bool no_rows = G == 1 && 16 * half0 + 8 * (wk % (2 * H)) >= b.nrows;
    auto copy_slot = [&](int32_t i, uint32_t slot) __attribute__((always_inline)) {
        const uint32_t at = slot * SLOT;
        // (uniform) Chunks beyond D repeat the last one: with as many copies as the others the last slot is waited for by count like
        // them (without, everything was waited for as soon as it was on its way: 1504 columns, 81 blocks of rank 64 10.0 -> 9.0 us,
        // 141 one-token blocks of rank 16 7.7 -> 7.3; 4104, 81 blocks of rank 128 20.0 -> 19.4)
        if (ktail && i + 1 == n) {
            if (!no_rows)
#pragma unroll
                for (int c = 0; c < ZC; ++c) dma16(zat[c] + at, zcur, zvo[c] - 2u * uint32_t(max(zk[c] - (ktail - 8), 0)));
#pragma unroll
            for (int c = 0; c < AC; ++c) dma16(aat[c] + at, mcur, avo[c] - 2u * uint32_t(max(ak[c] - (ktail - 8), 0)));
        } else {
            if (!no_rows)
#pragma unroll
                for (int c = 0; c < ZC; ++c) dma16(zat[c] + at, zcur, zvo[c]);
#pragma unroll
            for (int c = 0; c < AC; ++c) dma16(aat[c] + at, mcur, avo[c]);
        }
        zcur += KS * 2;
        mcur += KS * 2;
    };

    f32x4 acc[H][NRB];
#pragma unroll
    for (int h = 0; h < H; ++h)
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) acc[h][rb] = f32x4{0.f, 0.f, 0.f, 0.f};
    const u32x4 zero4 = {0u, 0u, 0u, 0u};
    const int sw = swz_row(j);
    // K step q of a slot: k 32 q + 8 kg .. + 7 per lane
    auto mac = [&](const unsigned char* st, int q, bool tail) __attribute__((always_inline)) {
        const unsigned char* zp = st + (q >> 1) * KTILE + (16 * H * blk + j) * 128 + (((4 * (q & 1) + kg) ^ sw) << 4);
        const unsigned char* ap = zp + 16 * H * (G - blk) * 128;
        u32x4 zf[H], af[NRB];
#pragma unroll
        for (int h = 0; h < H; ++h) zf[h] = *reinterpret_cast<const u32x4*>(zp + h * 2048);
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) af[rb] = *reinterpret_cast<const u32x4*>(ap + rb * 2048);
        if (tail) {                                  // (uniform) what lies beyond D belongs to other k, perhaps no finite one
            const bool in = 32 * q + 8 * kg < ktail;
#pragma unroll
            for (int h = 0; h < H; ++h) zf[h] = in ? zf[h] : zero4;
#pragma unroll
            for (int rb = 0; rb < NRB; ++rb) af[rb] = in ? af[rb] : zero4;
        }
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
            for (int h = 0; h < H; ++h)
                acc[h][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(af[rb]), as_bf16x8(zf[h]), acc[h][rb], 0, 0, 0);
    };

    for (int32_t i = 0; i < STAGES - 1 && i < n; ++i) copy_slot(i, uint32_t(i));
    uint32_t slot = 0, fill = STAGES - 1;
    for (int32_t i = 0; i < n; ++i) {
        // this slot's copies have landed
        if (i + STAGES - 1 > n) wait_vmcnt<0>();
        else if (no_rows) wait_vmcnt<(STAGES - 2) * AC>();
        else wait_vmcnt<(STAGES - 2) * CPW>();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();                // and everybody is done with the slot before, which is filled next
        asm volatile("" ::: "memory");
        if (i + STAGES - 1 < n) copy_slot(i + STAGES - 1, fill);
        const unsigned char* st = lds + slot * SLOT;
        const bool tail = ktail != 0 && i + 1 == n;
#pragma unroll
        for (int q = 0; q < STEPS; ++q)              // (the same sums whatever KS is)
            if (!tail || 32 * (wk + WK * q) < ktail) mac(st, wk + WK * q, tail);
        slot = slot + 1 == STAGES ? 0 : slot + 1;
        fill = fill + 1 == STAGES ? 0 : fill + 1;
    }
    // ---- the waves of a block add their sums through LDS in order; wave wk keeps the rank blocks wk, wk + WK, ...
    if constexpr (WK > 1) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __syncthreads();
        f32x4* red = reinterpret_cast<f32x4*>(lds);  // [wave][half][rank block][lane]
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
            for (int rb = 0; rb < NRB; ++rb) red[((wave * H + h) * NRB + rb) * 64 + lane] = acc[h][rb];
        __syncthreads();
    }
    if (blk >= cnt) return;
    const float st = s[b.task];
    const int32_t bi = tb0 + blk;
#pragma unroll
    for (int h = 0; h < H; ++h) {
        const int32_t tok = 16 * (half0 + h) + j;
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) {
            if (WK > 1 && (h * NRB + rb) % WK != wk) continue;
            f32x4 sum = acc[h][rb];
            if constexpr (WK > 1) {
                const f32x4* red = reinterpret_cast<const f32x4*>(lds);
                sum = red[((blk * H + h) * NRB + rb) * 64 + lane];
#pragma unroll
                for (int w = 1; w < WK; ++w) sum = sum + red[(((w * G + blk) * H + h) * NRB + rb) * 64 + lane];
            }
            const int32_t p0 = 16 * rb + 4 * kg;
            bf16x4 o;
#pragma unroll
            for (int v = 0; v < 4; ++v) o[v] = (__bf16)((p0 + v < r && tok < b.nrows) ? st * sum[v] : 0.f);
            if (p0 >= plim) continue;
            if (tok < b.nrows) *reinterpret_cast<bf16x4*>(P_tok + size_t(b.row0 + tok) * pd.r_pad + pofs + p0) = o;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                union { __bf16 b; uint16_t u; } c;
                c.b = o[v];
                P_blk[(size_t(bi) * pd.r_pad + pofs + p0 + v) * kTokenBlock + tok] = c.u;
            }
        }
    }
    if (wk == 0) store_zeros(pd, P_tok, P_blk, b, bi, half0, half0 + H, pofs, 16 * NRB, plim, lane);
}


// Item wi (a token block, or at G = 4 a run of them) of column `col`.  rparts: the widest rank window is dealt to that many workgroups, 16 MAXNRB ranks each (col = part + rparts * projection; H = 1: twice
// that, and the half).
// nproj > 1 (fused shared-input projections): a workgroup handles one projection only, `proj` or (proj < 0, Z is all of dy) the one in
// col - Z is that projection's column block of dy (row pitch ldz), M its rows of the compact up factors, and the task's rank
// rows it reads and writes are the window [proj r, (proj + 1) r).
template <int G, int H, int MAXNRB, int KS, int LDS>
__device__ __forceinline__ void ring_item(const PlanDev& pd, const uint16_t* __restrict__ Z, const uint16_t* __restrict__ M,
                                          const float* __restrict__ s, uint16_t* __restrict__ P_tok, uint16_t* __restrict__ P_blk,
                                          int32_t D, int32_t ldz, int32_t nproj, int32_t proj, int32_t rparts, int32_t wi, int32_t col,
                                          unsigned char* ring)
{
    const int32_t items = G == 4 ? pd.nsb : pd.ntb, half0 = H == 1 ? col & 1 : 0, y = col / (2 / H);
    if (wi >= items) return;
    if (proj < 0) {
        proj = y / rparts;
        Z += size_t(proj) * D;
    }
    // (a launch order by rank is dealt round-robin: contiguous ranges of it would give one XCD all the expensive blocks)
    const int32_t* order = G == 4 ? pd.sb_order : pd.tb_order;
    const int32_t run = order ? order[wi] : xcd_contiguous(wi, items);
    const int32_t tb0 = G == 4 ? pd.sb_off[run] : run;
    const int32_t cnt = G == 4 ? pd.sb_off[run + 1] - tb0 : 1;
    const int32_t mine = min(__builtin_amdgcn_readfirstlane(int32_t(threadIdx.x >> 6)) % G, cnt - 1);
    const TokenBlock b = pd.tb[tb0 + mine];
    const int32_t rw = (pd.rank_off[b.task + 1] - b.rank_row0) / nproj;
    // this part's ranks: r of them from pofs on (of the task's rank rows), and what it stores: plim, with the zero padding beyond
    const int32_t part = y % rparts, first = 16 * MAXNRB * part;
    const int32_t pofs = proj * rw + first, r = min(rw - first, 16 * MAXNRB);
    const int32_t wlim = (proj == nproj - 1 ? pd.r_pad - proj * rw : rw) - first;
    const int32_t plim = part == rparts - 1 ? wlim : min(wlim, 16 * MAXNRB);
    if (plim <= 0) return;
    const int32_t nrb = r <= 0 ? 0 : (r + 15) >> 4;  // (the same for all blocks of a run)
#define LOBRA_RING(NRB) ring_body<G, H, NRB, KS, LDS>(pd, Z, M, s, P_tok, P_blk, D, ldz, pofs, r, plim, tb0, cnt, b, half0, ring)
    if (nrb == 0 || (H == 1 && 16 * half0 >= b.nrows)) {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        if (wave < cnt) store_zeros(pd, P_tok, P_blk, b, tb0 + wave, half0, half0 + H, pofs, 0, plim, lane);
    } else if (MAXNRB == 1 || nrb == 1) {
        LOBRA_RING(1);
    } else if (MAXNRB == 2 || nrb <= 2) {
        if constexpr (MAXNRB >= 2) LOBRA_RING(2);
    } else if constexpr (MAXNRB >= 4) {
        if (MAXNRB == 4 || nrb <= 4) LOBRA_RING(4);
        else if constexpr (MAXNRB > 4) LOBRA_RING(8);
    }
#undef LOBRA_RING
}

}  // namespace

}  // namespace lobra

// Validation of the problem descriptor and construction of the host-side work lists.
// The lists turn the packed batch's segment table (paper section 1: a fused batch holds the
// sequences of several tasks, each tagged with its task) into what the kernels iterate over.
#include "plan.h"

#include <algorithm>
#include <cstring>
#include <new>

namespace lobra {

static inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

lobra_status validate(const lobra_mlora_desc* d)
{
    if (!d) return LOBRA_ERR_NULL;
    if (d->dtype != LOBRA_F32 && d->dtype != LOBRA_BF16) return LOBRA_ERR_DTYPE;
    if (d->T < 0 || d->T >= (int64_t(1) << 31)) return LOBRA_ERR_SHAPE;
    if (d->d_in < 1 || d->d_out < 1 || d->n_tasks < 0 || d->S < 0) return LOBRA_ERR_SHAPE;
    // what the kernels' launch grids and 32-bit offsets inside a tile can address (checked here so that
    // no call fails after its first launch): widths, and the number of 256 x 256 output tiles
    if (d->d_in > LOBRA_MAX_WIDTH || d->d_out > LOBRA_MAX_WIDTH) return LOBRA_ERR_SHAPE;
    {
        const int64_t tiles_m = (d->T + 255) / 256, tiles_n = (int64_t(d->d_in > d->d_out ? d->d_in : d->d_out) + 255) / 256;
        if (tiles_m * tiles_n > 0x7fffffff) return LOBRA_ERR_SHAPE;
    }
    if (d->dtype == LOBRA_F32 && d->T > kPlainMaxTokens) return LOBRA_ERR_SHAPE;
    if (d->S == 0 && d->T != 0) return LOBRA_ERR_SEGMENTS;
    if (d->dtype == LOBRA_BF16 && (d->d_in % 8 != 0 || d->d_out % 8 != 0)) return LOBRA_ERR_ALIGN;
    if (d->n_proj < 0 || d->n_proj > 16) return LOBRA_ERR_SHAPE;
    const int32_t P = d->n_proj > 1 ? d->n_proj : 1;
    if (P > 1 && d->d_out % (8 * P) != 0) return LOBRA_ERR_ALIGN;
    if (d->n_tasks > 0) {
        if (!d->rank_off) return LOBRA_ERR_NULL;
        if (d->rank_off[0] != 0) return LOBRA_ERR_RANK;
        for (int32_t t = 0; t < d->n_tasks; ++t) {
            const int64_t r = int64_t(d->rank_off[t + 1]) - d->rank_off[t];
            if (r < 1 || r > LOBRA_MAX_RANK) return LOBRA_ERR_RANK;
            if (P > 1 && r % (8 * P) != 0) return LOBRA_ERR_RANK;
        }
    }
    if (d->S > 0) {
        if (!d->seg_off || !d->seg_task) return LOBRA_ERR_NULL;
        if (d->seg_off[0] != 0) return LOBRA_ERR_SEGMENTS;
        for (int32_t k = 0; k < d->S; ++k)
            if (d->seg_off[k + 1] < d->seg_off[k]) return LOBRA_ERR_SEGMENTS;
        if (int64_t(d->seg_off[d->S]) != d->T) return LOBRA_ERR_SEGMENTS;
        for (int32_t k = 0; k < d->S; ++k)
            if (d->seg_task[k] < -1 || d->seg_task[k] >= d->n_tasks) return LOBRA_ERR_TASK_ID;
    }
    return LOBRA_OK;
}

lobra_status build_host_plan(const lobra_mlora_desc* d, uint32_t flags, Plan* p)
{
    try {
        p->desc = *d;
        p->flags = flags;
        p->mfma = kMfmaKernels && d->dtype == LOBRA_BF16 && !(flags & LOBRA_PLAN_PLAIN_KERNELS);
        if (!p->mfma && d->T > kPlainMaxTokens) return LOBRA_ERR_SHAPE;   // the plain kernels' grid
        p->n_proj = d->n_proj > 1 ? d->n_proj : 1;
        p->dg = d->d_out / p->n_proj;

        const int32_t n = d->n_tasks;
        p->rank_off.assign(size_t(n) + 1, 0);
        for (int32_t t = 0; t <= n && n > 0; ++t) p->rank_off[t] = d->rank_off[t];
        p->R_tot = p->rank_off[n];
        p->r_max = 0;
        for (int32_t t = 0; t < n; ++t)
            p->r_max = std::max(p->r_max, p->rank_off[t + 1] - p->rank_off[t]);
        p->r_pad = (p->r_max + 15) / 16 * 16;
        p->seg_off_in.assign(d->seg_off ? d->seg_off : nullptr,
                             d->seg_off ? d->seg_off + d->S + 1 : nullptr);
        p->seg_task_in.assign(d->seg_task ? d->seg_task : nullptr,
                              d->seg_task ? d->seg_task + d->S : nullptr);
        p->desc.rank_off = p->rank_off.data();
        p->desc.seg_off = p->seg_off_in.data();
        p->desc.seg_task = p->seg_task_in.data();

        // 1. compacted table: no empty segments, no two neighbours with the same task
        p->cseg_off.assign(1, 0);
        p->cseg_task.clear();
        for (int32_t k = 0; k < d->S; ++k) {
            const int32_t len = d->seg_off[k + 1] - d->seg_off[k];
            if (len == 0) continue;
            if (!p->cseg_task.empty() && p->cseg_task.back() == d->seg_task[k]) {
                p->cseg_off.back() += len;
            } else {
                p->cseg_task.push_back(d->seg_task[k]);
                p->cseg_off.push_back(p->cseg_off.back() + len);
            }
        }
        const int32_t nseg = int32_t(p->cseg_task.size());
        const int32_t T = int32_t(d->T);

        // 2. first segment of every 32-row block
        const int32_t nrb = (T + kRowBlock - 1) / kRowBlock;
        p->rowblk_seg.assign(size_t(nrb), 0);
        for (int32_t b = 0, k = 0; b < nrb; ++b) {
            while (p->cseg_off[k + 1] <= b * kRowBlock) ++k;
            p->rowblk_seg[b] = k;
        }

        // 2b. the segments that cross every tile row of the MFMA kernels' products
        p->gemm_tile_seg.clear();
        if (d->dtype == LOBRA_BF16) {
            const int32_t ntr = (T + kGemmTileRows - 1) / kGemmTileRows;
            p->gemm_tile_seg.assign(size_t(ntr) * kGemmTileSegRec, 0);
            for (int32_t i = 0, k = 0; i < ntr; ++i) {
                const int32_t row0 = std::max(0, std::min(i * kGemmTileRows, T - kGemmTileRows));
                while (p->cseg_off[k + 1] <= row0) ++k;      // row0 does not decrease with i
                int32_t* seg = &p->gemm_tile_seg[size_t(i) * kGemmTileSegRec];
                const int32_t row_end = std::min(row0 + kGemmTileRows, T);
                int32_t g = k, found = 0;
                for (; g < nseg && p->cseg_off[g] < row_end && found < kGemmTileSegs; ++g) {
                    const int32_t gt = p->cseg_task[g];
                    if (gt < 0) continue;
                    int32_t* e = seg + 4 * found++;
                    e[0] = p->cseg_off[g];
                    e[1] = p->cseg_off[g + 1];
                    e[2] = p->rank_off[gt];
                    e[3] = p->rank_off[gt + 1] - p->rank_off[gt];
                }
                seg[4 * kGemmTileSegs] = g;
            }
        }

        // 3. token blocks, grouped by task (counting sort keeps token order inside a task)
        p->task_tb_off.assign(size_t(n) + 1, 0);
        for (int32_t k = 0; k < nseg; ++k) {
            const int32_t t = p->cseg_task[k];
            if (t < 0) continue;
            const int32_t len = p->cseg_off[k + 1] - p->cseg_off[k];
            p->task_tb_off[t + 1] += (len + kTokenBlock - 1) / kTokenBlock;
        }
        for (int32_t t = 0; t < n; ++t) p->task_tb_off[t + 1] += p->task_tb_off[t];
        p->tb.assign(size_t(p->task_tb_off[n]), TokenBlock{0, 0, 0, 0});
        {
            std::vector<int32_t> cur(p->task_tb_off.begin(), p->task_tb_off.end() - (n >= 0 ? 1 : 0));
            for (int32_t k = 0; k < nseg; ++k) {
                const int32_t t = p->cseg_task[k];
                if (t < 0) continue;
                for (int32_t r0 = p->cseg_off[k]; r0 < p->cseg_off[k + 1]; r0 += kTokenBlock) {
                    const int32_t nr = std::min(kTokenBlock, p->cseg_off[k + 1] - r0);
                    p->tb[size_t(cur[t]++)] = TokenBlock{r0, nr, t, p->rank_off[t]};
                }
            }
        }

        // 3b. runs of token blocks that one workgroup of the rank-r projection handles.  From rank 24 or
        //     so the adapter rows are most of what a single token block's workgroup reads (r_t rows
        //     per 32 token rows), so long batches are projected in runs of four blocks that share the
        //     rows staged in LDS; otherwise every block is its own run.
        {
            int64_t wsum = 0;                      // token-block-weighted sum of ranks
            const int64_t ntb_all = p->task_tb_off[n];
            for (int32_t t = 0; t < n; ++t)
                wsum += int64_t(p->task_tb_off[t + 1] - p->task_tb_off[t]) * (p->rank_off[t + 1] - p->rank_off[t]);
            const int32_t g = (p->mfma && ntb_all >= 1024 && wsum >= 24 * ntb_all) ? 4 : 1;
            p->shrink_group = g;
            p->sb_off.assign(1, 0);
            for (int32_t t = 0; t < n; ++t)
                for (int32_t b = p->task_tb_off[t]; b < p->task_tb_off[t + 1]; b += g)
                    p->sb_off.push_back(std::min(b + g, p->task_tb_off[t + 1]));
            // 3c. launch order of the projection's workgroups by descending rank.  A workgroup's cost grows with
            //     its task's rank (the adapter rows it reads next to its 32 token rows), and the lists above are
            //     in task order, so with mixed ranks whichever task comes last would make up the launch's tail.
            //     (Inside a rank the stored, task-grouped order stays: ordering the blocks by their position in
            //     the batch as well measured 2 us slower on the shuffled workload 2, although the kernels deal
            //     their work items to the XCDs in contiguous ranges.)
            auto by_rank = [&](size_t count, auto task_of, std::vector<int32_t>& order) {
                order.resize(count);
                for (size_t i = 0; i < count; ++i) order[i] = int32_t(i);
                auto rank_of = [&](int32_t i) { const int32_t t = task_of(i); return p->rank_off[t + 1] - p->rank_off[t]; };
                std::stable_sort(order.begin(), order.end(),
                                 [&](int32_t a, int32_t b) { return rank_of(a) > rank_of(b); });
                bool identity = true;
                for (size_t i = 0; i < count && identity; ++i) identity = order[i] == int32_t(i);
                if (identity) order.clear();
            };
            by_rank(p->tb.size(), [&](int32_t i) { return p->tb[size_t(i)].task; }, p->tb_order);
            by_rank(p->sb_off.size() - 1, [&](int32_t i) { return p->tb[size_t(p->sb_off[size_t(i)])].task; }, p->sb_order);
        }

        // 3d. the K-sliced projection of dy (long batches, ranks up to 16) and whether dB rides with its pass over dy
        p->sliced_out = SlicedShape{};
        if (p->mfma && !p->tb.empty() && p->n_proj == 1) p->sliced_out = sliced_shrink_shape(int64_t(p->tb.size()), p->r_pad, d->d_out);
        // dB fused into the sliced projection of dy: the runs of (task, slice) that every workgroup meets, by
        // the same split of the items as the kernel's (shrink_sliced_kernel)
        p->fused_db = false;
        p->fb_wg_run_off.clear();
        p->fb_run_row.clear();
        p->fb_cnt.clear();
        p->fb_task_row0.clear();
        p->fb_rows = 0;
        if (p->sliced_out.nsl > 0) {
            const int32_t nsl = p->sliced_out.nsl, per_xcd = kSlicedGrid / 8, ntb32 = int32_t(p->tb.size());
            std::vector<int32_t> run_task, run_k;
            p->fb_cnt.assign(size_t(n) * nsl, 0);
            p->fb_wg_run_off.assign(1, 0);
            for (int32_t wg = 0; wg < kSlicedGrid; ++wg) {
                const int32_t xcd = wg & 7, idx = wg >> 3;
                const int32_t bx0 = int32_t((int64_t(ntb32) * xcd) >> 3), bx1 = int32_t((int64_t(ntb32) * (xcd + 1)) >> 3);
                const int32_t nbx = bx1 - bx0;
                const int64_t nit = int64_t(nbx) * nsl;
                int64_t e = nit * idx / per_xcd;
                const int64_t e1 = nit * (idx + 1) / per_xcd;
                while (e < e1) {
                    const int32_t sl = int32_t(e / nbx), bo = int32_t(e - int64_t(sl) * nbx);
                    const int32_t t = p->tb[size_t(bx0 + bo)].task;
                    // the run ends with the workgroup's range, the slice, or the task's blocks inside the piece
                    const int64_t task_end = int64_t(sl) * nbx + std::min<int64_t>(nbx, p->task_tb_off[t + 1] - bx0);
                    const int64_t next = std::min(e1, task_end);
                    run_task.push_back(t);
                    run_k.push_back(p->fb_cnt[size_t(t) * nsl + sl]++);
                    e = next;
                }
                p->fb_wg_run_off.push_back(int32_t(run_task.size()));
            }
            p->fb_task_row0.assign(size_t(n), 0);
            int64_t rows = 0;
            for (int32_t t = 0; t < n; ++t) {
                int32_t most = 0;
                for (int32_t sl = 0; sl < nsl; ++sl) most = std::max(most, p->fb_cnt[size_t(t) * nsl + sl]);
                p->fb_task_row0[t] = int32_t(rows);
                rows += int64_t(most) * 16;
            }
            // worth it while the partial sums stay a small part of the pass over dy (4 bytes x rows per column,
            // written and read once, against 2 bytes x T)
            if (rows > 0 && rows <= int64_t(T) / 8 && rows < 0x7fffffff / 2) {
                p->fused_db = true;
                p->fb_rows = int32_t(rows);
                p->fb_run_row.resize(run_task.size());
                for (size_t i = 0; i < run_task.size(); ++i)
                    p->fb_run_row[i] = p->fb_task_row0[run_task[i]] + 16 * run_k[i];
            } else {                         // (shrink_sliced_kernel says why the projection goes without slices then)
                p->sliced_out = SlicedShape{};
                p->fb_wg_run_off.clear();
                p->fb_cnt.clear();
                p->fb_task_row0.clear();
            }
        }
        // 4. reduction chunks: runs of token blocks of one task.  The chunk length is chosen so
        //    that (chunks x 128-column tiles) gives roughly a thousand workgroups, within
        //    [4, 64] token blocks ([1, 64] on the plain path); fewer, longer chunks mean less partial-sum traffic.
        const int64_t coltiles = (std::min(d->d_in, d->d_out) + 127) / 128;
        int64_t cb = (int64_t(T) * coltiles / 1024 + kTokenBlock - 1) / kTokenBlock;
        // (fp32: some hundred workgroups of 256 columns, whose waves share no work; shorter chunks make more partial
        //  sums than they are worth, longer ones a longer stage 1: chunks of 1 / 3 blocks at 3000 x 1024 x 1024 21 / 19 us for both
        //  stages, of 4 / 16 blocks at 8192 x 2048 x 2048 33 / 48 us)
        if (!p->mfma) cb = (int64_t(T) * coltiles / 512 + kTokenBlock - 1) / kTokenBlock;
        // Where dB rides with the projection of dy, stage 1 is one short launch for dA alone and what counts is
        // its balance: three workgroups per compute unit (at workload 2: 24 chunks of 21 or 22 blocks, 27.9 us,
        // against 36 of 16 or 3 blocks, 30.8 us; and a quarter fewer partial sums for stage 2)
        if (p->fused_db) cb = (int64_t(p->tb.size()) * ((d->d_in + 127) / 128) + 767) / 768;
        // (the MFMA kernel gives each of its four waves a token block of the chunk at a time; the plain
        //  kernel walks a chunk's tokens one after the other, so small batches want short chunks there)
        cb = std::max<int64_t>(p->mfma ? 4 : 1, std::min<int64_t>(64, cb));
        // fp32, short tasks: no partial sums and no second stage (grad_f32_one), while a task's blocks times the rank blocks are few: a
        // launch lasts as long as its longest chain of them.  Training steps, two stages / one, us, with n blocks in the largest task:
        //   rank 16   256 x 256, n = 13 29.4 / 26.7, 30 35.7 / 32.7, 39 64.7 / 62.3, 53 41.8 / 42.8; 1024 x 1024, n = 13 69.2 / 64.7, 31 107.5 /
        //             105.2, 57 161.6 / 162.2; 1999 x 500, n = 30 129.7 / 121.5
        //   rank 32   256 x 256, n = 10 34.9 / 32.3, 30 40.0 / 42.3;  rank 64  n = 4 39.9 / 36.7, 22 50.7 / 56.7;  rank 128  n = 13 64.1 / 69.6
        // (tasks within what the grid takes)
        p->f32_items = 0;
        p->fused_fwd = p->fused_bwd = false;
        if (d->dtype == LOBRA_F32 && p->n_proj == 1 && !p->tb.empty() && T <= kFusedTokens) {
            int32_t most = 0;
            for (int32_t b = 0; b < nrb; ++b) {
                int32_t items = 0;
                for (int32_t k = p->rowblk_seg[size_t(b)]; k < nseg && p->cseg_off[size_t(k)] < (b + 1) * kRowBlock; ++k) {
                    const int32_t t = p->cseg_task[size_t(k)];
                    if (t >= 0) items += (p->rank_off[t + 1] - p->rank_off[t] + 15) / 16;
                }
                most = std::max(most, items);
            }
            const int32_t items = most <= 2 ? 2 : most <= 4 ? 4 : 0;
            p->fused_fwd = f32_fused(T, d->d_in, d->d_out, items);
            p->fused_bwd = f32_fused(T, d->d_out, d->d_in, items);
            if (p->fused_fwd || p->fused_bwd) p->f32_items = items;
        }
        p->grad_one = false;
        if (d->dtype == LOBRA_F32 && p->n_proj == 1 && n <= 65535) {
            int64_t most = 0;
            for (int32_t t = 0; t < n; ++t) most = std::max<int64_t>(most, p->task_tb_off[t + 1] - p->task_tb_off[t]);
            p->grad_one = most > 0 && most * ((p->r_max + 15) / 16) <= 32;
        }
        // Small batches: one chunk per task where that is the faster way to the gradients: the sums are then final and there
        // is no second stage (6 us and the partial sums' way to memory and back), but a launch lasts as long as its longest chain
        // of blocks.  Both stages, several chunks per task against one, with n blocks in the largest task (us):
        //   ranks up to 16 (the kernel's four waves take blocks in turn, 128 columns a workgroup): one is better at every measured
        //     point, n = 5 .. 24, 1 .. 16 tasks: 4 tasks, 4096 x 4096, n = 24: 21.9 / 13.5
        //   ranks above 16 (every wave walks all blocks, 256 columns a workgroup: about 1 us a block): up to n = 12 one is better
        //     (4 tasks of rank 24, 4096 x 4096: 19.2 / 16.5; n = 16: 19.2 / 20.1, n = 24: 25.1 / 27.8), and beyond where there are so
        //     many partial sums that writing and adding them costs more: from 12800 rank rows x column tiles on, a task's rows
        //     counted by its share of the largest task's blocks (3 tasks of rank 48, 9216: n = 24 26.5 / 27.5; 4 of 64, 16384: 34.2 / 28.6;
        //     16 of 64: 74.9 / 41.6; one task of 24 blocks and 7 of 4, rank 64, 8832: 23.1 / 29.7; rank 128, 17728: 36.1 / 34.2)
        //   fused projections (dA and dB in launches of their own, each with fewer workgroups): up to n = 10, or from 40960 on
        //     (P = 2, 4096 x 8192, 4 tasks of stacked rank 64: n = 10 30.9 / 30.2, n = 12 31.4 / 33.6; 24576 against 49152, n = 24: 42.4 /
        //     49.5 and 61.5 / 53.1); where dB takes a launch per projection, up to n = 6 (P = 3, 2048 x 3192, 8 tasks of stacked rank
        //     24 and 96: n = 6 35.0 / 33.2 and 48.4 / 46.4, n = 8 37.2 / 36.4 and 51.6 / 53.0)
        // In every case only with a workgroup for most compute units.
        if (p->mfma && !p->fused_db) {
            int64_t most = 0, active = 0, rows = 0;
            for (int32_t t = 0; t < n; ++t) {
                const int64_t nb = p->task_tb_off[t + 1] - p->task_tb_off[t];
                most = std::max(most, nb);
                active += nb > 0;
                rows += nb * ((p->rank_off[t + 1] - p->rank_off[t] + 15) / 16 * 16);
            }
            if (most > 0) rows /= most;          // (a task with fewer blocks has fewer partial sums)
            const int64_t tiles = (d->d_in + 127) / 128 + (d->d_out + 127) / 128;
            int64_t limit = 24;
            if (p->n_proj > 1 && p->dg % 128 != 0) limit = 6;
            else if (p->r_pad > 16 && rows * tiles < (p->n_proj > 1 ? 40960 : 12800)) limit = p->n_proj > 1 ? 10 : 12;
            if (most <= limit && active * tiles >= 192) cb = std::max(cb, most);
        }
        // The higher the ranks the more the partial sums weigh, which stage 1 writes and stage 2 reads - r / 4 of the bytes of a chunk of one
        // block -: on long batches chunks of at least 5 blocks per 16 ranks (of the mean over the blocks), if that leaves the largest task
        // more than one (both stages, us, chunks as above / with this floor: rank 128, 42123 x 768 x 7168 541 / 315, 45263 x 2688 x
        // 832 226 / 172, 8000 x 3072 x 5000 130 / 75; twice the floor is no better).  A wave walks a chunk's blocks one after the other, some
        // 0.8 us each, so the floor ends where it would leave fewer than 320 workgroups, 224 where ranks above 64 make a chunk's sums the
        // dearer part, or 352 on average over the launches of fused projections, which follow each other (the kernel of ranks up to 16 has
        // tiles of 128 columns: 6390 x 1024 x 768 keeps chunks of 5 blocks).  Projection of dy and gradients,
        // us, chunks as above / the floor alone / ended like this (one task; P = 3: dB in three launches):
        //   1600 x 1024 x 1024, rank 128   25.8 / 40.3 / 25.8        10000 x 1024 x 1024, rank 128     80.5 / 74.8 / 55
        //   2500 x 768 x 768, rank 32      18.3 / 19.7 / 18.3        1696 x 832 x 1536, P = 3, rank 96     27.1 / 57.3 / 27.0
        // 557 batches of 600 to 49000 tokens, 768 to 11008 columns, ranks 8 to 128, P = 1 .. 3: no floor 1, the floor alone 1.015,
        // ended as here 0.927, with two batches more than 3 % behind no floor.
        if (p->mfma && !p->fused_db && !p->tb.empty()) {
            int64_t most = 0, wsum = 0;
            for (int32_t t = 0; t < n; ++t) {
                const int64_t nb = p->task_tb_off[t + 1] - p->task_tb_off[t];
                most = std::max(most, nb);
                wsum += nb * (p->rank_off[t + 1] - p->rank_off[t]);
            }
            const int64_t nb = int64_t(p->tb.size()), least = wsum * 5 / (16 * nb);
            const int64_t db_launches = p->n_proj > 1 && p->dg % 128 != 0 ? p->n_proj : 1, launches = p->n_proj > 1 ? 1 + db_launches : 1;
            const int64_t tw = p->r_pad <= 16 ? 128 : 256;
            const int64_t tiles = (d->d_in + tw - 1) / tw + (d->d_out / db_launches + tw - 1) / tw * db_launches;
            const int64_t wanted = p->n_proj > 1 ? 352 * launches : p->r_max > 64 ? 224 : 320;
            if (5 * most > 6 * least) cb = std::max(cb, std::min(least, nb * tiles / wanted));
        }
        p->chunk_blocks = int32_t(cb);
        p->chunks.clear();
        p->task_chunk_off.assign(size_t(n) + 1, 0);
        p->part_rows = 0;
        for (int32_t t = 0; t < n; ++t) {
            const int32_t r = p->rank_off[t + 1] - p->rank_off[t];
            const int32_t nb = p->task_tb_off[t + 1] - p->task_tb_off[t];
            // (a task's blocks are split evenly among its chunks: no short chunk at the end of a task; workload 3:
            //  stage 1 177 -> 169 us)
            const int32_t nck = (nb + p->chunk_blocks - 1) / p->chunk_blocks;
            const int32_t len = nck > 0 ? (nb + nck - 1) / nck : p->chunk_blocks;
            for (int32_t b = p->task_tb_off[t]; b < p->task_tb_off[t + 1]; b += len) {
                const int32_t e = std::min(b + len, p->task_tb_off[t + 1]);
                p->chunks.push_back(GradChunk{b, e, t, p->part_rows});
                p->part_rows += r;
            }
            p->task_chunk_off[t + 1] = int32_t(p->chunks.size());
        }

        p->single_chunks = n > 0;
        p->empty_tasks = false;
        for (int32_t t = 0; t < n; ++t) {
            const int32_t c = p->task_chunk_off[t + 1] - p->task_chunk_off[t];
            p->single_chunks &= c <= 1;
            p->empty_tasks |= c == 0;
        }
        if (p->empty_tasks && n > kMaxClearedTasks) p->single_chunks = false;

        // (the reduction kernels put chunks x column tiles of at least 64 columns on grid.x, and behind them the tasks whose rows stage 1
        // clears, if there is room)
        const int64_t red_tiles = (int64_t(d->d_in) + 63) / 64 + (int64_t(d->d_out) + 63) / 64;
        if (int64_t(p->chunks.size()) * red_tiles > 0x7fffffff) return LOBRA_ERR_SHAPE;
        if (p->empty_tasks && (int64_t(p->chunks.size()) + n) * red_tiles > 0x7fffffff) p->single_chunks = false;

        // 5. buffer sizes
        BufferLayout& L = p->p_layout;
        const size_t ntb = p->tb.size();
        if (ntb == 0) {
            L = BufferLayout{};
        } else if (p->mfma) {
            L.p_tok = 0;
            L.p_blk = align_up(size_t(T) * p->r_pad * 2, 256);
            L.total = L.p_blk + align_up(ntb * size_t(p->r_pad) * kTokenBlock * 2, 256);
        } else {
            L.p_tok = 0;
            L.p_blk = 0;
            L.total = align_up(size_t(T) * p->r_max * 4, 256);
        }
        const size_t spart = align_up(size_t(p->sliced_out.nsl) * size_t(T) * 64, 256);
        p->h_save_bytes = L.total;
        if (p->mfma && T > 0) {
            // fused projections: one launch over all of them if its tiles fit their widths - at a width like 53 x 64 only
            // narrow tiles do, and a long batch is better off with a launch per projection (45861 x 904 x 2 x 3392: 1171
            // against 732 us)
            p->fwd_group = 0;
            const int32_t ns = ntb > 0 ? nseg : 0, rk = p->r_max / p->n_proj;
            if (p->n_proj > 1 && p->dg % 64 == 0 &&
                choose_gemm(T, d->d_in, d->d_out, p->dg, ns, rk, 0).cost <=
                    float(p->n_proj) * (choose_gemm(T, d->d_in, p->dg, 0, ns, rk, 0).cost + 3.f))
                p->fwd_group = p->dg;
            p->beside_fwd = p->beside_bwd = GemmChoice{};
            if (p->n_proj == 1) {
                int32_t halves = 1;
                for (const TokenBlock& b : p->tb) halves = std::max(halves, (b.nrows + 15) / 16);
                p->beside_fwd = choose_beside(T, d->d_in, d->d_out, ns, p->r_max, int64_t(ntb), halves);
                if (p->sliced_out.nsl == 0) p->beside_bwd = choose_beside(T, d->d_out, d->d_in, ns, p->r_max, int64_t(ntb), halves);
            }
            p->fwd_part = align_up(gemm_part_bytes(T, d->d_in, p->n_proj > 1 && !p->fwd_group ? p->dg : d->d_out, p->fwd_group, ns, rk, p->beside_fwd), 256);
            p->bwd_part = align_up(gemm_part_bytes(T, d->d_out, d->d_in, 0, ns, p->r_max, p->beside_bwd), 256);
        }
        p->fwd_ws_bytes = p->fwd_part + L.total;
        p->bwd_off_g = 0;
        p->bwd_off_h = L.total;
        p->bwd_off_part_b = 2 * L.total;
        // (with dB fused into the projection of dy, its partial sums are the fused kernel's)
        p->bwd_off_part_a = p->bwd_off_part_b +
                            align_up(size_t(p->fused_db ? p->fb_rows : p->part_rows) * size_t(d->d_out) * 4, 256);
        p->bwd_off_spart = p->bwd_off_part_a + align_up(size_t(p->part_rows) * size_t(d->d_in) * 4, 256);
        p->bwd_need = p->bwd_off_spart + spart;
        p->bwd_ws_bytes = std::max(p->bwd_need, p->bwd_off_spart + p->bwd_part);
    } catch (const std::bad_alloc&) {
        return LOBRA_ERR_NOMEM;
    }
    return LOBRA_OK;
}

constexpr int64_t cus = 256;                 // fixed, so that the choice does not depend on the device

// The time of so many workgroups of a tile with so many K tiles each.
static float rounds_cost(const GemmTile& t, int64_t wgs, int32_t kt, float fixed)
{
    const int64_t slots = cus * t.per_cu, full = wgs / slots, rest = wgs % slots;
    const float per = float(kt), most = t.per_cu == 2 ? t.k2 : t.k1;
    return float(full) * (most * per + fixed) + (rest ? (rest <= cus ? t.k1 : most) * per + fixed : 0.f);
}

GemmChoice choose_gemm(int64_t T, int32_t K, int32_t N, int32_t group, int32_t nseg, int32_t rank, size_t part_bytes)
{
    const int32_t kt = (K + kGemmKTile - 1) / kGemmKTile;
    const bool ktail = K % (2 * kGemmKTile) != 0;
    const float segments = std::max(0.f, float(nseg) * kGemmTileRows / float(T) - 1.f);      // per tile row, beyond the first
    GemmChoice best;
    float least = -1.f;
    for (int32_t i = 0; i < int32_t(sizeof(kGemmTiles) / sizeof(kGemmTiles[0])); ++i) {
        const GemmTile& t = kGemmTiles[i];
        // the persistent kernel: at least one whole output tile, and enough K for its special last pairs of K tiles; where
        // it runs without those the staged kernel is never better
        const bool whole = T >= t.tm && N >= t.tn;
        if (i == kPersistentTile && !(whole && (!ktail || K >= kPersistentMinKTail))) continue;
        if (i == kStagedTile && whole && !ktail) continue;
        if (group > 0 && group % t.tn != 0) continue;
        // a Z beyond the 256 MB infinity cache is read once where one column tile takes all of N (47000 x 3200 x 248: 128 x 256
        // 99 us, 128 x 128 118, 128 x 64 145)
        if (group == 0 && N <= 256 && t.tn < N && int64_t(T) * K * 2 > (int64_t(256) << 20)) continue;
        float fixed = t.fixed;
        if (i == kPersistentTile && ktail)
            fixed = kKTailFixed + (N % 32 ? kKTailOddRows : 0.f) + kKTailRank * std::max(0.f, float(rank - 32) / 32.f);
        if (i == kPersistentTile) fixed += kSegmentCost.persistent * segments;
        if (i == kStagedTile) fixed += kSegmentCost.staged * segments;
        const int64_t tiles = (T + t.tm - 1) / t.tm * ((N + t.tn - 1) / t.tn), slots = cus * t.per_cu;
        for (int32_t s = 1; s <= kMaxSplits; ++s) {
            const int64_t bytes = int64_t(s + 1) * T * N * 4;      // (one more for the adapter term)
            if (s > 1 && (i == kPersistentTile || i == kStagedTile || K < kMinSplitK || kt < 4 * s || tiles * s > slots ||
                          uint64_t(bytes) > part_bytes))
                break;
            float cost = rounds_cost(t, tiles * s, (kt + s - 1) / s, fixed) + t.once;
            if (s > 1) cost += 3.f + float(bytes) / 3e6f;
            if (least < 0.f || cost < least) best = GemmChoice{i, s, cost}, least = cost;
        }
    }
    return best;
}

GemmChoice choose_beside(int64_t T, int32_t K, int32_t N, int32_t nseg, int32_t rank, int64_t ntb, int32_t halves)
{
    GemmChoice best;
    const int64_t items = ntb * ((rank + 15) / 16);
    if (ntb == 0 || K < kMinSplitK || items > kMaxBesideItems || T * N * rank > kMaxBesideRankRows) return best;
    const int32_t kt = (K + kGemmKTile - 1) / kGemmKTile;
    float least = choose_gemm(T, K, N, 0, nseg, rank, kMaxPartBytes).cost + beside_gain(K);
    const float spread = 1.f + 0.3f * std::max(0.f, float(T) * float(K) / 5e6f - 1.f);
    for (int32_t i = 3; i <= 4; ++i) {               // (two workgroups of these, or of the projection, share a compute unit)
        GemmTile t = kGemmTiles[i];
        t.k2 *= spread;
        const int64_t tiles = (T + t.tm - 1) / t.tm * ((N + t.tn - 1) / t.tn);
        for (int32_t s = 1; s <= kMaxSplits; ++s) {
            const int64_t bytes = int64_t(s) * T * N * 4;
            if (tiles * s + items * halves > cus * t.per_cu || uint64_t(bytes) > kMaxPartBytes || (s > 1 && kt < 4 * s)) break;
            const float cost = rounds_cost(t, tiles * s + items, (kt + s - 1) / s, t.fixed) + t.once + 3.f + float(bytes) / 3e6f;
            if (cost < least) best = GemmChoice{i, s, cost}, least = cost;
        }
    }
    return best;
}

size_t gemm_part_bytes(int64_t T, int32_t K, int32_t N, int32_t group, int32_t nseg, int32_t rank, const GemmChoice& beside)
{
    const GemmChoice c = choose_gemm(T, K, N, group, nseg, rank, kMaxPartBytes);
    return std::max(c.splits > 1 ? size_t(c.splits + 1) * size_t(T) * size_t(N) * 4 : 0,
                    beside.tile >= 0 ? size_t(beside.splits) * size_t(T) * size_t(N) * 4 : 0);
}

SlicedShape sliced_shrink_shape(int64_t ntb, int32_t r_pad, int32_t D)
{
    SlicedShape none;
    // whole slices only (the kernel's copies carry no bound); at least a dozen items per compute unit
    if (r_pad != 16 || ntb <= 0 || D <= 0 || D % 512 != 0) return none;
    const int64_t nsl = D / 512;
    const int64_t items = ntb * nsl;
    if (items < 3072 || items >= 0x7fffffff) return none;
    return SlicedShape{int32_t(nsl)};
}

std::vector<int32_t> product_tables(const Plan& p)
{
    if (p.desc.dtype == LOBRA_F32) {
        const int32_t nseg = int32_t(p.cseg_task.size());
        const size_t blocks = p.rowblk_seg.size();
        constexpr size_t kRec = sizeof(F32BlockRec) / sizeof(int32_t), kItem = sizeof(F32Item) / sizeof(int32_t);
        std::vector<int32_t> list;
        list.reserve(blocks * (kRec + size_t(p.f32_items) * kItem));
        list.resize(blocks * kRec);
        for (size_t b = 0; b < blocks; ++b) {
            const int32_t row0 = int32_t(b) * kRowBlock, own = p.rowblk_seg[b], first = p.cseg_task[size_t(own)] >= 0 ? own : own + 1;
            auto rows = [&](int32_t k) { return uint8_t(std::max(0, std::min(p.cseg_off[size_t(k)] - row0, 255))); };    // to where segment k starts
            F32BlockRec r{255, 255, 255, 0, 0, own};
            if (own + kFewSegments < nseg) r.fifth = rows(own + kFewSegments);
            if (first < nseg) {
                const int32_t t = p.cseg_task[size_t(first)];
                r.lo = rows(first);
                r.hi = rows(first + 1);
                r.rank = uint8_t(p.rank_off[t + 1] - p.rank_off[t]);
                r.rank0 = p.rank_off[t];
            }
            std::memcpy(&list[b * kRec], &r, sizeof(r));
        }
        for (size_t b = 0; p.f32_items > 0 && b < blocks; ++b) {
            int32_t left = p.f32_items;
            for (int32_t k = p.rowblk_seg[b]; k < nseg && p.cseg_off[size_t(k)] < int32_t(b + 1) * kRowBlock; ++k) {
                const int32_t t = p.cseg_task[size_t(k)];
                const int32_t r = t >= 0 ? p.rank_off[t + 1] - p.rank_off[t] : 0;
                for (int32_t c = 0; c < r; c += 16, --left)
                    list.insert(list.end(), {p.cseg_off[size_t(k)], p.cseg_off[size_t(k) + 1], p.rank_off[t] + c, std::min(r - c, 16), t, c, r, 0});
            }
            list.resize(list.size() + size_t(left) * kItem, 0);
        }
        return list;
    }

    // behind the records, for every segment: its task's first rank row, then, for every segment again, its stacked rank (see cseg_rank)
    // (nothing of it without adapters)
    const size_t nseg = p.tb.empty() ? 0 : p.cseg_task.size(), at = p.tb.empty() ? 0 : p.gemm_tile_seg.size();
    std::vector<int32_t> list(p.gemm_tile_seg.begin(), p.gemm_tile_seg.begin() + at);
    list.resize(at + 2 * nseg, 0);
    for (size_t k = 0; k < nseg; ++k) {
        const int32_t t = p.cseg_task[k];
        if (t < 0) continue;
        list[at + k] = p.rank_off[t];
        list[at + nseg + k] = p.rank_off[t + 1] - p.rank_off[t];
    }
    // and, where the sum of a split product adds the adapter term, the same for every row (see row_rank)
    if ((p.beside_fwd.tile >= 0 || p.beside_bwd.tile >= 0) && p.desc.T <= kRowTableTokens)
        for (size_t k = 0; k < nseg; ++k)
            for (int32_t i = p.cseg_off[k]; i < p.cseg_off[k + 1]; ++i) list.insert(list.end(), {list[at + k], list[at + nseg + k]});
    return list;
}

std::vector<int32_t> pack_blob(Plan* p)
{
    std::vector<int32_t> blob;
    auto put = [&](const int32_t* src, size_t n) {
        while (blob.size() % 4) blob.push_back(0);   // 16-byte alignment of every list
        const size_t off = blob.size();
        blob.insert(blob.end(), src, src + n);
        if (n == 0) blob.push_back(0);               // keep every list pointer valid
        return off;
    };
    p->o_cseg_off = put(p->cseg_off.data(), p->cseg_off.size());
    p->o_cseg_task = put(p->cseg_task.data(), p->cseg_task.size());
    p->o_rowblk = put(p->rowblk_seg.data(), p->rowblk_seg.size());
    p->o_tb = put(reinterpret_cast<const int32_t*>(p->tb.data()), p->tb.size() * 4);
    p->o_chunks = put(reinterpret_cast<const int32_t*>(p->chunks.data()), p->chunks.size() * 4);
    p->o_task_chunk = put(p->task_chunk_off.data(), p->task_chunk_off.size());
    p->o_rank_off = put(p->rank_off.data(), p->rank_off.size());
    p->o_task_tb = put(p->task_tb_off.data(), p->task_tb_off.size());
    const size_t runs = p->shrink_group > 1;         // (runs of one block are the blocks)
    p->o_sb = put(p->sb_off.data(), runs * p->sb_off.size());
    p->o_tb_order = put(p->tb_order.data(), p->tb_order.size());
    p->o_sb_order = put(p->sb_order.data(), runs * p->sb_order.size());
    p->o_fb_wg = put(p->fb_wg_run_off.data(), p->fb_wg_run_off.size());
    p->o_fb_run = put(p->fb_run_row.data(), p->fb_run_row.size());
    p->o_fb_cnt = put(p->fb_cnt.data(), p->fb_cnt.size());
    p->o_fb_row0 = put(p->fb_task_row0.data(), p->fb_task_row0.size());
    const std::vector<int32_t> list = product_tables(*p);
    p->o_tile_seg = put(list.data(), list.size());
    while (blob.size() % 4) blob.push_back(0);
    return blob;
}

}  // namespace lobra

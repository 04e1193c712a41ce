// Host side of a batch plan: validation of the descriptor and the work lists that the
// kernels walk.  Pure C++ (no HIP), so that it can be built and tested without a GPU.
#pragma once
#include <cstddef>
#include <cstdint>
#include <vector>

#include "lobra_mlora.h"

namespace lobra {

constexpr int kTokenBlock = 32;   // tokens per token block (one MFMA K step of the reductions)
constexpr int kRowBlock = 32;     // granularity of the row -> segment lookup table
constexpr int kGemmTileRows = 256;    // token rows of a base-GEMM output tile
constexpr int32_t kRowTableTokens = 256;  // batches that get a table of rows: 2 KiB of tables at most
constexpr int kGemmTileSegs = 3, kGemmTileSegRec = 16;     // adapter segments and ints per record of Plan::gemm_tile_seg
constexpr int kMaxClearedTasks = 4096;    // up to here stage 1 of the gradients clears the rows of tasks without tokens
constexpr bool kMfmaKernels = true;   // bf16 storage runs on the MFMA kernels
// Most tokens of an fp32 batch and of LOBRA_PLAN_PLAIN_KERNELS: the plain kernels put 64-token tiles on grid.y, and the
// projections start up to 512 threads per token, which a launch of less than 2^32 threads has room for.
constexpr int64_t kPlainMaxTokens = 65535 * 64;

// fp32: what a 32-row block says about the tiles that start with it.  In rows from its first on, at most 255: where the segment
// kFewSegments further on starts, and first row and last + 1 of the first segment from there on that has an adapter (255, 255: none) - the
// block's own, or the next one, since no two without an adapter are neighbours.  That segment's task: its stacked rank and first rank
// row.  And the segment of the block's first row (Plan::rowblk_seg once more: a second line of the tables would be a second round trip).
constexpr int kFewSegments = 4;
struct F32BlockRec { uint8_t fifth, lo, hi, rank; int32_t rank0, own; };
static_assert(LOBRA_MAX_RANK < 256 && sizeof(F32BlockRec) == 12, "a record is three numbers of 32 bits");

// fp32, short batches: a block of up to 16 ranks that a 32-row block's product meets - the rows of its segment, its first rank row, how many
// there are (0: no such block), the task, the block's first rank within the task and the task's rank
struct F32Item { int32_t lo, hi, row, n, task, c0, r, pad; };
// The projection runs inside its product (gemm_f32_fused) in tiles of 32 x 32, each of which projects its own rows: of a batch whose 32-row
// blocks meet at most four blocks of ranks (`items` 2 or 4), while that costs less than a launch: training steps, us, apart / inside, with
// tiles x K x items in Ki: 200 x 1024 x 512 38.7 / 28.5 (224), 32 x 2048 x 2048 59.3 / 53.4 (256), 618 x 512 x 512 35.7 / 31.5 (320),
// 1000 x 256 x 1024 at rank 32 48.4 / 49.0 (1024).  The table of items is 4 KiB at most, which one-shot calls send.
constexpr int64_t kFusedTokens = 1024, kFusedTiles = 1024;
inline bool f32_fused(int64_t T, int32_t K, int32_t N, int32_t items)
{
    const int64_t n = (T + 31) / 32 * ((int64_t(N) + 31) / 32);
    return items > 0 && T <= kFusedTokens && n <= kFusedTiles && n * K * items <= 640 * 1024;
}

// A one-shot call's tables go to the device as arguments of launches, kUploadPiece numbers each, up to this many bytes; larger ones by a copy.
// A piece takes 2.3 us of stream time and some 3.5 of the host's; a copy from pageable memory and the host callback that releases it take
// 55 to 62 us of either (73 to 166 KB of tables), and some 180 us a call where the host is not ahead of the stream (padded chunks of 3072
// tokens, four calls, 730 -> 173 us).  Calls that the host bounds take as long either way at 21 pieces (2070 one-token segments, 512 x 512,
// 175 and 173 us); 24 keep what lists of the products add to tables of 64 KiB from turning such a call into a copy.
constexpr size_t kUploadPiece = 1008;         // with the other arguments just below the 4 KiB of a launch
constexpr size_t kUploadByArgument = 24 * kUploadPiece * sizeof(int32_t);

struct TokenBlock { int32_t row0, nrows, task, rank_row0; };
struct GradChunk  { int32_t tb_begin, tb_end, task, part_row0; };

// The pass over dy that projects it and accumulates dB, for long batches of ranks up to 16, cuts K into slices of 512 columns and lets one
// workgroup per compute unit walk (token block, slice) items (shrink_sliced_kernel).  nsl = slices; nsl = 0: dB is left to the
// reduction kernels.
struct SlicedShape { int32_t nsl = 0; };
constexpr int kSlicedGrid = 256;      // its workgroups: 8 XCDs x 32 compute units
// The shape for ntb token blocks projected from width D, or none: widths that are not a multiple of the slice,
// other ranks, too few items to keep every compute unit busy.
SlicedShape sliced_shrink_shape(int64_t ntb, int32_t r_pad, int32_t D);

// The kernels a bf16 product can run on and what a K tile of 64 costs there, measured (us, K = 4096; the tiled kernels with
// one workgroup per compute unit and, where two fit, with two; `fixed`: start, adapter term and stores of a tile; `once`: what
// the persistent kernel, whose tiles follow each other in one stream, pays only at the start):
//     tile        persistent 256 x 256   128 x 256   128 x 128   128 x 64      64 x 64
//     T = 40      112 us                 44          31          24            18
//     T = 200     113                    46          33          25            21
//     T = 500      80                    48          35          28 (256 wgs)  32 (512 wgs)
//     T = 1000     81                    49          39 (256)    45 (512)      57
//     T = 2000     84                    62 (256)    75          81            110
//     T = 4096    102 (256)              122        156          193           261
// (x [T, 4096] times W [4096, 4096]; a register-staged kernel took 112 us below 256 tokens.)
// A tile's bytes through the copy path and its LDS reads grow slower than its MFMAs, so the largest tile that still
// gives every compute unit one is the best; what remains is the count of rounds, which the choice estimates.
// K that is no multiple of 128: the persistent kernel's form for it works its epilogue's addresses out anew per tile (kKTailFixed
// for its `fixed`) and pays more again for rows of C that start inside a 64-byte sector (kKTailOddRows where N is no multiple
// of 32: 20000 x 840 x 5240 268 us, the staged kernel 251; x 4096 154, 174) and for ranks above 32, a step of the up projection each
// (kKTailRank; 47000 x 600 x 7232 at rank 32, 64 and 128, this kernel / the staged one: 579, 560 and 625 / 621, 613 and 646 us).
// The persistent and the staged kernel do the up projection segment by segment - the persistent one with the operands of two segments of
// up to 16 ranks at a time -, the tiled kernels by task (kSegmentCost).  Measured, us per round of 256 tiles (N = 7552, 55000 tokens),
// and us in all for 12000 x 584 x 1000 and 12000 x 1024 x 1024 in segments of n tokens, rank 16:
//     K                 64    200   328   520   712   968   1376  2248      n = 400   20    4     n = 400   20    4
//     persistent                          23.6  26.9  33.7  41.6  65.5      35        42    85        30    43    88
//     staged            9.3   15.0  18.6  25.1  31.0  38.6  48.6  75.8      30        46    103       42    58    113
//     128 x 256 (x 2)   14.8  21    24    29    35    42    50    73        38        41    47        43    46    51
struct GemmTile { int32_t tm, tn, per_cu; float k1, k2, fixed, once; };
constexpr GemmTile kGemmTiles[] = {
    {256, 256, 1, 1.35f, 0.f, 5.f, 7.f},     // gemm_persistent_kernel
    {128, 256, 1, 0.86f, 0.f, 6.5f, 0.f},
    {128, 128, 1, 0.48f, 0.f, 7.f, 0.f},
    {128, 64, 2, 0.36f, 0.59f, 7.f, 0.f},
    {64, 64, 2, 0.23f, 0.39f, 6.f, 0.f},
    {256, 256, 1, 2.0f, 0.f, 5.5f, 0.f},     // gemm_staged_kernel
};
constexpr int32_t kPersistentTile = 0, kStagedTile = 5;
constexpr float kKTailFixed = 10.f, kKTailOddRows = 4.f, kKTailRank = 0.75f;  // (kKTailRank: per 32 ranks beyond the first 32)
// us per round and segment of a tile row beyond the first.  (Persistent kernel, training steps at rank 16, us, with 0.8 / 1.4: 16384 x 2048 x
// 2048 in segments of 12 tokens 354 / 326, of 16 349 / 323, 9000 x 4096 x 4096 of 20 643 / 602, 12000 x 1376 x 4096 of 22 365 / 362, 30000 x
// 1024 x 4096 of 18 630 / 612, 49152 x 768 x 768 of 36 252 / 241, 6000 x 2048 x 2048 of 20 152 / 159; 19 batches on which the two
// differ, 0.98 on average.)
struct SegmentCost { float persistent, staged; };
constexpr SegmentCost kSegmentCost = {1.4f, 1.0f};
constexpr int32_t kGemmKTile = 64;
// The persistent kernel's loop for such a K needs an ordinary pair of K tiles in front of the two special ones (K > 256).  It runs
// from here on, where it is the better one for wide products (30000 x 520 x 1000 / 2048 / 7552, staged / persistent: 62 / 76,
// 102 / 98, 336 / 329 us; the estimate tells them apart); below, it would lose at 264 (136 / 145 at 4096 columns), gain
// nothing at 392 (165 / 167) and gain 5 .. 10 % at 456 and 504 (181 / 166).
constexpr int32_t kPersistentMinKTail = 520;
// Where a product has fewer tiles than compute units and a long K (decoding, narrow shards), K is split among up to eight
// workgroups per tile, each of which writes its fp32 sums to scratch; a small kernel adds them in order (3 us, and the
// sums' way to memory and back, mostly through the caches, at 6 TB/s: with a tile's time as above that puts 519 x 5504 x 1928
// on two splits of 128 x 128, 29 us instead of 36, 1720 x 8192 x 768 likewise, 39 instead of 46, and leaves 200 x 4096 x 4096
// unsplit, 21 instead of 24): x [40, 4096] W [4096, 4096] with 8 adapters 24 -> 13.6 + 4.0 us, x [7, 5248]
// W [5248, 1024] 22.8 -> 8.4 + 2.5 us.  At most kMaxPartBytes of them, so that they fit the library's static scratch
// array next to the projected activations.
constexpr int32_t kMaxSplits = 8, kMinSplitK = 1024;
constexpr size_t kMaxPartBytes = size_t(12) << 20;
struct GemmChoice { int32_t tile = -1, splits = 1; float cost = -1.f; };    // tile: of kGemmTiles, -1: none; cost: the estimate, us
// The choice for C [T, N] = Z [T, K] op(W) given part_bytes of scratch.  group > 0: no tile may straddle a multiple of
// `group` columns (a multiple of 64).  nseg: segments of the batch (0: no adapter); rank: the widest rank window.
GemmChoice choose_gemm(int64_t T, int32_t K, int32_t N, int32_t group, int32_t nseg, int32_t rank, size_t part_bytes);
// The same where the projection runs in the product's launch and the adapter term comes with the sum of the splits, of which there may
// be one (gemm_mfma_beside; ntb: token blocks; halves: 2 if one has more than 16 tokens, else 1): tile -1 where a projection of its own is better.  Given kMaxPartBytes of scratch.
// Forward passes, a projection of its own / beside the product, us (K x N, rank, n one-token requests or tokens of segments of m):
//     4096 x 4096    16   n = 1 20.7 / 13.0   40 22.3 / 15.0   100 28.1 / 17.9   150 29.9 / 22.4   128 of 40  25.7 / 17.8
//                    128  n = 1 22.3 / 18.4   40 31.4 / 23.1
//     8192 x 1024    64   n = 8 22.8 / 18.9   200 of 60  28.4 / 23.0   500 of 200  42.2 / 36.2
//     4096 x 11008   16   n = 1 29.0 / 22.6   40 35.3 / 28.7   100 45.2 / 38.6   (one split)
//     2048 x 2048    16   n = 40 18.2 / 11.6  300 of 100  18.6 / 15.8
// The estimate counts a projection's items (token blocks x rank blocks) with the product's workgroups, as if they took as long: without
// that, a product that filled the compute units by itself was split as far (100 of 4096 x 4096: 20.4; 1284 x 8160 x 768, both
// passes: 108 where it is 97 now and 102 apart).  An item is a workgroup per half of its block, and all have to run at once: on one
// that has to wait for another to end the launch waits too (apart / one too many, us: 600 x 1504 x 1536, rank 16 15.8 / 18.5; 800 x 1024 x
// 1024, rank 32 13.7 / 17.0; 1100 x 2048 x 768, rank 32 18.3 / 21.7).  Halves without tokens end at once, but leave room on their own XCD
// only, so they count unless all blocks are short.  Where two workgroups share a compute unit the splits of a Z of more than 5 million
// elements find less of it in the L2 than the table's k2 says (per K tile of 128 x 64: 0.59 us at 1500 x 4096, 0.76 at 1800 x 5504, 0.93
// at 1500 x 11008, where a product beside took 93 us and one apart 72).  What is saved, a launch and the chain of tables and adapter copies behind
// a tile, is beside_gain, and more with a longer K, which a projection of its own takes longer for (apart / beside where the estimates differ
// by about that: 1100 x 1024 x 1024, 4.5 us, 14.9 / 15.7; 600 x 2048 x 2048, 4.2, 20.8 / 19.5; 1500 x 2048 x 768, 4.0, 22.1 / 20.5; both passes
// of 158 x 3456 x 8576, 4.8, 67.9 / 64.3).  The sum reads T N rank elements of the adapters: from 32 million on that takes the gain
// (200 x 1024 x 3072 at rank 64, 39 million: 15.0 / 17.0; 700 x 8192 x 1024 39.2 / 44.8; 128 x 4096 x 4096 at rank 128 25.5 / 26.6).
// Below K = kMinSplitK a token's result shall not depend on the size of its batch.
inline float beside_gain(int32_t K) { return K < 3414 ? 3.5f + 0.45f * float(K) / 1024.f : 5.f; }
constexpr int64_t kMaxBesideItems = 256, kMaxBesideRankRows = int64_t(32) << 20;
GemmChoice choose_beside(int64_t T, int32_t K, int32_t N, int32_t nseg, int32_t rank, int64_t ntb, int32_t halves);
// The scratch that these choices would like to have (0: none).
size_t gemm_part_bytes(int64_t T, int32_t K, int32_t N, int32_t group, int32_t nseg, int32_t rank, const GemmChoice& beside);

// Byte offsets of the sub-buffers inside h_save and the workspaces.
struct BufferLayout {
    size_t p_tok = 0;     // token-major projected activations  [T][pstride]
    size_t p_blk = 0;     // block-transposed copy              [n_tb][rpad][32]  (MFMA path)
    size_t total = 0;
};

struct Plan {
    lobra_mlora_desc desc{};            // table pointers point into the vectors below
    uint32_t flags = 0;
    bool mfma = false;                  // bf16 storage and MFMA kernels
    int32_t r_max = 0, r_pad = 0, R_tot = 0;
    int32_t n_proj = 1;                 // shared-input projections fused into the call
    int32_t dg = 0;                     // d_out / n_proj: width of B and dB
    std::vector<int32_t> rank_off;      // [n_tasks+1]
    std::vector<int32_t> seg_off_in, seg_task_in;   // the caller's table, as given
    std::vector<int32_t> cseg_off, cseg_task;       // compacted table
    std::vector<int32_t> rowblk_seg;    // [ceil(T/32)]
    // One record of kGemmTileSegRec ints per tile row of the base GEMM (tile row i starts at token min(i kGemmTileRows, T - kGemmTileRows),
    // never below 0), which one 64-byte read brings to a GEMM workgroup: the first kGemmTileSegs
    // segments with an adapter that cross it - first token, last + 1, the task's first rank row and stacked rank (0 where there
    // is no such segment) - and the compacted segment at which to look for further ones.
    std::vector<int32_t> gemm_tile_seg; // [ceil(T/kGemmTileRows)][kGemmTileSegRec]
    std::vector<TokenBlock> tb;         // grouped by task, token order inside a task
    std::vector<int32_t> task_tb_off;   // [n_tasks+1]
    std::vector<int32_t> sb_off;        // [nsb+1] runs of <= shrink_group token blocks of one task
    int32_t shrink_group = 1;           // token blocks that one shrink workgroup handles (1 or 4)
    // launch order of the shrink workgroups when ranks differ: token blocks / runs by descending rank
    // (stable), so that the most expensive ones do not form the tail of the launch.  Empty: as stored.
    std::vector<int32_t> tb_order, sb_order;
    std::vector<GradChunk> chunks;      // grouped by task
    std::vector<int32_t> task_chunk_off;// [n_tasks+1]
    // no task has more than one chunk: no partial sums to add (tasks without tokens, which stage 1 then clears: only while
    // there are few tasks, since it starts a workgroup for each of them and column tile)
    bool single_chunks = false, empty_tasks = false;
    int32_t f32_items = 0;      // fp32: blocks of ranks per 32-row block in the table of items (2 or 4), 0: no table
    bool fused_fwd = false, fused_bwd = false;      // fp32: the projection inside its product
    bool grad_one = false;      // fp32: both gradients without partial sums (grad_f32_one)
    int32_t part_rows = 0;              // rows of the partial-sum buffer = sum over chunks of r_t
    int32_t chunk_blocks = 0;           // token blocks per reduction chunk

    BufferLayout p_layout;              // layout of h_save (and of the G buffer in bwd)
    size_t h_save_bytes = 0, fwd_ws_bytes = 0, bwd_ws_bytes = 0;
    size_t bwd_off_g = 0, bwd_off_h = 0, bwd_off_part_b = 0, bwd_off_part_a = 0;
    // K-sliced projection of dy (fused_db): its shape, and where its fp32 partial projections [nsl][T][16] go: at bwd_off_spart in the workspace
    SlicedShape sliced_out;
    // A split base product's partial sums (fwd_part / bwd_part bytes, see choose_gemm) go to the start of the forward workspace, in front
    // of the projected activations (which the caller may have elsewhere: h_save), and in the backward one to bwd_off_spart, where the
    // projection is done by that time.  They are welcome and not needed: fwd_ws_bytes and bwd_ws_bytes have room for them, but
    // a call is refused only below what it cannot do without - without h_save the projected activations in a forward call (then at
    // the start), bwd_need in a backward one.
    // (fwd_group: fused projections' forward products run as one launch whose tiles do not straddle multiples of this
    // many columns; 0: one launch per projection)
    int32_t fwd_group = 0;
    GemmChoice beside_fwd, beside_bwd;  // the projection in the launch of its product, given scratch for it (tile -1: not)
    size_t bwd_off_spart = 0, fwd_part = 0, bwd_part = 0, bwd_need = 0;
    // dB fused into the sliced projection of dy (one pass over dy for s_t B_t dy_i and for dB): a workgroup
    // keeps the dB sums of the (task, slice) it is working on and writes them out - 16 rank rows x 512
    // columns - whenever task or slice changes.  These tables say where: the runs of workgroup g are
    // fb_wg_run_off[g] .. fb_wg_run_off[g + 1] - 1 in the order it meets them, run i goes to the rows
    // fb_run_row[i] .. + 15 of the partial array [fb_rows][d_out]; the k-th run of (task t, slice s) over all
    // workgroups sits at row fb_task_row0[t] + 16 k, and there are fb_cnt[t * nsl + s] of them (stage 2 adds
    // them in that order).
    bool fused_db = false;
    std::vector<int32_t> fb_wg_run_off, fb_run_row, fb_cnt, fb_task_row0;
    int32_t fb_rows = 0;

    // optional launch trace (see lobra_mlora_plan_set_trace)
    mutable void* const* trace_events = nullptr;
    mutable int32_t trace_pairs = 0;
    mutable int32_t* trace_ids = nullptr;
    mutable int32_t* trace_count = nullptr;
    mutable int32_t trace_next = 0;

    // device copy (absent for host-only plans)
    int device = -1;
    void* dev_blob = nullptr;
    bool owns_blob = false;             // dev_blob came from hipMalloc (plan_create), not from the caller (plan_init)
    std::vector<int32_t> host_blob;     // what dev_blob holds
    size_t blob_bytes = 0;
    void* static_ws = nullptr;          // this device's copy of the library's static scratch array
    // offsets (in int32 units) of the lists inside the blob
    size_t o_cseg_off = 0, o_cseg_task = 0, o_rowblk = 0, o_tb = 0, o_chunks = 0,
           o_task_chunk = 0, o_rank_off = 0, o_task_tb = 0, o_sb = 0, o_tb_order = 0, o_sb_order = 0,
           o_fb_wg = 0, o_fb_run = 0, o_fb_cnt = 0, o_fb_row0 = 0, o_tile_seg = 0;
};

lobra_status validate(const lobra_mlora_desc* d);
// Fills every host field of `p` (not the device copy).  `d` has been validated.
lobra_status build_host_plan(const lobra_mlora_desc* d, uint32_t flags, Plan* p);
// The list that the products read besides the segments: for the MFMA kernels Plan::gemm_tile_seg and, behind it, rank rows and ranks per segment
// and per row (cseg_rank, row_rank), for fp32 an F32BlockRec per 32-row block and, behind them, the F32Items.
std::vector<int32_t> product_tables(const Plan& p);
// Packs the lists into one int32 blob; sets the o_* offsets.
std::vector<int32_t> pack_blob(Plan* p);

}  // namespace lobra

struct lobra_mlora_plan : lobra::Plan {};

// host-only sanitizer run of the plan builder and the bucketing programme (random tables)
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>
#include "plan.h"
extern "C" lobra_status lobra_dynamic_buckets(const int32_t*, int64_t, const int32_t*, int32_t, int32_t, int32_t*, int32_t*, int64_t*);
int main() {
  std::mt19937 rng(7);
  for (int it = 0; it < 3000; ++it) {
    int S = rng() % 40, n = rng() % 6;
    std::vector<int32_t> off(1, 0), task, ro(1, 0);
    // every third table describes fused shared-input projections: ranks and width multiples of 8 P
    const int P = it % 3 == 2 ? 2 + int(rng() % 3) : 1;
    for (int t = 0; t < n; ++t) ro.push_back(ro.back() + (P > 1 ? 8 * P * (1 + int(rng() % (16 / P))) : 1 + int(rng() % 128)));
    static const int L[] = {0, 1, 2, 15, 16, 17, 31, 32, 33, 64, 100, 255, 256, 257, 1000};
    for (int k = 0; k < S; ++k) { off.push_back(off.back() + L[rng() % 15]); task.push_back(int(rng() % (n + 1)) - 1); }
    lobra_mlora_desc d{};
    d.dtype = rng() % 2; d.d_in = 8 * (1 + rng() % 600); d.d_out = 8 * (1 + rng() % 600); d.T = off.back(); d.n_tasks = n; d.S = S;
    d.rank_off = ro.data(); d.seg_off = off.data(); d.seg_task = task.data();
    if (P > 1) { d.n_proj = P; d.d_out = 8 * P * (1 + rng() % 100); }
    if (S == 0) d.T = 0;
    lobra_status st = lobra::validate(&d);
    if (st != LOBRA_OK) { printf("validate %d at it %d\n", st, it); return 1; }
    lobra::Plan p;
    st = lobra::build_host_plan(&d, rng() % 4, &p);
    if (st != LOBRA_OK) { printf("plan %d\n", st); return 1; }
    // the last list holds what the kernels look for behind each other: tile rows, segments, rows; fp32 blocks and items
    const size_t behind = lobra::pack_blob(&p).size() - p.o_tile_seg, T = size_t(d.T), nseg = p.cseg_task.size();
    const bool rows = T <= 256 && (p.beside_fwd.tile >= 0 || p.beside_bwd.tile >= 0);
    const size_t want = d.dtype == LOBRA_F32 ? (T + 31) / 32 * (3 + 8 * size_t(p.f32_items))
                        : p.tb.empty() ? 0 : (T + 255) / 256 * 16 + 2 * nseg + (rows ? 2 * T : 0);
    if (behind != (want > 0 ? (want + 3) / 4 * 4 : 4)) { printf("%zu numbers behind the lists, %zu wanted, it %d\n", behind, want, it); return 1; }
    // bucketing
    int U = 1 + rng() % 64, R = 1 + rng() % 20;
    std::vector<int32_t> u; int32_t b = 0; for (int i = 0; i < U; ++i) { b += 1 + rng() % 300; u.push_back(b); }
    std::vector<int32_t> lens; int ns = rng() % 200; for (int i = 0; i < ns; ++i) lens.push_back(1 + rng() % u.back());
    std::vector<int32_t> ob(R); int32_t on = 0; int64_t pad = 0;
    st = lobra_dynamic_buckets(lens.data(), ns, u.data(), U, R, ob.data(), &on, &pad);
    if (st != LOBRA_OK || on > R) { printf("bucket %d\n", st); return 1; }
  }
  // long tables: the lists of the products (from o_tile_seg on) must not make a one-shot call's tables too large for launch arguments
  // where all other lists, the runs and their order also where they are not sent, and eight numbers for each 256 rows are no more than 64 KiB
  for (int it = 0; it < 1500; ++it) {
    const int n = 1 + int(rng() % (it % 2 ? 16 : 2)), S = it % 5 == 4 ? 1 + int(rng() % 40) : 1500 + int(rng() % 2500), most = it % 3 == 0 ? 1 : 1 + int(rng() % 60);
    std::vector<int32_t> off(1, 0), task, ro(1, 0);
    for (int t = 0; t < n; ++t) ro.push_back(ro.back() + (it % 4 < 2 ? 16 : 1 + int(rng() % 128)));
    for (int k = 0; k < S; ++k) {
      off.push_back(off.back() + (it % 5 == 4 ? int(rng() % 10000) : 1 + int(rng() % most)));
      task.push_back(it % 7 == 0 ? k % 2 - 1 : int(rng() % (n + 1)) - 1);
    }
    lobra_mlora_desc d{};
    d.dtype = rng() % 2; d.d_in = 8 * (1 + rng() % 600); d.d_out = 8 * (1 + rng() % 600); d.T = off.back(); d.n_tasks = n; d.S = S;
    d.rank_off = ro.data(); d.seg_off = off.data(); d.seg_task = task.data();
    lobra::Plan p;
    lobra_status st = lobra::build_host_plan(&d, 0, &p);
    if (st != LOBRA_OK) { printf("long plan %d\n", st); return 1; }
    const size_t bytes = lobra::pack_blob(&p).size() * 4, runs = p.shrink_group > 1 ? 0 : p.sb_off.size() + p.sb_order.size();
    const size_t before = (p.o_tile_seg + runs + 8 * size_t((d.T + 255) / 256)) * 4;
    if (before <= 65536 && bytes > lobra::kUploadByArgument) { printf("%zu bytes of tables, %zu without the products'\n", bytes, before); return 1; }
  }
  printf("host fuzz ok\n");
  return 0;
}

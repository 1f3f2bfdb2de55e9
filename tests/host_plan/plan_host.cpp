// The device planner (pg_plan.hpp) compiled for the host and run on grouping arrays read
// from stdin, so the tests can check its plans and its handling of inconsistent arrays
// under AddressSanitizer (every array is allocated at exactly the size the library's host
// code gives it, so a read past the end is reported).
//
// stdin: mode (0 = one-block planner, 1 = multi-kernel planner), ng, ns, tp, ts, bm, bkv,
//        kv_chunks, split, max_q, max_kv, then cu_prefix_lens[ng+1], cu_suffix_lens[ns+1],
//        group_sizes[ng]; or mode 2 (the library's choices for a backward of these sizes) and
//        lines of dtype, ng, ns, tp, ts, h_q, h_kv, d, wide, wide_q, the last two 0 or 1 for a
//        given tiling or -1 for the library's rule; or mode 3 / 4 (the final-token call's plan in one
//        kernel / in two), ng, ns, tp, ts, members per block, most blocks, then the arrays.
// stdout: error n_qtiles n_kvtiles, then one line per query tile in rank order
//         ("q kind group row0 row1 aux work chunk nchunks"), the same for kv tiles ("k ..."),
//         then "s" followed by the per-row member starts (when the plan is valid); in mode 2, per
//         line: bm bkv kv_chunks split max_q max_kv one_block workspace size_query; in modes 3 and 4
//         error and the number of member blocks, then "b group m_first m_count" per block.
#include <cstdio>
#include <memory>

#include "pg_layout.hpp"
#include "pg_plan.hpp"

using namespace pg;

static int print_layouts() {
  int dtype, ng, ns, tp, ts, hq, hkv, d, wide, wide_q;
  while (scanf("%d %d %d %d %d %d %d %d %d %d", &dtype, &ng, &ns, &tp, &ts, &hq, &hkv, &d, &wide, &wide_q) == 10) {
    const Layout L = wide < 0 ? bwd_layout(dtype, ng, ns, tp, ts, hq, hkv, d)
                              : make_layout(ng, ns, tp, ts, hq, hkv, d, true, wide != 0, wide_q != 0);
    printf("%d %d %d %d %ld %ld %d %zu %zu\n", L.bm, L.bkv, L.kv_chunks, L.split, L.max_q, L.max_kv,
           (int)one_block_plan(L, true), L.total, bwd_workspace(ng, ns, tp, ts, hq, hkv, d));
  }
  return 0;
}

int main() {
  int mode, ng, ns, tp, ts, bm = kFwdBM, bkv = kKvBN, kvc = 1, split = 0, mpw = 0, nb_max = 0;
  long max_q = 0x7fffffffL, max_kv = 0x7fffffffL;
  if (scanf("%d", &mode) != 1) return 2;
  if (mode == 2) return print_layouts();
  const bool last = mode >= 3;
  if (last) {
    if (scanf("%d %d %d %d %d %d", &ng, &ns, &tp, &ts, &mpw, &nb_max) != 6) return 2;
  } else if (scanf("%d %d %d %d %d %d %d %d %ld %ld", &ng, &ns, &tp, &ts, &bm, &bkv, &kvc, &split, &max_q,
            &max_kv) != 10) {
    return 2;
  }
  std::unique_ptr<int[]> cu_p(new int[ng + 1]), cu_s(new int[ns + 1]), gsz(new int[ng > 0 ? ng : 1]);
  for (int i = 0; i <= ng; ++i) if (scanf("%d", &cu_p[i]) != 1) return 2;
  for (int i = 0; i <= ns; ++i) if (scanf("%d", &cu_s[i]) != 1) return 2;
  for (int i = 0; i < ng; ++i) if (scanf("%d", &gsz[i]) != 1) return 2;
  PlanHeader hdr{};
  std::unique_ptr<GroupInfoEx[]> gi(new GroupInfoEx[ng > 0 ? ng : 1]);
  std::unique_ptr<int[]> qoff(new int[ng + 1]), kvoff(new int[ng + 1]);
  if (last) {
    std::unique_ptr<LastBlock[]> blocks(new LastBlock[nb_max > 0 ? nb_max : 1]);
    int n = -1;
    if (mode == 3) {
      host_launch(1, kPlanThreads, [&] {
        plan_last_fused_kernel(cu_p.get(), cu_s.get(), gsz.get(), ng, ns, tp, ts, bm, bkv, &hdr, gi.get(), qoff.get(),
                               kvoff.get(), mpw, nb_max, blocks.get(), &n);
      });
    } else {
      host_launch(1, kPlanThreads, [&] {
        plan_groups_kernel(cu_p.get(), cu_s.get(), gsz.get(), ng, ns, tp, ts, bm, bkv, kvc, split, max_q, max_kv, &hdr,
                           gi.get(), qoff.get(), kvoff.get());
      });
      host_launch(1, kPlanThreads, [&] { plan_last_kernel(&hdr, gi.get(), ng, mpw, nb_max, blocks.get(), &n); });
    }
    printf("%d %d\n", hdr.error, n);
    for (int b = 0; b < n; ++b) printf("b %d %d %d\n", blocks[b].group, blocks[b].m_first, blocks[b].m_count);
    return 0;
  }
  const long nq_cap = max_q > 0 ? max_q : 1, nkv_cap = max_kv > 0 ? max_kv : 1;
  std::unique_ptr<TileDesc[]> qt(new TileDesc[nq_cap]), kt(new TileDesc[nkv_cap]);
  std::unique_ptr<int[]> qo(new int[nq_cap]), ko(new int[nkv_cap]);
  std::unique_ptr<int[]> seg(new int[ts > 0 ? ts : 1]);
  if (mode == 0) {
    host_launch(1, kPlanThreads, [&] {
      plan_fused_kernel(cu_p.get(), cu_s.get(), gsz.get(), ng, ns, tp, ts, bm, bkv, kvc, split, max_q, max_kv, &hdr,
                        gi.get(), qoff.get(), kvoff.get(), qt.get(), qo.get(), kt.get(), ko.get(), seg.get());
    });
  } else {
    host_launch(1, kPlanThreads, [&] {
      plan_groups_kernel(cu_p.get(), cu_s.get(), gsz.get(), ng, ns, tp, ts, bm, bkv, kvc, split, max_q, max_kv, &hdr,
                         gi.get(), qoff.get(), kvoff.get());
    });
    const unsigned bq = (unsigned)((max_q + 255) / 256), bk = (unsigned)((max_kv + 255) / 256);
    if (max_q > 0) {
      host_launch(bq, 256, [&] {
        plan_tiles_kernel(cu_s.get(), ng, bm, bkv, 1, split, (int)max_q, &hdr, gi.get(), qoff.get(), qt.get(), 0);
      });
      host_launch(bq, 256, [&] { plan_rank_kernel(&hdr, qt.get(), qo.get(), 0); });
    }
    if (max_kv > 0) {
      host_launch(bk, 256, [&] {
        plan_tiles_kernel(cu_s.get(), ng, bm, bkv, kvc, split, (int)max_kv, &hdr, gi.get(), kvoff.get(), kt.get(), 1);
      });
      host_launch(bk, 256, [&] { plan_rank_kernel(&hdr, kt.get(), ko.get(), 1); });
    }
  }
  if (mode == 1 && ts > 0) {
    host_launch((unsigned)((ts + 1023) / 1024), 1024, [&] { seg_start_kernel(cu_s.get(), ns, ts, &hdr, seg.get()); });
  }
  printf("%d %d %d\n", hdr.error, hdr.n_qtiles, hdr.n_kvtiles);
  if (hdr.error) return 0;
  for (int r = 0; r < hdr.n_qtiles; ++r) {
    const TileDesc& d = qt[qo[r]];
    printf("q %d %d %d %d %d %d %d %d\n", d.kind, d.group, d.row0, d.row1, d.aux, d.work, d.chunk, d.nchunks);
  }
  for (int r = 0; r < hdr.n_kvtiles; ++r) {
    const TileDesc& d = kt[ko[r]];
    printf("k %d %d %d %d %d %d %d %d\n", d.kind, d.group, d.row0, d.row1, d.aux, d.work, d.chunk, d.nchunks);
  }
  printf("s");
  for (int r = 0; r < ts; ++r) printf(" %d", seg[r]);
  printf("\n");
  return 0;
}

// Host-side choices that depend on a call's sizes alone: which kernels it runs (their tile sizes), into how
// many pieces prefix walks are cut, and where each array of the plan lies in the workspace. Plain C++: the
// tests compile it for the host and read these choices from it.
#pragma once
#include <stddef.h>

#include <algorithm>

#include "../../include/pg_attn.h"
#include "pg_plan.hpp"

namespace pg {

constexpr size_t kAlign = 256;
inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

inline long ceil_div_l(long a, long b) { return (a + b - 1) / b; }

// Workspace layout shared by the forward and backward calls.
struct Layout {
  size_t hdr, ginfo, qoff, kvoff, qtiles, qorder, kvtiles, kvorder, seg, dsum, lse2, part, xrow, total;
  long max_q, max_kv;
  int kv_chunks, split;
  int bkv;  // keys per key tile: kKvBN, or kWideBN for dkdv_wide_kernel
  int bm;   // query rows per query tile: kFwdBM, or kWideBM for the 256-row kernels
};

// Mean walk of a prefix key tile for 256-key tiles, in steps (32 query rows x 256 keys), from the mean group.
inline double wide_walk(int ng, int tp, int ts, int h_q, int h_kv) {
  return (double)(h_q / h_kv) * (0.5 * tp + ts) / ((double)(ng > 0 ? ng : 1) * kWideBQ);
}

// Pieces each prefix key tile's query walk is split into for the dK/dV kernel: enough
// workgroups to balance the long prefix walks over the CUs (about 512 prefix pieces, i.e.
// two per CU), at most 8, and 1 when there are already that many prefix key tiles. More
// pieces balance better but each adds a full fp32 partial to write and reduce; measured on
// the single-group and large-group workloads, 512 beats 256 and 1024-4096. A piece keeps at
// least 16 64-row query tiles of the average walk (a group's rows, once per query head of
// the kv head): shorter pieces cost more in their fixed start-up and in the reduce launch
// than they save. A grid of at most 128 key tiles (half the CUs) runs as long as its
// longest walk whatever the total work, so there pieces of one such tile pay off.
inline int kv_chunks_narrow(int ng, int tp, int ts, int h_q, int h_kv) {
  const long tiles = (ceil_div_l(tp, kKvBN) + ng) * (long)h_kv;
  long c = ceil_div_l(512, tiles);
  const long walk = ceil_div_l((long)tp + ts, (long)(ng > 0 ? ng : 1) * 64) * (h_q / h_kv);
  const long min_piece = 2 * tiles <= 256 ? 1 : 16;
  if (c > walk / min_piece) c = walk / min_piece;
  return (int)(c < 1 ? 1 : (c > 8 ? 8 : c));
}

// The same for 256-key tiles, which run one workgroup per CU. Where there is more than one, each piece costs
// 8 * total_prefix * h_kv * head_dim bytes of workspace. Measured on 660 random shapes (1..16 groups, 1..8 kv heads,
// 1..8 query heads each, both head dims), us of dK/dV and its reduction at 1, 2, .. pieces:
// * up to about 400 tiles the longest walk or a nearly empty last round sets the time, and about 384 pieces are
//   best: 106 tiles 2326, 1286, 949, 777 and 843 at five; 214 tiles 1658, 948; 388 tiles 2267, 1753;
// * above, one piece does as well (mean ratio of one to two 0.98 for walks of 260..1000 steps, 1.02 beyond) and
//   needs no partial sums, but for tiles just above two per CU with long walks: 544 tiles 7769, 6758; 560 tiles
//   6014, 5488. At 720 tiles (5077, 4737) two pieces would take 376 MB, at 512 (P 16384, 32/8 heads: 2%) 268 MB;
// * a piece of few steps does not pay for its start-up and partial sums (fewer than 50 steps, or 150 where the tiles
//   fill the CUs anyway): 432 tiles of 121 steps 453, 545; 652 tiles of 75 steps 394, 509.
inline int kv_chunks_wide(int ng, int tp, int ts, int h_q, int h_kv) {
  const long least = ceil_div_l(tp, kWideBN) * (long)h_kv, tiles = least + (long)ng * h_kv;
  const bool few = tiles <= 400;
  const long c = few || (least > 512 && tiles <= 640) ? std::max(2L, ceil_div_l(384, tiles)) : 1;
  const long most = (long)(wide_walk(ng, tp, ts, h_q, h_kv) / (few ? 50 : 150));
  return (int)std::max(1L, std::min({c, most, 8L}));
}

inline int kv_chunks_for(int ng, int tp, int ts, int h_q, int h_kv, int bkv) {
  if (tp <= 0 || h_kv <= 0) return 1;
  return bkv == kWideBN ? kv_chunks_wide(ng, tp, ts, h_q, h_kv) : kv_chunks_narrow(ng, tp, ts, h_q, h_kv);
}

// Problems whose stacked query tiles x heads cannot fill the 256 CUs tile each member's
// responses on their own (see response_tiles in the planner): their time is the longest
// tile walk, not the total work.
constexpr long kSplitBelow = 256;

// Whether the backward runs dkdv_wide_kernel (256-key tiles). It does the same work in fewer, longer
// workgroups, one per CU. Measured (dK/dV plus reduction, dkdv_kernel -> wide, us):
// * it needs work: at least 80 steps (32 query rows x 256 keys) per CU in the prefix walks. 24 steps 112 -> 123, 55
//   194 -> 203, 112 335 -> 297, 232 718 -> 675;
// * and pieces that share it: with few tiles the eight pieces a walk may have leave CUs idle while the longest ones
//   run, so no piece may take 1.5 times as long as all of them spread over the CUs. 5/1 heads, P 2440, 10 tiles
//   334 -> 515; 8/1, P 7653, d 64, 30 tiles 249 -> 320; the other side: 8/1, P 12122, 48 tiles 846 -> 697;
// * the line at prefixes of 1024 rows on average (ragged 256-key tiles below) is on the safe side: mean 300 rows
//   540 -> 608, but 773 rows, 488 tiles 4104 -> 3826 and 966 rows, d 64, 464 tiles 2313 -> 2236; above it 1451 rows
//   3842 -> 3505.
// Over 563 random shapes on this side of the lines it takes 0.89 of dkdv_kernel's time; 26 of them lose more than
// 1.5%, most of those with 64-wide heads and about 100 steps per CU (the worst 175 -> 219).
inline bool use_wide(int dtype, int ng, int tp, int ts, int h_q, int h_kv) {
  if (dtype != PG_BF16 || ng <= 0 || h_kv <= 0 || tp / 1024 < ng) return false;
  const double walk = wide_walk(ng, tp, ts, h_q, h_kv), longest = walk * ((double)tp + ts) / (0.5 * tp + ts);
  const double per_cu = walk * (double)ceil_div_l(tp, kWideBN) * h_kv / 256;
  return per_cu >= 80 && longest / kv_chunks_for(ng, tp, ts, h_q, h_kv, kWideBN) <= 1.5 * per_cu;
}

// Whether the backward runs dq_wide_kernel (256-row query tiles). Its workgroups have a CU to themselves,
// so loading their rows and storing dQ is not hidden: it needs long key walks, and enough tiles to give
// every CU two. Measured (dq_kernel -> wide), one group of 16/4 or 32/8 heads: P 1024 1278 -> 1468 us, 4096
// 2477 -> 2500 us, 8192 804 -> 770 us, 16384 4664 -> 4420 us; over 166 random shapes of 128-wide heads, 0.96 of
// dq_kernel's time on this side of the lines (0.94..1.02), 1.03 below 8192 rows, 1.09 below 4096, 1.2 below
// 2000. With 64-wide heads the vector work per product doubles and one wave per SIMD cannot issue it
// (206 -> 278 us on prefixes of 179..2530).
inline bool use_wide_q(int dtype, int ng, int tp, int ts, int h_q, int d) {
  return dtype == PG_BF16 && d == 128 && ng > 0 && tp / 8192 >= ng &&
         (ceil_div_l(tp, kWideBM) + ceil_div_l(ts, kWideBM)) * h_q >= 512;
}

inline Layout make_layout(int ng, int ns, int tp, int ts, int h_q, int h_kv, int d, bool bwd, bool wide = false,
                          bool wide_q = false) {
  Layout L{};
  L.bm = wide_q ? kWideBM : kFwdBM;
  L.bkv = wide ? kWideBN : kKvBN;
  L.kv_chunks = bwd ? kv_chunks_for(ng, tp, ts, h_q, h_kv, L.bkv) : 1;
  L.split = !wide_q && (ceil_div_l(tp, kFwdBM) + ceil_div_l(ts, kFwdBM) + ng) * (long)h_q < kSplitBelow ? 1 : 0;
  // bounds of the tile lists in either tiling (splitting adds at most one tile per member)
  L.max_q = ceil_div_l(tp, L.bm) + ceil_div_l(ts, L.bm) + 2L * ng + ns;
  L.max_kv = bwd ? (ceil_div_l(tp, L.bkv) + ng) * L.kv_chunks + ceil_div_l(ts, L.bkv) + ng + ns : 0;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off += align_up(bytes); return o; };
  const size_t rows = (size_t)tp + (size_t)ts;  // sizes are non-negative ints: no overflow in 64 bits
  L.hdr = take(sizeof(PlanHeader));
  L.ginfo = take(sizeof(GroupInfoEx) * (size_t)(ng > 0 ? ng : 1));
  L.qoff = take(sizeof(int) * ((size_t)ng + 1));
  L.kvoff = take(sizeof(int) * ((size_t)ng + 1));
  L.qtiles = take(sizeof(TileDesc) * (size_t)(L.max_q > 0 ? L.max_q : 1));
  L.qorder = take(sizeof(int) * (size_t)(L.max_q > 0 ? L.max_q : 1));
  L.kvtiles = take(sizeof(TileDesc) * (size_t)(L.max_kv > 0 ? L.max_kv : 1));
  L.kvorder = take(sizeof(int) * (size_t)(L.max_kv > 0 ? L.max_kv : 1));
  L.seg = take(sizeof(int) * (size_t)(ts > 0 ? ts : 1));
  L.dsum = bwd ? take(sizeof(float) * (size_t)h_q * (rows > 0 ? rows : 1)) : off;
  L.lse2 = bwd && wide ? take(sizeof(float) * (size_t)h_q * (rows > 0 ? rows : 1)) : off;
  L.part = (bwd && L.kv_chunks > 1) ? take(sizeof(float) * (size_t)L.kv_chunks * 2 * (size_t)tp * h_kv * d) : off;
  L.xrow = bwd ? take(sizeof(int) * (rows > 0 ? rows : 1)) : off;
  L.total = off;
  return L;
}

// The layout pg_attn_bwd and pg_attn_bwd_xours use.
inline Layout bwd_layout(int dtype, int ng, int ns, int tp, int ts, int h_q, int h_kv, int d) {
  return make_layout(ng, ns, tp, ts, h_q, h_kv, d, true, use_wide(dtype, ng, tp, ts, h_q, h_kv),
                     use_wide_q(dtype, ng, tp, ts, h_q, d));
}

// Bytes for a backward of these sizes in either type (the query does not know which).
inline size_t bwd_workspace(int ng, int ns, int tp, int ts, int h_q, int h_kv, int d) {
  return std::max(bwd_layout(PG_BF16, ng, ns, tp, ts, h_q, h_kv, d).total,
                  bwd_layout(PG_FP32, ng, ns, tp, ts, h_q, h_kv, d).total);
}

// Whether plan_fused_kernel plans the call: every tile list fits its one block.
inline bool one_block_plan(const Layout& L, bool bwd) {
  return L.max_q <= kPlanThreads && (!bwd || L.max_kv <= kPlanThreads);
}

}  // namespace pg

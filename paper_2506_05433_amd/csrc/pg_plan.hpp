// Device-side planner: validates the grouping arrays and builds the tile lists
// that the attention kernels walk, ordered longest-first.
//
// Query tiles follow the two attention calls of Eq. (4): prefix query tiles
// (causal self-attention over the prefix) and response query tiles. Response
// rows of all members of a group are stacked into common tiles: every one of
// them sees the whole group prefix, so the prefix part of a tile is a dense
// rectangle regardless of member boundaries, and only the response part needs
// the per-member causal mask. Key/value tiles are the mirror image for the
// key-stationary gradient kernel.
#pragma once
#include <hip/hip_runtime.h>

#include "pg_types.hpp"

namespace pg {

struct PlanHeader {
  int error;     // nonzero when the grouping arrays are inconsistent
  int n_qtiles;  // number of query tiles
  int n_kvtiles; // number of key/value tiles
  int pad[61];
};

struct GroupInfoEx {
  int p0, p1, s0, s1, m0, m1, pad0, pad1;
};

__device__ inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Inclusive scan of one value per thread over a block of NT threads.
template <int NT, typename V>
__device__ __forceinline__ V block_inclusive_scan(V v, V* tmp) {
  const int t = threadIdx.x;
  tmp[t] = v;
  __syncthreads();
  for (int off = 1; off < NT; off <<= 1) {
    V add = (t >= off) ? tmp[t - off] : 0;
    __syncthreads();
    tmp[t] += add;
    __syncthreads();
  }
  V r = tmp[t];
  __syncthreads();
  return r;
}

// Largest index i in [lo, hi) with a[i] <= x (a nondecreasing, a[lo] <= x).
__device__ __forceinline__ int upper_index(const int* a, int lo, int hi, int x) {
  while (hi - lo > 1) {
    int mid = (lo + hi) >> 1;
    if (a[mid] <= x) lo = mid; else hi = mid;
  }
  return lo;
}

constexpr int kPlanThreads = 1024;

// Shared memory of the one-block planner steps.
struct PlanShared {
  int tmp[kPlanThreads];
  long long tmp64[kPlanThreads];
  long long members;  // running sum of group sizes
  int err;
  int carry[3];
};

// Response tiles of a group: its response rows stacked into b-row tiles across member
// boundaries, or (split) each member's rows tiled on their own. Stacking wastes no rows
// and lets every tile share the group's prefix; splitting gives more, shorter tiles, which
// is what a problem too small to fill the GPU needs (its time is the longest tile walk).
__device__ inline int response_tiles(const int* __restrict__ cu_s, const GroupInfoEx& gi, int b, int split) {
  if (!split) return ceil_div(gi.s1 - gi.s0, b);
  int n = 0;
  // unrolled so that several members' lengths are loaded at once (one thread walks a group's members)
#pragma unroll 4
  for (int m = gi.m0; m < gi.m1; ++m) n += ceil_div(cu_s[m + 1] - cu_s[m], b);
  return n;
}

// One block of kPlanThreads threads. Validates and computes per-group ranges and tile offsets.
__device__ inline void plan_groups_body(const int* __restrict__ cu_p, const int* __restrict__ cu_s,
                                        const int* __restrict__ gsz, int ng, int ns, int tp, int ts, int bm, int bkv,
                                        int kv_chunks, int split, long max_q, long max_kv, PlanHeader* hdr,
                                        GroupInfoEx* ginfo, int* qoff, int* kvoff, PlanShared& sh) {
  int* tmp = sh.tmp;
  int& err = sh.err;
  int* carry = sh.carry;
  const int t = threadIdx.x;
  if (t == 0) { err = 0; carry[0] = carry[1] = carry[2] = 0; sh.members = 0; }
  __syncthreads();
  int bad = 0;
  for (int g = t; g <= ng; g += kPlanThreads) {
    int v = cu_p[g];
    if (g == 0 && v != 0) bad = 1;
    if (g == ng && v != tp) bad = 1;
    if (g > 0 && v < cu_p[g - 1]) bad = 1;
    if (g < ng && (gsz[g] < 0 || gsz[g] > ns)) bad = 1;
  }
  for (int m = t; m <= ns; m += kPlanThreads) {
    int v = cu_s[m];
    if (m == 0 && v != 0) bad = 1;
    if (m == ns && v != ts) bad = 1;
    if (m > 0 && v < cu_s[m - 1]) bad = 1;
  }
  if (bad) atomicOr(&err, 1);
  __syncthreads();
  // member starts: exclusive scan of group sizes, in 64 bits so that no sum of sizes can wrap
  // around to n_suffixes; checked against it afterwards, and only then are the starts used to
  // index cu_suffix_lens
  for (int base = 0; base < ng; base += kPlanThreads) {
    const int g = base + t;
    const long long v = (g < ng && !err) ? gsz[g] : 0;
    const long long inc = block_inclusive_scan<kPlanThreads>(v, sh.tmp64);
    const long long m1 = sh.members + inc;
    if (g < ng) { ginfo[g].m0 = (int)(m1 - v); ginfo[g].m1 = (int)m1; }
    __syncthreads();
    if (t == kPlanThreads - 1) sh.members = m1;
    __syncthreads();
  }
  if (t == 0 && sh.members != ns) err = 1;
  __syncthreads();
  const int ok = !err;
  for (int base = 0; base < ng; base += kPlanThreads) {
    const int g = base + t;
    int nq = 0, nkv = 0;
    if (g < ng && ok) {
      GroupInfoEx gi = ginfo[g];
      gi.p0 = cu_p[g]; gi.p1 = cu_p[g + 1];
      gi.s0 = cu_s[gi.m0]; gi.s1 = cu_s[gi.m1];
      gi.pad0 = gi.pad1 = 0;
      ginfo[g] = gi;
      nq = ceil_div(gi.p1 - gi.p0, bm) + response_tiles(cu_s, gi, bm, split);
      nkv = ceil_div(gi.p1 - gi.p0, bkv) * kv_chunks + response_tiles(cu_s, gi, bkv, split);
    }
    const int iq = block_inclusive_scan<kPlanThreads>(nq, tmp);
    const int ikv = block_inclusive_scan<kPlanThreads>(nkv, tmp);
    if (g < ng) { qoff[g] = carry[1] + iq - nq; kvoff[g] = carry[2] + ikv - nkv; }
    __syncthreads();
    if (t == kPlanThreads - 1) { carry[1] += iq; carry[2] += ikv; }
    __syncthreads();
  }
  // the host sized the tile arrays from the totals; a list longer than that bound
  // can only come from inconsistent arrays, so it is treated as an error too
  if (t == 0 && ok && (carry[1] > max_q || carry[2] > max_kv)) err = 1;
  __syncthreads();
  if (t == 0) {
    const int ok = !err;
    qoff[ng] = ok ? carry[1] : 0;
    kvoff[ng] = ok ? carry[2] : 0;
    hdr->error = err;
    hdr->n_qtiles = ok ? carry[1] : 0;
    hdr->n_kvtiles = ok ? carry[2] : 0;
  }
}

// Grouping arrays small enough for LDS (the usual case) are planned from there. The one-block steps are
// all latency: every dependent global load costs 0.5 to 1 us and a 1024-wide scan twenty barriers, so the
// arrays are loaded once, side by side, searched in LDS, and summed by wave scans (one barrier, or none up to 63
// groups). Measured, plan_groups_kernel (the rotary embedding's plan), from memory -> from LDS: 1 group 9.9 -> 6.2
// us, 100 groups 9.9 -> 6.6, 1000 groups 11.2 -> 8.4; with each thread adding up the entries before its own instead
// 6.2, 11.7, 91.7 (the sums are the only step that grows with the square of the groups, so they stay scans).
// plan_fused_kernel: 1 group of 4 members, 6 tiles 10.8 -> 6.3 us; 7 groups of 6 (6210 + 19050 rows, about 400
// key tiles) 19.5 -> 11.0 us, of which the ranks took half before their comparisons were shared out and cut to
// four instructions.
constexpr int kLdsGroups = kPlanThreads - 1;  // one thread per group, and one for the totals
constexpr int kLdsMembers = 4096;

__host__ __device__ inline bool plan_fits_lds(int ng, int ns) { return ng <= kLdsGroups && ns <= kLdsMembers; }

struct PlanLds {
  alignas(16) int work[2][kPlanThreads];  // the tiles' ranking keys, -1 past the last tile
  alignas(16) int tot[4][kPlanThreads / 64];  // sums of each wave, one row per prefix sum
  int part[kPlanThreads];                 // partial ranks
  int cu_p[kLdsGroups + 1], cu_s[kLdsMembers + 1], qoff[kLdsGroups + 1], kvoff[kLdsGroups + 1];
  GroupInfoEx gi[kLdsGroups + 1];
  int err;
};

struct alignas(16) Int4 {
  int v[4];
};

// Exclusive prefix sums over the block of N values per thread, of which only those of the first n threads may be
// nonzero; results are meant for threads 0 .. n. A wave scan, then the sums of the waves before (tot, N rows of
// one entry per wave, not used again by the caller before a barrier); up to 63 values need neither barrier nor tot.
template <int N>
__device__ __forceinline__ void block_exclusive_sums(int (&v)[N], int n, int (*tot)[kPlanThreads / 64]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int x[N];
#pragma unroll
  for (int k = 0; k < N; ++k) x[k] = v[k];
#pragma unroll
  for (int off = 1; off < 64; off <<= 1)
#pragma unroll
    for (int k = 0; k < N; ++k) {
      const int y = __shfl_up(x[k], off);
      x[k] += lane >= off ? y : 0;
    }
  if (n >= 64) {
    if (lane == 63)
#pragma unroll
      for (int k = 0; k < N; ++k) tot[k][wave] = x[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < N; ++k)
#pragma unroll
      for (int w = 0; w < kPlanThreads / 64; w += 4) {
        const Int4 q = *(const Int4*)(tot[k] + w);
#pragma unroll
        for (int e = 0; e < 4; ++e) x[k] += w + e < wave ? q.v[e] : 0;
      }
  }
#pragma unroll
  for (int k = 0; k < N; ++k) v[k] = x[k] - v[k];
}

// plan_groups_body for arrays that fit PlanLds: the same checks, ranges and offsets. Leaves copies of
// the arrays, ranges and offsets in `sh` (valid when it returns true, that is without an error).
__device__ inline bool plan_groups_lds(const int* __restrict__ cu_p, const int* __restrict__ cu_s,
                                       const int* __restrict__ gsz, int ng, int ns, int tp, int ts, int bm, int bkv,
                                       int kv_chunks, int split, long max_q, long max_kv, PlanHeader* hdr,
                                       GroupInfoEx* ginfo, int* qoff, int* kvoff, PlanLds& sh) {
  const int t = threadIdx.x;
  for (int m = t; m <= ns; m += kPlanThreads) sh.cu_s[m] = cu_s[m];
  if (t <= ng) sh.cu_p[t] = cu_p[t];
  const int size = t < ng ? gsz[t] : 0;
  // sizes out of range are an error; they are kept out of the sums, whose results are used as indices
  // (and which fit 32 bits: at most kLdsGroups sizes of at most kLdsMembers)
  const bool bad_size = size < 0 || size > ns;
  const int members = bad_size ? 0 : size;
  if (t == 0) sh.err = 0;
  __syncthreads();
  int bad = bad_size;
  if (t <= ng) {
    const int v = sh.cu_p[t];
    if ((t == 0 && v != 0) || (t == ng && v != tp) || (t > 0 && v < sh.cu_p[t - 1])) bad = 1;
  }
  for (int m = t; m <= ns; m += kPlanThreads) {
    const int v = sh.cu_s[m];
    if ((m == 0 && v != 0) || (m == ns && v != ts) || (m > 0 && v < sh.cu_s[m - 1])) bad = 1;
  }
  int start[1] = {members};
  block_exclusive_sums(start, ng, sh.tot);
  const int m0 = start[0];
  if (t <= ng && ((t == ng && m0 != ns) || m0 + members > ns)) bad = 1;
  if (bad) atomicOr(&sh.err, 1);
  __syncthreads();
  const bool ok = !sh.err;
  int n[2] = {0, 0};  // query and key tiles
  if (ok && t < ng) {
    GroupInfoEx gi;
    gi.m0 = m0;
    gi.m1 = m0 + members;
    gi.p0 = sh.cu_p[t];
    gi.p1 = sh.cu_p[t + 1];
    gi.s0 = sh.cu_s[gi.m0];
    gi.s1 = sh.cu_s[gi.m1];
    gi.pad0 = gi.pad1 = 0;
    sh.gi[t] = gi;
    ginfo[t] = gi;
    n[0] = ceil_div(gi.p1 - gi.p0, bm) + response_tiles(sh.cu_s, gi, bm, split);
    n[1] = ceil_div(gi.p1 - gi.p0, bkv) * kv_chunks + response_tiles(sh.cu_s, gi, bkv, split);
  }
  block_exclusive_sums(n, ng, sh.tot + 1);
  if (t <= ng) {
    sh.qoff[t] = n[0];
    sh.kvoff[t] = n[1];
    // the host sized the tile arrays from the totals; a list longer than that bound can only come
    // from inconsistent arrays, so it is treated as an error too
    if (t == ng && ok && (n[0] > max_q || n[1] > max_kv)) sh.err = 1;
  }
  __syncthreads();
  const bool good = !sh.err;
  if (t <= ng) {
    qoff[t] = t < ng || good ? sh.qoff[t] : 0;
    kvoff[t] = t < ng || good ? sh.kvoff[t] : 0;
  }
  if (t == 0) {
    hdr->error = sh.err;
    hdr->n_qtiles = good ? sh.qoff[ng] : 0;
    hdr->n_kvtiles = good ? sh.kvoff[ng] : 0;
  }
  return good;
}

__global__ void __launch_bounds__(kPlanThreads) plan_groups_kernel(
    const int* __restrict__ cu_p, const int* __restrict__ cu_s, const int* __restrict__ gsz,
    int ng, int ns, int tp, int ts, int bm, int bkv, int kv_chunks, int split, long max_q, long max_kv,
    PlanHeader* hdr, GroupInfoEx* ginfo, int* qoff, int* kvoff) {
  if (plan_fits_lds(ng, ns)) {
    __shared__ PlanLds lds;
    plan_groups_lds(cu_p, cu_s, gsz, ng, ns, tp, ts, bm, bkv, kv_chunks, split, max_q, max_kv, hdr, ginfo, qoff,
                    kvoff, lds);
    return;
  }
  __shared__ PlanShared sh;
  plan_groups_body(cu_p, cu_s, gsz, ng, ns, tp, ts, bm, bkv, kv_chunks, split, max_q, max_kv, hdr, ginfo, qoff, kvoff,
                   sh);
}

// Descriptor of tile i (< the number of tiles). `which` 0 = query tiles, 1 = kv tiles.
// Returns the tile's work (the ranking key).
__device__ inline int plan_tile(int i, const int* __restrict__ cu_s, int ng, int bm, int bkv, int kv_chunks,
                                 int split, const GroupInfoEx* __restrict__ ginfo, const int* __restrict__ off,
                                 TileDesc* tiles, int which) {
  const int g = upper_index(off, 0, ng, i);  // off[ng] == n > i, groups with no tile share offsets
  // skip groups with zero tiles that share the offset of the next one
  const GroupInfoEx gi = ginfo[g];
  const int b = which ? bkv : bm;
  const int chunks = which ? kv_chunks : 1;
  int local = i - off[g];
  const int np = ceil_div(gi.p1 - gi.p0, b) * chunks;
  TileDesc d;
  d.group = g;
  d.chunk = 0;
  d.nchunks = 1;
  if (local < np) {
    d.kind = 0;
    d.chunk = local % chunks;
    d.nchunks = chunks;
    local /= chunks;
    d.row0 = gi.p0 + local * b;
    d.row1 = min(d.row0 + b, gi.p1);
    if (!which) {
      d.aux = 0;
      d.work = d.row1 - gi.p0;                          // keys seen by the last row
    } else {
      d.aux = 0;
      d.work = ((gi.p1 - d.row0) + (gi.s1 - gi.s0)) / chunks;  // query rows that see these keys
    }
  } else {
    d.kind = 1;
    int lo = gi.s0, hi = gi.s1;  // the rows the tile is cut from: the group's, or one member's
    local -= np;
    if (split) {
#pragma unroll 4
      for (int m = gi.m0; m < gi.m1; ++m) {
        const int t = ceil_div(cu_s[m + 1] - cu_s[m], b);
        if (local < t) {
          lo = cu_s[m];
          hi = cu_s[m + 1];
          break;
        }
        local -= t;
      }
    }
    d.row0 = lo + local * b;
    d.row1 = min(d.row0 + b, hi);
    if (!which) {
      const int m = upper_index(cu_s, gi.m0, gi.m1, d.row0);
      d.aux = cu_s[m];                                  // first response key of the tile
      d.work = (gi.p1 - gi.p0) + (d.row1 - d.aux);
    } else {
      const int m = upper_index(cu_s, gi.m0, gi.m1, d.row1 - 1);
      d.aux = cu_s[m + 1];                              // end of queries that see the keys
      d.work = d.aux - d.row0;
    }
  }
  tiles[i] = d;
  return d.work;
}

// One thread per (possible) tile: fills the descriptors.
__global__ void plan_tiles_kernel(const int* __restrict__ cu_s, int ng, int bm, int bkv, int kv_chunks, int split,
                                  int max_tiles, const PlanHeader* hdr, const GroupInfoEx* __restrict__ ginfo,
                                  const int* __restrict__ off, TileDesc* tiles, int which) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int n = which ? hdr->n_kvtiles : hdr->n_qtiles;
  if (i >= n || i >= max_tiles) return;
  plan_tile(i, cu_s, ng, bm, bkv, kv_chunks, split, ginfo, off, tiles, which);
}

// How many of the works w[lo .. hi) come before work `mine` of index i, w[0] having index `base`: by
// (work desc, index asc). lo and hi are multiples of four; places past the last tile hold -1.
__device__ inline int rank_among(const int* w, int lo, int hi, int base, int mine, int i) {
  int rank = 0;
#pragma unroll 4
  for (int k = lo; k < hi; k += 4) {
    const Int4 x = *(const Int4*)(w + k);
#pragma unroll
    for (int e = 0; e < 4; ++e) rank += x.v[e] >= mine + (base + k + e >= i);
  }
  return rank;
}

// Longest-first order: order[rank] = tile, rank by (work desc, index asc). Deterministic.
__global__ void __launch_bounds__(256) plan_rank_kernel(const PlanHeader* hdr, const TileDesc* __restrict__ tiles,
                                                        int* order, int which) {
  alignas(16) __shared__ int w[1024];
  const int n = which ? hdr->n_kvtiles : hdr->n_qtiles;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if ((int)(blockIdx.x * blockDim.x) >= n) return;
  const int mine = i < n ? tiles[i].work : 0;
  int rank = 0;
  for (int base = 0; base < n; base += 1024) {
    __syncthreads();
    for (int k = threadIdx.x; k < 1024; k += blockDim.x) w[k] = (base + k < n) ? tiles[base + k].work : -1;
    __syncthreads();
    if (i < n) rank += rank_among(w, 0, (min(1024, n - base) + 3) & ~3, base, mine, i);
  }
  if (i < n) order[rank] = i;
}

// seg_start[r] = first row of the member that owns response row r.
__global__ void seg_start_kernel(const int* __restrict__ cu_s, int ns, int ts, const PlanHeader* hdr,
                                 int* seg_start) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= ts || hdr->error) return;
  seg_start[r] = cu_s[upper_index(cu_s, 0, ns, r)];
}

// Row map of the single-buffer layout of Eq. (2) (per group [P; R_1; ...; R_G], groups
// one after another): xrow[t] for packed prefix row t, xrow[total_prefix + s] for packed
// response row s. Prefix row t of group g is preceded by the responses of the earlier
// groups (s0 of g rows); response row s of group g by the prefixes of groups 0..g (p1).
__device__ inline void xrow_of(int row, const int* __restrict__ cu_p, const int* __restrict__ cu_s, int ng, int ns,
                               int tp, const GroupInfoEx* __restrict__ ginfo, int* xrow) {
  if (row < tp) {
    const int g = upper_index(cu_p, 0, ng, row);
    xrow[row] = row + ginfo[g].s0;
    return;
  }
  const int s = row - tp;
  const int m = upper_index(cu_s, 0, ns, s);
  int lo = 0, hi = ng;  // the group of member m: the last group whose members start at or before m
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (ginfo[mid].m0 <= m) lo = mid; else hi = mid;
  }
  xrow[row] = s + ginfo[lo].p1;
}

__global__ void xrow_kernel(const int* __restrict__ cu_p, const int* __restrict__ cu_s, int ng, int ns, int tp,
                            int ts, const PlanHeader* hdr, const GroupInfoEx* __restrict__ ginfo, int* xrow) {
  const int row = blockIdx.x * blockDim.x + threadIdx.x;
  if (row >= tp + ts || hdr->error) return;
  xrow_of(row, cu_p, cu_s, ng, ns, tp, ginfo, xrow);
}

// Groups, tile descriptors and longest-first ranks in one block, for plans whose tile
// lists each fit in kPlanThreads entries (the host checks the bounds): the steps above in
// order, separated by block barriers instead of kernel boundaries, with the same results.
// Saves the launch and memory latency of two to four dependent one-block kernels per call.
// The per-row tables (seg_start_kernel, xrow_kernel) stay separate wide launches: one
// block would walk every row.
__global__ void __launch_bounds__(kPlanThreads) plan_fused_kernel(
    const int* __restrict__ cu_p, const int* __restrict__ cu_s, const int* __restrict__ gsz, int ng, int ns, int tp,
    int ts, int bm, int bkv, int kv_chunks, int split, long max_q, long max_kv, PlanHeader* hdr, GroupInfoEx* ginfo,
    int* qoff, int* kvoff, TileDesc* qtiles, int* qorder, TileDesc* kvtiles, int* kvorder, int* seg_start) {
  // the host takes this kernel where 2 ng + ns <= kPlanThreads, so the arrays always fit
  __shared__ PlanLds lds;
  const int t = threadIdx.x;
  const GroupInfoEx* gi = lds.gi;
  const int *cs = lds.cu_s, *oq = lds.qoff, *okv = lds.kvoff;
  const bool ok = plan_groups_lds(cu_p, cu_s, gsz, ng, ns, tp, ts, bm, bkv, kv_chunks, split, max_q, max_kv, hdr,
                                  ginfo, qoff, kvoff, lds);
  const int nq = ok ? lds.qoff[ng] : 0, nkv = ok && kvtiles ? lds.kvoff[ng] : 0;
  // both counts are at most kPlanThreads, a host bound
  const int wq = t < nq ? plan_tile(t, cs, ng, bm, bkv, 1, split, gi, oq, qtiles, 0) : -1;
  const int wkv = t < nkv ? plan_tile(t, cs, ng, bm, bkv, kv_chunks, split, gi, okv, kvtiles, 1) : -1;
  lds.work[0][t] = wq;
  lds.work[1][t] = wkv;
  // the per-row member starts (what seg_start_kernel computes), when asked for
  if (seg_start && ok)
    for (int r = t; r < ts; r += kPlanThreads) seg_start[r] = cs[upper_index(cs, 0, ns, r)];
  __syncthreads();
  // longest-first ranks, the rule of plan_rank_kernel; `parts` threads share a tile's comparisons
  for (int which = 0; which < 2; ++which) {
    const int n = which ? nkv : nq;
    if (n == 0) continue;  // the same for every thread
    int np = 64;
    while (np < n) np *= 2;
    const int i = t & (np - 1), part = t / np, parts = kPlanThreads / np;
    const int* w = lds.work[which];
    const int len = ((n + parts - 1) / parts + 3) & ~3, lo = min(part * len, kPlanThreads), hi = min(lo + len, (n + 3) & ~3);
    lds.part[t] = i < n ? rank_among(w, lo, hi, 0, w[i], i) : 0;
    __syncthreads();
    if (t < n) {
      int rank = 0;
      for (int k = 0; k < parts; ++k) rank += lds.part[t + k * np];
      (which ? kvorder : qorder)[rank] = t;
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------- final-token call (pg_last.hpp)
// A run of a group's members whose final queries share a workgroup.
struct LastBlock {
  int group, m_first, m_count, pad;
};

// Member blocks: group g's members in runs of at most mpw, groups in order (one block of
// kPlanThreads threads; groups processed in passes with a running offset).
__global__ void __launch_bounds__(kPlanThreads) plan_last_kernel(const PlanHeader* hdr, const GroupInfoEx* ginfo,
                                                                 int ng, int mpw, int nb_max, LastBlock* blocks,
                                                                 int* n_blocks) {
  __shared__ int tmp[kPlanThreads];
  __shared__ int carry;
  const int t = threadIdx.x;
  if (t == 0) carry = 0;
  __syncthreads();
  const bool ok = !hdr->error;
  for (int base = 0; base < ng; base += kPlanThreads) {
    const int g = base + t;
    const int members = (g < ng && ok) ? ginfo[g].m1 - ginfo[g].m0 : 0;
    const int nb = (members + mpw - 1) / mpw;
    const int inc = block_inclusive_scan<kPlanThreads>(nb, tmp);
    const int first = carry + inc - nb;
    for (int k = 0; k < nb; ++k) {
      if (first + k < nb_max) {
        LastBlock b;
        b.group = g;
        b.m_first = ginfo[g].m0 + k * mpw;
        b.m_count = min(mpw, members - k * mpw);
        b.pad = 0;
        blocks[first + k] = b;
      }
    }
    __syncthreads();
    if (t == kPlanThreads - 1) carry += inc;
    __syncthreads();
  }
  if (t == 0) *n_blocks = ok ? min(carry, nb_max) : 0;
}

// The planner's groups and the member blocks in one launch, for grouping arrays that fit LDS: the calls
// this serves are short (one text of 4096 rows and 8 questions: the two launches were 10.8 of 26 us).
__global__ void __launch_bounds__(kPlanThreads) plan_last_fused_kernel(
    const int* __restrict__ cu_p, const int* __restrict__ cu_s, const int* __restrict__ gsz, int ng, int ns, int tp,
    int ts, int bm, int bkv, PlanHeader* hdr, GroupInfoEx* ginfo, int* qoff, int* kvoff, int mpw, int nb_max,
    LastBlock* blocks, int* n_blocks) {
  __shared__ PlanLds lds;
  const bool ok = plan_groups_lds(cu_p, cu_s, gsz, ng, ns, tp, ts, bm, bkv, 1, 0, 0x7fffffffL, 0x7fffffffL, hdr, ginfo,
                                  qoff, kvoff, lds);
  const int t = threadIdx.x;
  const int members = ok && t < ng ? lds.gi[t].m1 - lds.gi[t].m0 : 0;
  const int nb = (members + mpw - 1) / mpw;
  int below[1] = {nb};
  block_exclusive_sums(below, ng, lds.tot + 3);
  if (t > ng) return;
  const int first = below[0];
  for (int k = 0; k < nb; ++k)
    if (first + k < nb_max) {
      LastBlock b;
      b.group = t;
      b.m_first = lds.gi[t].m0 + k * mpw;
      b.m_count = min(mpw, members - k * mpw);
      b.pad = 0;
      blocks[first + k] = b;
    }
  if (t == ng) *n_blocks = ok ? min(first, nb_max) : 0;
}

}  // namespace pg

// The backward of large bf16 problems: dkdv_wide_kernel (256 keys per workgroup, 64 per wave) and
// dq_wide_kernel (256 query rows per workgroup, 64 per wave), one wave per SIMD with all 512 registers.
//
// What bounds them: the chip's power. On N(0,1) data a loop of nothing but 32x32x16 products reaches
// 1841 TFLOP/s (the clock falls to 1.76 GHz); with one LDS operand fragment read per product it
// reaches 1461, with one per two products 1590. dkdv_kernel reads one per product, hands P from one
// wave to another through LDS and walks every query tile once per 128 keys. Here a fragment serves
// both 32-key blocks of a wave, P and dS never leave their wave, and a query tile is walked once per
// 256 keys (half the cache traffic).
//
// With one wave per SIMD the wave issues one instruction about every four clocks and nothing else
// hides a wait, so the order of instructions is the design: each step's products, LDS reads, vector
// work and address arithmetic are interleaved by hand and pinned (sched_barrier), operands are read
// two to four steps ahead, address arithmetic is incremental, and the accumulators (256 registers)
// sit in AGPRs named in the instructions.
//
// Measured on 8 groups x 16 members, P 1246..26888, 64/8 heads, d 128: 240.1 -> 203.2 ms (1190 TFLOP/s of
// its four products; matrix cores 63% busy at 1.81 GHz); 1 x 16, P 16384, 32/8: 7.35 -> 6.30 ms; 1 x 8, P 4096, 32/8:
// 1.056 -> 0.909 ms with the reduction; 4 x 16, P 8192, 32/8, d 64: 16.05 -> 13.89 ms. Waves there (one per SIMD) issue
// 55% of their time, wait for a dependency 24% and to issue 21% (dq_wide_kernel 57, 21 and 23%).
// Measured and not kept: V (or more of K) in LDS instead of registers; S, dP, dV, dK each in turn with
// P beside dP and dS beside dV only (3% slower: the vector work does not fit those phases); two wait
// states before every product instead of before the first that reads new operands (2% slower).
#pragma once
#include "pg_bwd.hpp"
#include "pg_wide.hpp"

namespace pg {

constexpr int kWideKeys = kWideBN / 4;  // keys per wave

constexpr int kDenseRow = 1 << 30;  // stands for a row that sees every key

template <int D>
__global__ void __launch_bounds__(kWideThreads, 1) dkdv_wide_kernel(const BwdArgs a) {
  using T = bf16;
  using E = Elt<bf16>;
  using Frag = E::Frag;
  constexpr int BQ = kWideBQ;
  constexpr int KK = D / 16, DB = D / 32;
  constexpr int NBUF = 4;
  constexpr int PF = D == 128 ? 3 : 2;  // row fragments read ahead of their products
  constexpr int AHEAD = 3;              // transposed fragments read ahead
  constexpr int DR = 4;                 // steps over which Dsum is loaded into the accumulators
  // K fragments of the second key block that are kept in LDS: at head_dim 128 not all fit the registers
  constexpr int KL = D == 128 ? 5 : 0;
  constexpr int TILE = LdsTile<T, D>::bytes(BQ);
  constexpr int STAGE = 2 * TILE + 1024;  // Q, dO, per-row values (four arrays of 64 floats)
  constexpr int PW = TILE / 1024 / 2;     // copies per wave and tile: two waves fill Q, two dO
  static_assert(TILE % 2048 == 0, "copies split evenly over the waves");
  __shared__ __attribute__((aligned(1024))) char stage[NBUF * STAGE];
  __shared__ __attribute__((aligned(16))) Frag s_k[4][KL > 0 ? KL : 1][64];

  const BlockSlot slot = xcd_slot(blockIdx.x, a.h_kv, 1);
  const int rank = uniform(slot.unit), kvh = uniform(slot.head);
  if (rank >= a.hdr->n_kvtiles) return;
  // the descriptors in scalar registers, so that everything derived from them is too
  const TileDesc* tp = a.kvtiles + uniform(a.kvorder[rank]);
  const GroupInfoEx* gp = a.ginfo + uniform(tp->group);
  struct { int row0, row1, aux, chunk, nchunks; } td = {uniform(tp->row0), uniform(tp->row1), uniform(tp->aux),
                                                        uniform(tp->chunk), uniform(tp->nchunks)};
  struct { int p0, p1, s0, s1; } gi = {uniform(gp->p0), uniform(gp->p1), uniform(gp->s0), uniform(gp->s1)};
  const bool kv_suffix = uniform(tp->kind) == 1;
  const int xo_pre = a.xl ? gi.s0 : 0, xo_suf = a.xl ? gi.p1 : 0;
  const int xk = kv_suffix ? xo_suf : xo_pre;
  const int ratio = uniform(a.h_q / a.h_kv);
  const int rows_all = a.total_prefix + a.total_suffix;

  const int tid = threadIdx.x, wave = uniform(tid >> 6), lane = tid & 63;
  const int n = lane & 31, hh = lane >> 5;
  const int wk0 = td.row0 + kWideKeys * wave;
  const bool wave_active = wk0 < td.row1;
  const int wk1 = min(wk0 + kWideKeys, td.row1) - 1;

  // B operands: K, and V negated: dP accumulates Dsum - dO V^T, so that the accumulator can start at
  // Dsum; the sign goes into dK's final scale
  Frag kf[2][KK], vf[2][KK];
  int key_c[2];
  bool kvalid[2];
#pragma unroll
  for (int kb = 0; kb < 2; ++kb) {
    const int key = wk0 + 32 * kb + n;
    kvalid[kb] = key < td.row1;
    key_c[kb] = kvalid[kb] ? key : td.row1 - 1;
    const size_t off = ((size_t)(key_c[kb] + xk) * a.h_kv + kvh) * D + 8 * hh;
    const T* K = (const T*)(kv_suffix ? a.k_suf : a.k_pre) + off;
    const T* V = (const T*)(kv_suffix ? a.v_suf : a.v_pre) + off;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      kf[kb][kk] = E::global_row(K + 16 * kk, kvalid[kb]);
      if (kb == 1 && kk >= KK - KL) s_k[wave][kk - (KK - KL)][lane] = kf[kb][kk];
      const u32x4 v = __builtin_bit_cast(u32x4, E::global_row(V + 16 * kk, kvalid[kb]));
      vf[kb][kk] = __builtin_bit_cast(Frag, v ^ 0x80008000u);
    }
  }
  // accumulators: dV^T blocks (kb, db) from a0, dK^T blocks from a[32 DB]
  static_for<64 * DB>([](auto r) { acc_zero<decltype(r)::value>(); });

  // query ranges that see these keys, in the order of dkdv_kernel
  const int rc_lo = td.row0;                       // causal range
  const int rc_hi = kv_suffix ? td.aux : gi.p1;
  const int rd_lo = kv_suffix ? 0 : gi.s0;         // dense range
  const int rd_hi = kv_suffix ? 0 : gi.s1;
  const int nd = (rd_hi - rd_lo + BQ - 1) / BQ;
  const int nc = (rc_hi - rc_lo + BQ - 1) / BQ;
  const int per_head = nd + nc;
  const int walk = per_head * ratio;
  const int it0 = uniform((int)((long)walk * td.chunk / td.nchunks));
  const int it1 = uniform((int)((long)walk * (td.chunk + 1) / td.nchunks));
  const float c = a.scale_log2;

  // Copies: waves 0, 1 fill the Q tile and waves 2, 3 the dO tile (copy w = wave % 2 + 2 k fills
  // bytes [1024 w, 1024 w + 1024) of it), and each wave one array of per-row values: lse, Dsum,
  // member starts (zeros for prefix keys, which need none), and wave 3 Dsum again, so that every
  // wave has the same number of copies in flight. lse comes in log2 units, as dq_kernel stored it.
  int voff[PW];
#pragma unroll
  for (int k = 0; k < PW; ++k) {
    const int p = 1024 * ((wave & 1) + 2 * k) + 16 * lane;
    const int row = p / LdsTile<T, D>::kPitch, pc = (p % LdsTile<T, D>::kPitch) / 16;
    voff[k] = pc < LdsTile<T, D>::kChunks ? row * a.h_q * D * 2 + 16 * (pc ^ LdsTile<T, D>::swz(row)) : 0x7ffffff0;
  }
  const unsigned lds_tile = lds_addr(stage) + TILE * (wave >> 1) + 1024 * (wave & 1);
  const unsigned lds_row = lds_addr(stage) + 2 * TILE + 256 * wave;
  const int row_bytes = a.h_q * D * 2, val_bytes = wave == 2 && !kv_suffix ? 0 : 4;
  // this wave's source arrays at row 0, head 0 of the prefix and the response side, and the row
  // count between two heads' values
  const uint64_t src_pre = (uint64_t)((const T*)(wave < 2 ? a.q_pre : a.do_pre) + (size_t)xo_pre * a.h_q * D);
  const uint64_t src_suf = (uint64_t)((const T*)(wave < 2 ? a.q_suf : a.do_suf) + (size_t)xo_suf * a.h_q * D);
  const float* val = wave == 2 ? (const float*)a.seg_start : wave == 0 ? a.lse2 : a.dsum;
  const uint64_t val_pre = (uint64_t)val, val_suf = (uint64_t)(val + (wave == 2 ? 0 : a.total_prefix));
  const int val_ld = wave == 2 ? 0 : rows_all;
  // The run of tiles (one range of one head) that the copies are in: the sources of the next tile
  // and its rows left. Advancing a tile adds constants; only a new run computes addresses.
  int ld_hd = uniform(it0 / (per_head > 0 ? per_head : 1)), ld_j = it0 - ld_hd * per_head;
  const int first_j = ld_j;
  int ld_left = 0;
  u32x4 rs_t, rs_r;  // buffer descriptors of the next tile and of its per-row values
  rs_t[3] = rs_r[3] = 0x00020000;
  auto move_to = [&](u32x4& rs, uint64_t addr) PG_INLINE {
    rs[0] = uniform((int)(unsigned)addr);
    rs[1] = uniform((int)(unsigned)(addr >> 32));
  };
  auto set_rows = [&]() PG_INLINE {
    const int rows = min(ld_left, BQ);  // past the walk's end a tile has no rows: zeros are stored
    rs_t[2] = rows * row_bytes;
    rs_r[2] = rows * val_bytes;
  };
  auto new_run = [&](int hd, int j) PG_INLINE {
    const int hq = kvh * ratio + hd;
    const bool causal = j >= nd, qsuf = !causal || kv_suffix;
    const int q0 = pick(causal, rc_lo + (j - nd) * BQ, rd_lo + j * BQ);
    ld_left = pick(causal, rc_hi, rd_hi) - q0;
    move_to(rs_t, pick(qsuf, src_suf, src_pre) + ((uint64_t)q0 * a.h_q + hq) * (D * 2));
    move_to(rs_r, pick(qsuf, val_suf, val_pre) + ((uint64_t)hq * val_ld + q0) * 4);
  };
  auto copy_next = [&]() PG_INLINE {
    move_to(rs_t, (rs_t[0] | (uint64_t)rs_t[1] << 32) + (unsigned)(BQ * row_bytes));
    move_to(rs_r, (rs_r[0] | (uint64_t)rs_r[1] << 32) + 4 * BQ);
    ld_left = max(ld_left - BQ, 0);
    ++ld_j;
    if (__builtin_expect(ld_left == 0, 0)) {
      asm volatile("");
      if (ld_j == per_head) { ld_j = 0; ++ld_hd; }
      if (ld_hd < ratio) new_run(ld_hd, ld_j);
    }
    set_rows();
  };
  auto copy_part = [&](int k, int off) PG_INLINE {
    if (k < PW) dma16(rs_t, lds_tile + off + 2048 * k, voff[k]);
    else dma4(rs_r, lds_row + off, 4 * lane);
  };
  if (it0 < it1) {
    new_run(ld_hd, ld_j);
    set_rows();
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      if (b > 0) copy_next();
#pragma unroll
      for (int k = 0; k <= PW; ++k) copy_part(k, b * STAGE);
    }
  }
  FragOffsets<T, D> fo;
  fo.init(lane);
  __builtin_amdgcn_s_waitcnt(0);  // the compiler then knows that the K and V operands have landed
  __syncthreads();

  // The tile being worked on: its first row (kDenseRow + in the dense range, where no mask and no
  // skip applies) and the tiles left in its run.
  int q0 = first_j >= nd ? rc_lo + (first_j - nd) * BQ : kDenseRow;
  int run_left = first_j >= nd ? per_head - first_j : nd - first_j;
  int off = 0, off_p = 0;  // stage of this tile and of the one before
  Frag qf[KK];
  u32x4 dk[2][2] = {};  // dS of the tile before, as bf16 operand fragments [key block][16 rows]; zero if there is none
  int sg0 = 0, sg1 = 0;
  bool skip = false, full = true;
  auto seg_at = [&](int o, int row) PG_INLINE { return *(const int*)(stage + o + 2 * TILE + 512 + 4 * row); };
  auto last_row = [&]() PG_INLINE { return max(min(rc_hi - q0, BQ), 1) - 1; };
  auto visibility = [&]() PG_INLINE {
    skip = (q0 + BQ - 1 < wk0) | (uniform(sg0) > wk1) | !wave_active;
    full = (q0 >= wk1) & (uniform(sg1) <= wk0);
  };
  if (it0 < it1) {
#pragma unroll
    for (int kk = 0; kk < PF; ++kk) qf[kk] = fo.row(stage, 0, kk);
    sg0 = seg_at(0, 0);
    sg1 = seg_at(0, last_row());
    visibility();
  }

  // One step: S, P, dP, dV and dS of tile `it` (CUR) and dK of the tile before (PREV). The matrix
  // products are ordered S, dK of the tile before, dP, dV, so that each phase's vector work has its
  // inputs ready and runs beside other products: P beside dK and dP, dS beside dV, addresses beside S.
  // Operand fragments are read from LDS steps ahead of their products, and every step's order is
  // pinned: with one wave per SIMD nothing else hides a wait.
  auto step = [&](auto prev_, auto cur_) PG_INLINE {
    constexpr bool PREV = decltype(prev_)::value, CUR = decltype(cur_)::value;
    const char* Qt = stage + off;
    const char* Gt = Qt + TILE;
    const char* Qp = stage + off_p;
    const float* rv = (const float*)(Qt + 2 * TILE);
    const int off_n = off == (NBUF - 1) * STAGE ? 0 : off + STAGE;
    const int off_w = off_n == (NBUF - 1) * STAGE ? 0 : off_n + STAGE;
    const int off_c = off_w == (NBUF - 1) * STAGE ? 0 : off_w + STAGE;  // stage of tile it + 3 (and it - 1)
    const int q0_it = q0;
    auto advance = [&]() PG_INLINE {
      q0 += BQ;
      if (__builtin_expect(--run_left == 0, 0)) {
        asm volatile("");
        const bool to_causal = (q0 >= kDenseRow && nc > 0) || nd == 0;
        q0 = pick(to_causal, rc_lo, kDenseRow);
        run_left = pick(to_causal, nc, nd);
      }
    };
    f32x16 s[2], dp[2];
    u32x4 pk[2][2];
    f32x4 l4[4];
    Frag gf[KK], gt[2 * DB], qt[2 * DB], kl[KK];
    // Elements go in pairs, by rows: pair p -> row block i = p / 4, key block (p / 2) % 2, rows
    // 2 (p % 2) and + 1 of the block, so that a row block's values live briefly.
    auto q_tr = [&](auto k) PG_INLINE {
      constexpr int i = decltype(k)::value;
      if constexpr (i < 2 * DB) qt[i] = fo.tr(Qp, i / DB, i % DB);
    };
    auto g_tr = [&](auto k) PG_INLINE {
      constexpr int i = decltype(k)::value;
      if constexpr (i < 2 * DB) gt[i] = fo.tr(Gt, i / DB, i % DB);
    };
    auto l_row = [&](auto k) PG_INLINE {
      constexpr int i = decltype(k)::value;
      if constexpr (i < 4) l4[i] = *(const f32x4*)&rv[8 * i + 4 * hh];
    };
    auto d_row = [&](auto k) PG_INLINE {  // both key blocks' accumulators start at Dsum
      constexpr int i = decltype(k)::value % 4, kb = decltype(k)::value / 4;
      const f32x4 d = *(const f32x4*)&rv[64 + 8 * i + 4 * hh];
#pragma unroll
      for (int e = 0; e < 4; ++e) dp[kb][4 * i + e] = d[e];
    };
    auto p_pair = [&](auto k) PG_INLINE {
      constexpr int p = decltype(k)::value, i = p / 4, kb = p / 2 % 2, q = 2 * (p % 2), r = 4 * i + q;
      if constexpr (p % 4 == 0) l_row(Int<i + 1>{});
      s[kb][r] = fast_exp2(fmaf(s[kb][r], c, -l4[i][q]));
      s[kb][r + 1] = fast_exp2(fmaf(s[kb][r + 1], c, -l4[i][q + 1]));
      pk[kb][r / 8][r % 8 / 2] = pack_bf16(s[kb][r], s[kb][r + 1]);
    };
    auto d_pair = [&](auto k) PG_INLINE {
      constexpr int p = decltype(k)::value, i = p / 4, kb = p / 2 % 2, q = 2 * (p % 2), r = 4 * i + q;
      dk[kb][r / 8][r % 8 / 2] = pack_bf16(s[kb][r] * dp[kb][r], s[kb][r + 1] * dp[kb][r + 1]);
    };
    if constexpr (CUR) {
      s[0] = f32x16{}; s[1] = f32x16{};
      static_for<2 * KK>([&](auto x_) PG_INLINE {
        constexpr int x = decltype(x_)::value, kk = x / 2;
        if constexpr (x % 2 == 0) {
          if constexpr (kk + PF < KK) qf[kk + PF] = fo.row(Qt, 0, kk + PF);
          if constexpr (PREV && kk >= KK - AHEAD) q_tr(Int<kk - (KK - AHEAD)>{});
          if constexpr (kk == KK - 1) l_row(Int<0>{});
        }
        if constexpr (x % 2 == 0 && kk + 3 >= KK - KL && kk + 3 < KK) kl[kk + 3] = s_k[wave][kk + 3 - (KK - KL)][lane];
        s[x % 2] = E::mma(qf[kk], x % 2 == 1 && kk >= KK - KL ? kl[kk] : kf[x % 2][kk], s[x % 2]);
        if constexpr (x == 1) advance();
        if constexpr (x == 5) copy_next();
        __builtin_amdgcn_sched_barrier(0);
      });
    } else {
      advance();
      copy_next();
      if constexpr (PREV) static_for<AHEAD>([&](auto k) PG_INLINE { q_tr(k); });
    }
    // dK^T += Q^T dS of the tile before; beside it the first half of P = exp2(S c - lse)
    if constexpr (PREV) {
      static_for<4 * DB>([&](auto x_) PG_INLINE {
        constexpr int x = decltype(x_)::value, I = x / 2, t = I / DB, db = I % DB;
        if constexpr (x % 2 == 0) {
          q_tr(Int<I + AHEAD>{});
          if constexpr (CUR && I >= 2 * DB - PF) gf[I - (2 * DB - PF)] = fo.row(Gt, 0, I - (2 * DB - PF));
        }
        if constexpr (CUR && x >= 4 * DB - DR)
          static_for<8 / DR>([&](auto y) PG_INLINE { d_row(Int<(x - (4 * DB - DR)) * (8 / DR) + decltype(y)::value>{}); });
        mma_acc<16 * (DB * (2 + x % 2) + db), db == 0>(qt[I], __builtin_bit_cast(Frag, dk[x % 2][t]));
        if constexpr (CUR) {
          constexpr int p0 = 8 * x / (4 * DB), p1 = 8 * (x + 1) / (4 * DB);
          static_for<p1 - p0>([&](auto y) PG_INLINE { p_pair(Int<p0 + decltype(y)::value>{}); });
        }
        __builtin_amdgcn_sched_barrier(0);
      });
    }
    // publishes tile it + 1 (the copies of tile it + 2 may still be on their way) and frees the
    // buffer of tile it - 1, which the copies of tile it + 3 then fill
    wait_vm<PW + 1>();
    block_meet();
    if constexpr (CUR) {
      // dP = dO V^T; beside it the other half of P, and the copies
      static_for<2 * KK>([&](auto x_) PG_INLINE {
        constexpr int x = decltype(x_)::value, kk = x / 2;
        if constexpr (x % 2 == 0) {
          if constexpr (kk + PF < KK) gf[kk + PF] = fo.row(Gt, 0, kk + PF);
          if constexpr (kk >= KK - AHEAD) g_tr(Int<kk - (KK - AHEAD)>{});
        }
        dp[x % 2] = E::mma(gf[kk], vf[x % 2][kk], dp[x % 2]);
        constexpr int p0 = 8 + 8 * x / (2 * KK), p1 = 8 + 8 * (x + 1) / (2 * KK);
        static_for<p1 - p0>([&](auto y) PG_INLINE { p_pair(Int<p0 + decltype(y)::value>{}); });
        if constexpr (p1 == p0 && x / 2 <= PW) copy_part(x / 2, off_c);
        __builtin_amdgcn_sched_barrier(0);
      });
      if constexpr (KK < 8) static_for<PW + 1>([&](auto k) PG_INLINE { copy_part(decltype(k)::value, off_c); });
      // Boundary tile: P = 0 for pairs that do not see each other, after the exponential as in dkdv_kernel:
      // nothing of a row (its log-sum-exp may be NaN) reaches the dV of keys it does not see.
      if (__builtin_expect(!full, 0)) {
        asm volatile("");
        const int* sg = (const int*)rv + 128;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int4 g4 = *(const int4*)&sg[8 * i + 4 * hh];
          const int gs[4] = {g4.x, g4.y, g4.z, g4.w};
#pragma unroll
          for (int kb = 0; kb < 2; ++kb) {
            const int lim = key_c[kb] - (q0_it + 4 * hh) - 8 * i;
#pragma unroll
            for (int e = 0; e < 4; e += 2) {
              const int r = 4 * i + e;
              s[kb][r] = ((e >= lim) & (key_c[kb] >= gs[e])) ? s[kb][r] : 0.f;
              s[kb][r + 1] = ((e + 1 >= lim) & (key_c[kb] >= gs[e + 1])) ? s[kb][r + 1] : 0.f;
              pk[kb][r / 8][r % 8 / 2] = pack_bf16(s[kb][r], s[kb][r + 1]);
            }
          }
          __builtin_amdgcn_sched_barrier(0);  // one row block's values at a time: registers are all in use
        }
      }
      // dV^T += dO^T P; beside it -dS = P (Dsum - dP), and the first operands of the next tile
      static_for<4 * DB>([&](auto x_) PG_INLINE {
        constexpr int x = decltype(x_)::value, I = x / 2, t = I / DB, db = I % DB;
        if constexpr (x % 2 == 0) {
          g_tr(Int<I + AHEAD>{});
          if constexpr (I == 0) { sg0 = seg_at(off_n, 0); sg1 = seg_at(off_n, last_row()); }
          if constexpr (I >= 2 * DB - PF) qf[I - (2 * DB - PF)] = fo.row(stage + off_n, 0, I - (2 * DB - PF));
        }
        mma_acc<16 * (DB * (x % 2) + db), db == 0>(gt[I], __builtin_bit_cast(Frag, pk[x % 2][t]));
        constexpr int p0 = 16 * x / (4 * DB), p1 = 16 * (x + 1) / (4 * DB);
        static_for<p1 - p0>([&](auto y) PG_INLINE { d_pair(Int<p0 + decltype(y)::value>{}); });
        if constexpr (I == 2 * DB - 1 && x % 2 == 0) visibility();
        __builtin_amdgcn_sched_barrier(0);
      });
    } else {
#pragma unroll
      for (int k = 0; k <= PW; ++k) copy_part(k, off_c);
#pragma unroll
      for (int kk = 0; kk < PF; ++kk) qf[kk] = fo.row(stage + off_n, 0, kk);
      sg0 = seg_at(off_n, 0);
      sg1 = seg_at(off_n, last_row());
      visibility();
    }
    if constexpr (CUR) {
      off_p = off;
    } else {
      // the next tile worked on has no dS before it: a zero one, against its own Q rows
#pragma unroll
      for (int k = 0; k < 4; ++k) dk[k >> 1][k & 1] = u32x4{0, 0, 0, 0};
      off_p = off_n;
    }
    off = off_n;
  };
  bool prev = false;
  for (int it = it0; it < it1; ++it) {
    const bool cur = !skip;
    if (__builtin_expect(cur, 1)) step(std::true_type{}, std::true_type{});
    else if (prev) step(std::true_type{}, std::false_type{});
    else step(std::false_type{}, std::false_type{});
    prev = cur;
  }
  if (prev) {  // dK of the last tile
    static_for<2 * DB>([&](auto i) PG_INLINE {
      constexpr int I = decltype(i)::value, t = I / DB, db = I % DB;
      const Frag q = fo.tr(stage + off_p, t, db);
      mma_acc<16 * (2 * DB + db), true>(q, __builtin_bit_cast(Frag, dk[0][t]));
      mma_acc<16 * (3 * DB + db), true>(q, __builtin_bit_cast(Frag, dk[1][t]));
    });
  }
  wait_vm<0>();  // no copy may land after the workgroup's LDS is given back
  acc_settle();
  if (!wave_active) return;
  static_for<4>([&](auto bw) {
    constexpr int kb = decltype(bw)::value & 1, w = decltype(bw)::value >> 1;  // w 0: dV, 1: dK
    if (!kvalid[kb]) return;
    const int key = wk0 + 32 * kb + n;
    const float sc = w ? -a.scale : 1.f;  // dS was formed negated
    float* part = a.part + (((size_t)td.chunk * 2 + 1 - w) * a.total_prefix + key) * a.h_kv * D + (size_t)kvh * D;
    T* out = (T*)(w ? (kv_suffix ? a.dk_suf : a.dk_pre) : (kv_suffix ? a.dv_suf : a.dv_pre)) +
             ((size_t)(key + xk) * a.h_kv + kvh) * D;
    static_for<DB * 4>([&](auto q) {
      constexpr int db = decltype(q)::value / 4, i = decltype(q)::value % 4;
      constexpr int R = 16 * ((2 * w + kb) * DB + db) + 4 * i;
      const int d0 = 32 * db + 8 * i + 4 * hh;
      const f32x4 x = f32x4{acc_read<R>() * sc, acc_read<R + 1>() * sc, acc_read<R + 2>() * sc, acc_read<R + 3>() * sc};
      if (td.nchunks > 1) *(f32x4*)(part + d0) = x;
      else E::store4(out + d0, x[0], x[1], x[2], x[3]);
    });
  });
}


// ------------------------------------------------------------------ dQ (query-stationary)
// Per 32-key tile and wave: S^T = K Q^T and dP^T = V dO^T (keys x 64 queries), dQ^T += K^T dS^T. Q and dO
// stay in AGPRs beside the accumulators, which leaves the VGPRs to two tiles' P and dP: the matrix
// products of a tile then run beside the vector work of the one before. One wave per SIMD is bound by
// the instructions it issues (about 4.5 clocks each), so dP's accumulator starts at -Dsum instead of
// subtracting it per element (that alone 146.5 -> 142.4 ms on the case below), and P and dP alternate
// between two sets of registers in a loop unrolled by two, so that nothing is copied.
// Measured on 8 groups x 16 members, P 1246..26888, 64/8 heads: 154.2 -> 142.4 ms (1274 TFLOP/s of its three
// products; matrix cores 64% busy at 1.91 GHz, before 66% at 1.73); 1 x 16, P 16384, 32/8: 4.66 -> 4.42 ms.
template <int D>
__global__ void __launch_bounds__(kWideThreads, 1) dq_wide_kernel(const BwdArgs a) {
  using T = bf16;
  using E = Elt<bf16>;
  using Frag = E::Frag;
  using Copies = KvCopies<D>;
  constexpr int BN = kWideBK;
  constexpr int KK = D / 16, DB = D / 32;
  constexpr int NBUF = 4;
  static_assert(D == 128, "the library runs head_dim 64 on dq_kernel (use_wide_q)");
  constexpr int PF = 3;                 // row fragments read ahead of their products
  constexpr int AHEAD = 3;              // transposed fragments read ahead
  // AGPRs: dQ^T blocks (qb, db) from a0, then the B operands Q and dO
  constexpr int RQ = 32 * DB, RG = RQ + 8 * KK;
  constexpr int PB = 5;                 // pairs of P beside dQ, the rest beside dP
  constexpr int TILE = Copies::TILE, STAGE = Copies::STAGE, PW = Copies::PW;
  __shared__ __attribute__((aligned(1024))) char stage[NBUF * STAGE];

  const BlockSlot slot = xcd_slot(blockIdx.x, a.h_q, a.h_q / a.h_kv);
  const int rank = uniform(slot.unit), head = uniform(slot.head);
  if (rank >= a.hdr->n_qtiles) return;
  const TileDesc* tp = a.qtiles + uniform(a.qorder[rank]);
  const GroupInfoEx* gp = a.ginfo + uniform(tp->group);
  const int row0 = uniform(tp->row0), row1 = uniform(tp->row1), aux = uniform(tp->aux);
  const bool suffix = uniform(tp->kind) == 1;
  const int g_p0 = uniform(gp->p0), g_p1 = uniform(gp->p1), g_s0 = uniform(gp->s0);
  const int kvh = uniform(head / (a.h_q / a.h_kv));
  const int rows_all = a.total_prefix + a.total_suffix;
  const int xo_pre = a.xl ? g_s0 : 0, xo_suf = a.xl ? g_p1 : 0;
  const int xq = suffix ? xo_suf : xo_pre;

  const int tid = threadIdx.x, wave = uniform(tid >> 6), lane = tid & 63;
  const int n = lane & 31, hh = lane >> 5;
  const int wq0 = row0 + 64 * wave;
  const bool wave_active = wq0 < row1;
  const int wq1 = min(wq0 + 64, row1) - 1;

  const int kA0 = g_p0, kA1 = suffix ? g_p1 : row1;
  const int kB0 = suffix ? aux : 0, kB1 = suffix ? row1 : 0;
  const int nA = (kA1 - kA0 + BN - 1) / BN, nB = (kB1 - kB0 + BN - 1) / BN;
  const int ntiles = nA + nB;
  const int kvstride = a.h_kv * D;
  Copies cp;
  {
    const T* p = (const T*)(wave < 2 ? a.k_pre : a.v_pre) + (size_t)(kA0 + xo_pre) * kvstride + kvh * D;
    const T* q = (const T*)(wave < 2 ? a.k_suf : a.v_suf) + (size_t)(kB0 + xo_suf) * kvstride + kvh * D;
    cp.init(stage, p, kA1 - kA0, q, kB1 - kB0, kvstride, wave, lane);
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      if (b > 0) cp.next();
#pragma unroll
      for (int k = 0; k < PW; ++k) cp.part(k, b * STAGE);
    }
  }

  int qrow_c[2], seg_q[2];
  bool qvalid[2];
  float lse2[2];
  f32x16 ndsum[2];  // -Dsum of the lane's query in every register: what dP starts at
  static_for<32 * DB>([](auto r) { acc_zero<decltype(r)::value>(); });
  static_for<2>([&](auto b_) PG_INLINE {
    constexpr int qb = decltype(b_)::value;
    const int qrow = wq0 + 32 * qb + n;
    qvalid[qb] = qrow < row1;
    qrow_c[qb] = qvalid[qb] ? qrow : row1 - 1;
    const size_t off = ((size_t)(qrow_c[qb] + xq) * a.h_q + head) * D + 8 * hh;
    const T* Q = (const T*)(suffix ? a.q_suf : a.q_pre) + off;
    const T* G = (const T*)(suffix ? a.do_suf : a.do_pre) + off;
    const T* O = (const T*)(suffix ? a.o_suf : a.o_pre) + off;
    float part = 0.f;
    Frag qf[KK], gf[KK], of[KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      qf[kk] = E::global_row(Q + 16 * kk, qvalid[qb]);
      gf[kk] = E::global_row(G + 16 * kk, qvalid[qb]);
      of[kk] = E::global_row(O + 16 * kk, qvalid[qb]);
    }
    static_for<KK>([&](auto k) PG_INLINE {
      constexpr int kk = decltype(k)::value;
      acc_put_frag<RQ + 4 * (KK * qb + kk)>(qf[kk]);
      acc_put_frag<RG + 4 * (KK * qb + kk)>(gf[kk]);
#pragma unroll
      for (int e = 0; e < 8; ++e) part = fmaf(E::frag_elem(of[kk], e), E::frag_elem(gf[kk], e), part);
    });
    const float* L = suffix ? a.lse_suf : a.lse_pre;
    const int ld = a.xl ? rows_all : (suffix ? a.total_suffix : a.total_prefix);
    lse2[qb] = L[(size_t)head * ld + qrow_c[qb] + xq] * kLog2e;
    const float dsum = wave_swap32_sum(part);
#pragma unroll
    for (int r = 0; r < 16; ++r) ndsum[qb][r] = -dsum;
    if (qvalid[qb] && hh == 0) {  // for the dK/dV kernel
      const size_t at = (size_t)head * rows_all + (suffix ? a.total_prefix : 0) + qrow;
      a.dsum[at] = dsum;
      if (a.lse2) a.lse2[at] = lse2[qb];
    }
    seg_q[qb] = suffix ? a.seg_start[qrow_c[qb]] : 0;
  });
  const int seg_lo = uniform((suffix && wave_active) ? a.seg_start[wq0] : 0);
  const int seg_hi = uniform((suffix && wave_active) ? a.seg_start[wq1] : 0);
  const float c = a.scale_log2;
  FragOffsets<T, D> fo;
  fo.init(lane);
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();

  // the tile being worked on: its first key, the end of its run, and whether it is of the first run
  int k0 = nA > 0 ? kA0 : kB0, kend = nA > 0 ? kA1 : kB1;
  bool seg_a = nA > 0;
  int off = 0, off_p = 0;
  bool skip = false, full = true;
  auto visibility = [&]() PG_INLINE {
    const bool cross = seg_a & suffix;  // response rows x prefix keys: no causal limit
    skip = !wave_active | (!cross & (k0 > wq1)) | (!seg_a & (k0 + BN <= seg_lo));
    full = (k0 + BN <= kend) & (cross | (k0 + BN - 1 <= wq0)) & (seg_a | (k0 >= seg_hi));
  };
  visibility();
  Frag kr[KK];
#pragma unroll
  for (int kk = 0; kk < PF; ++kk) kr[kk] = fo.row(stage, 0, kk);
  // P and dP - Dsum of this tile and of the one before (they alternate)
  f32x16 sb[2][2] = {}, db_[2][2] = {};

  // One step: S of tile j beside dS of the tile before, dQ of the tile before beside P of tile j, and
  // dP of tile j beside the rest of P.
  auto step = [&](auto b_, auto prev_, auto cur_) PG_INLINE {
    constexpr bool PREV = decltype(prev_)::value, CUR = decltype(cur_)::value;
    f32x16(&s)[2] = sb[decltype(b_)::value];
    f32x16(&p_prev)[2] = sb[1 - decltype(b_)::value];
    f32x16(&dp)[2] = db_[decltype(b_)::value];
    f32x16(&dp_prev)[2] = db_[1 - decltype(b_)::value];
    const char* Kt = stage + off;
    const char* Vt = Kt + TILE;
    const char* Kp = stage + off_p;
    const int off_n = off == (NBUF - 1) * STAGE ? 0 : off + STAGE;
    const int off_w = off_n == (NBUF - 1) * STAGE ? 0 : off_n + STAGE;
    const int off_c = off_w == (NBUF - 1) * STAGE ? 0 : off_w + STAGE;
    const int k0_it = k0, kend_it = kend;
    const bool seg_it = seg_a;
    auto advance = [&]() PG_INLINE {
      k0 += BN;
      if (__builtin_expect(k0 >= kend, 0)) {
        asm volatile("");
        k0 = kB0;
        kend = kB1;
        seg_a = false;
      }
    };
    u32x4 ds[2][2];
    Frag vr[KK], kt[2 * DB];
    auto k_tr = [&](auto k) PG_INLINE {
      constexpr int i = decltype(k)::value;
      if constexpr (i < 2 * DB) kt[i] = fo.tr(Kp, i / DB, i % DB);
    };
    auto p_pair = [&](auto k) PG_INLINE {
      constexpr int p = decltype(k)::value, i = p / 4, qb = p / 2 % 2, r = 4 * i + 2 * (p % 2);
      s[qb][r] = fast_exp2(fmaf(s[qb][r], c, -lse2[qb]));
      s[qb][r + 1] = fast_exp2(fmaf(s[qb][r + 1], c, -lse2[qb]));
    };
    auto d_pair = [&](auto k) PG_INLINE {
      constexpr int p = decltype(k)::value, i = p / 4, qb = p / 2 % 2, r = 4 * i + 2 * (p % 2);
      ds[qb][r / 8][r % 8 / 2] = pack_bf16(p_prev[qb][r] * dp_prev[qb][r], p_prev[qb][r + 1] * dp_prev[qb][r + 1]);
    };
    if constexpr (CUR) {
      static_for<2 * KK>([&](auto x_) PG_INLINE {
        constexpr int x = decltype(x_)::value, kk = x / 2;
        if constexpr (x % 2 == 0) {
          if constexpr (kk + PF < KK) kr[kk + PF] = fo.row(Kt, 0, kk + PF);
          if constexpr (kk >= KK - AHEAD) k_tr(Int<kk - (KK - AHEAD)>{});
        }
        mma_v<RQ + 4 * (KK * (x % 2) + kk), kk == 0>(s[x % 2], kr[kk]);
        if constexpr (x == 1) advance();
        if constexpr (x == 3) cp.next();
        constexpr int p0 = x < 2 ? 0 : 8 * (x - 2) / (2 * KK - 2), p1 = x < 2 ? 0 : 8 * (x - 1) / (2 * KK - 2);
        static_for<p1 - p0>([&](auto y) PG_INLINE { d_pair(Int<p0 + decltype(y)::value>{}); });
        __builtin_amdgcn_sched_barrier(0);
      });
      if (__builtin_expect(!full, 0)) {
        settle(s[0], s[1]);
        const int base = k0_it + 4 * hh;
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
          int hi = kend_it - base;
          if (!(seg_it & suffix)) hi = min(hi, qrow_c[qb] + 1 - base);
          const int lo = seg_it ? -(1 << 30) : seg_q[qb] - base;
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int o = 8 * (r >> 2) + (r & 3);
            s[qb][r] = ((o >= lo) & (o < hi)) ? s[qb][r] : -INFINITY;
          }
        }
      }
    } else {
      advance();
      cp.next();
      if constexpr (PREV) {
        static_for<AHEAD>([&](auto k) PG_INLINE { k_tr(k); });
        settle(dp_prev[0], dp_prev[1]);
        static_for<16>([&](auto k) PG_INLINE { d_pair(k); });
      }
    }
    if constexpr (PREV) {
      // dQ^T += K^T dS of the tile before
      static_for<4 * DB>([&](auto x_) PG_INLINE {
        constexpr int x = decltype(x_)::value, I = x / 2, t = I / DB, db = I % DB;
        if constexpr (x % 2 == 0) {
          k_tr(Int<I + AHEAD>{});
          if constexpr (CUR && I >= 2 * DB - PF) vr[I - (2 * DB - PF)] = fo.row(Vt, 0, I - (2 * DB - PF));
        }
        mma_acc<16 * (DB * (x % 2) + db), db == 0>(kt[I], __builtin_bit_cast(Frag, ds[x % 2][t]));
        if constexpr (CUR && t == 0) {
          constexpr int p0 = 8 + 8 * x / (2 * DB), p1 = 8 + 8 * (x + 1) / (2 * DB);
          static_for<p1 - p0>([&](auto y) PG_INLINE { d_pair(Int<p0 + decltype(y)::value>{}); });
        } else if constexpr (CUR) {
          constexpr int p0 = PB * (x - 2 * DB) / (2 * DB), p1 = PB * (x - 2 * DB + 1) / (2 * DB);
          static_for<p1 - p0>([&](auto y) PG_INLINE { p_pair(Int<p0 + decltype(y)::value>{}); });
        }
        __builtin_amdgcn_sched_barrier(0);
      });
    }
    // publishes tile j + 1 and frees the stage of tile j - 1 for the copies of tile j + 3
    wait_vm<PW>();
    block_meet();
    if constexpr (CUR) {
      static_for<2 * KK>([&](auto x_) PG_INLINE {
        constexpr int x = decltype(x_)::value, kk = x / 2;
        if constexpr (x % 2 == 0) {
          if constexpr (kk + PF < KK) vr[kk + PF] = fo.row(Vt, 0, kk + PF);
          if constexpr (kk >= KK - PF) kr[kk - (KK - PF)] = fo.row(stage + off_n, 0, kk - (KK - PF));
        }
        if constexpr (kk == 0) mma_v_from<RG + 4 * KK * (x % 2)>(dp[x % 2], vr[0], ndsum[x % 2]);
        else mma_v<RG + 4 * (KK * (x % 2) + kk), false>(dp[x % 2], vr[kk]);
        constexpr int p0 = PB + (16 - PB) * x / (2 * KK), p1 = PB + (16 - PB) * (x + 1) / (2 * KK);
        static_for<p1 - p0>([&](auto y) PG_INLINE { p_pair(Int<p0 + decltype(y)::value>{}); });
        if constexpr (x % 2 == 0 && kk < PW) cp.part(kk, off_c);
        if constexpr (x == 2 * KK - 2) visibility();
        __builtin_amdgcn_sched_barrier(0);
      });
      static_assert(PW <= KK, "every copy has its step");
      off_p = off;
    } else {
#pragma unroll
      for (int k = 0; k < PW; ++k) cp.part(k, off_c);
#pragma unroll
      for (int kk = 0; kk < PF; ++kk) kr[kk] = fo.row(stage + off_n, 0, kk);
      visibility();
      // the next tile worked on has no tile before it: P = 0 gives dS = 0, against its own K rows
      s[0] = f32x16{}; s[1] = f32x16{};
      dp[0] = f32x16{}; dp[1] = f32x16{};
      off_p = off_n;
    }
    off = off_n;
  };
  bool prev = false;
  auto visit = [&](auto b_) PG_INLINE {
    const bool cur = !skip;
    if (__builtin_expect(cur, 1)) step(b_, std::true_type{}, std::true_type{});
    else if (prev) step(b_, std::true_type{}, std::false_type{});
    else step(b_, std::false_type{}, std::false_type{});
    prev = cur;
  };
  for (int j = 0; j < ntiles; j += 2) {
    visit(Int<0>{});
    if (j + 1 < ntiles) visit(Int<1>{});
  }
  if (prev) {  // dS and dQ of the last tile
    settle(db_[0][0], db_[0][1]);
    settle(db_[1][0], db_[1][1]);
    f32x16 p_last[2] = {sb[0][0], sb[0][1]};
    if (ntiles % 2 == 0) { p_last[0] = sb[1][0]; p_last[1] = sb[1][1]; }
    f32x16 dp[2] = {db_[0][0], db_[0][1]};
    if (ntiles % 2 == 0) { dp[0] = db_[1][0]; dp[1] = db_[1][1]; }
    Frag dsf[2][2];
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
#pragma unroll
      for (int r = 0; r < 16; ++r) dp[qb][r] *= p_last[qb][r];
      dsf[qb][0] = E::acc_to_frag(dp[qb], 0);
      dsf[qb][1] = E::acc_to_frag(dp[qb], 1);
    }
    static_for<2 * DB>([&](auto i) PG_INLINE {
      constexpr int I = decltype(i)::value, t = I / DB, db = I % DB;
      const Frag k = fo.tr(stage + off_p, t, db);
      mma_acc<16 * db, true>(k, dsf[0][t]);
      mma_acc<16 * (DB + db), true>(k, dsf[1][t]);
    });
  }
  wait_vm<0>();  // no copy may land after the workgroup's LDS is given back
  acc_settle();
  if (!wave_active) return;
  static_for<2>([&](auto b) {
    constexpr int qb = decltype(b)::value;
    if (!qvalid[qb]) return;
    T* out = (T*)(suffix ? a.dq_suf : a.dq_pre) + ((size_t)(wq0 + 32 * qb + n + xq) * a.h_q + head) * D;
    static_for<DB * 4>([&](auto q) {
      constexpr int db = decltype(q)::value / 4, i = decltype(q)::value % 4;
      constexpr int R = 16 * (qb * DB + db) + 4 * i;
      const float sc = a.scale;
      E::store4(out + 32 * db + 8 * i + 4 * hh, acc_read<R>() * sc, acc_read<R + 1>() * sc, acc_read<R + 2>() * sc,
                acc_read<R + 3>() * sc);
    });
  });
}

}  // namespace pg

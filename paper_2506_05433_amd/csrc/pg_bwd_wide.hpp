// dK, dV of large bf16 problems (key-stationary, like dkdv_kernel): 256 keys per workgroup, 64 per
// wave, one wave per SIMD with all 512 registers.
//
// What bounds it: the chip's power. On N(0,1) data a loop of nothing but 32x32x16 products reaches
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
// its four products; matrix cores 63% busy at 1.81 GHz); 1 x 16, P 16384, 32/8: 7.35 -> 6.17 ms with the
// reduction; 1 x 8, P 4096, 32/8: 1.056 -> 0.909 ms; 4 x 16, P 8192, 32/8, d 64: 16.05 -> 13.89 ms.
// Measured and not kept: V (or more of K) in LDS instead of registers; S, dP, dV, dK each in turn with
// P beside dP and dS beside dV only (3% slower: the vector work does not fit those phases); two wait
// states before every product instead of before the first that reads new operands (2% slower).
#pragma once
#include <type_traits>

#include "pg_bwd.hpp"

namespace pg {

// Accumulators pinned in AGPRs. The products below name their accumulator registers themselves and
// declare every AGPR clobbered, so the compiler keeps nothing of its own there between them. R is
// the first of the 16 registers. The compiler knows neither that these are matrix instructions nor
// their hazards: FRESH puts the two wait states a vector write of an operand needs before the first
// product that reads it (later ones are further away), and acc_settle() comes before the first
// acc_read(). tests/test_wide_codegen.py checks both rules in the generated code.
#define PG_ALL_AGPRS "a0", "a1", "a2", "a3", "a4", "a5", "a6", "a7", "a8", "a9", "a10", "a11", "a12", "a13", "a14", "a15", "a16", "a17", "a18", "a19", "a20", "a21", "a22", "a23", "a24", "a25", "a26", "a27", "a28", "a29", "a30", "a31", "a32", "a33", "a34", "a35", "a36", "a37", "a38", "a39", "a40", "a41", "a42", "a43", "a44", "a45", "a46", "a47", "a48", "a49", "a50", "a51", "a52", "a53", "a54", "a55", "a56", "a57", "a58", "a59", "a60", "a61", "a62", "a63", "a64", "a65", "a66", "a67", "a68", "a69", "a70", "a71", "a72", "a73", "a74", "a75", "a76", "a77", "a78", "a79", "a80", "a81", "a82", "a83", "a84", "a85", "a86", "a87", "a88", "a89", "a90", "a91", "a92", "a93", "a94", "a95", "a96", "a97", "a98", "a99", "a100", "a101", "a102", "a103", "a104", "a105", "a106", "a107", "a108", "a109", "a110", "a111", "a112", "a113", "a114", "a115", "a116", "a117", "a118", "a119", "a120", "a121", "a122", "a123", "a124", "a125", "a126", "a127", "a128", "a129", "a130", "a131", "a132", "a133", "a134", "a135", "a136", "a137", "a138", "a139", "a140", "a141", "a142", "a143", "a144", "a145", "a146", "a147", "a148", "a149", "a150", "a151", "a152", "a153", "a154", "a155", "a156", "a157", "a158", "a159", "a160", "a161", "a162", "a163", "a164", "a165", "a166", "a167", "a168", "a169", "a170", "a171", "a172", "a173", "a174", "a175", "a176", "a177", "a178", "a179", "a180", "a181", "a182", "a183", "a184", "a185", "a186", "a187", "a188", "a189", "a190", "a191", "a192", "a193", "a194", "a195", "a196", "a197", "a198", "a199", "a200", "a201", "a202", "a203", "a204", "a205", "a206", "a207", "a208", "a209", "a210", "a211", "a212", "a213", "a214", "a215", "a216", "a217", "a218", "a219", "a220", "a221", "a222", "a223", "a224", "a225", "a226", "a227", "a228", "a229", "a230", "a231", "a232", "a233", "a234", "a235", "a236", "a237", "a238", "a239", "a240", "a241", "a242", "a243", "a244", "a245", "a246", "a247", "a248", "a249", "a250", "a251", "a252", "a253", "a254", "a255"
template <int R, bool FRESH>
__device__ __forceinline__ void mma_acc(const bf16x8& a, const bf16x8& b) {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (FRESH)
    asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 a[%0:%1], %2, %3, a[%0:%1]" ::"n"(R), "n"(R + 15), "v"(a), "v"(b)
                 : PG_ALL_AGPRS);
  else
    asm volatile("v_mfma_f32_32x32x16_bf16 a[%0:%1], %2, %3, a[%0:%1]" ::"n"(R), "n"(R + 15), "v"(a), "v"(b)
                 : PG_ALL_AGPRS);
#endif
}
template <int R>
__device__ __forceinline__ void acc_zero() {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("v_accvgpr_write_b32 a[%0], 0" ::"n"(R) : PG_ALL_AGPRS);
#endif
}
template <int R>
__device__ __forceinline__ float acc_read() {
  float v = 0.f;
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("v_accvgpr_read_b32 %0, a[%1]" : "=v"(v) : "n"(R));
#endif
  return v;
}
__device__ __forceinline__ void acc_settle() {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_nop 15\n\ts_nop 15" ::: PG_ALL_AGPRS);
#endif
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (N > 0) {
    static_for<N - 1>(f);
    f(std::integral_constant<int, N - 1>{});
  }
}

#define PG_INLINE __attribute__((always_inline))

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// 16 (or 4) bytes per lane from a buffer into LDS at byte `lds` + 16 (4) * lane, issued in asm so
// that the compiler does not make every later LDS read wait for it: the caller waits (wait_vm)
// and meets a barrier before anybody reads the bytes.
__device__ __forceinline__ void dma16(u32x4 rs, unsigned lds, int voff) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds), "v"(voff), "s"(rs) : "memory");
#endif
}
__device__ __forceinline__ void dma4(u32x4 rs, unsigned lds, int voff) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds" ::"s"(lds), "v"(voff), "s"(rs) : "memory");
#endif
}
__device__ __forceinline__ void block_meet() {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_barrier" ::: "memory");
#endif
}
template <int N>
__device__ __forceinline__ void wait_vm() {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
#endif
}
__device__ __forceinline__ u32x4 make_rsrc(const void* p, int bytes) {
  const uint64_t a = (uint64_t)p;
  u32x4 r;
  r[0] = uniform((int)(unsigned)a);
  r[1] = uniform((int)(unsigned)(a >> 32)) & 0xffff;
  r[2] = uniform(bytes);
  r[3] = 0x00020000;
  return r;
}
__device__ __forceinline__ unsigned lds_addr(const void* p) {
  return (unsigned)(uintptr_t)(__attribute__((address_space(3))) const char*)p;
}

// Two floats rounded to bf16, kept where the call stands: left to itself the compiler gathers the
// conversions of a phase at its end, where no matrix instruction is in flight to hide them.
__device__ __forceinline__ unsigned pack_bf16(float x, float y) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const bf16x2 v = {(bf16)x, (bf16)y};
  unsigned u = __builtin_bit_cast(unsigned, v);
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(u));
#endif
  return u;
}

// cond ? a : b on values: on captured variables the operator selects between their addresses, which
// keeps the whole closure in memory
template <typename V>
__device__ __forceinline__ V pick(bool cond, V a, V b) { return cond ? a : b; }

constexpr int kWideThreads = 256;
constexpr int kWideKeys = 64;                    // keys per wave
constexpr int kWideBN = 4 * kWideKeys;           // keys per workgroup
constexpr int kWideBQ = 32;                      // query rows per staged tile

template <int N>
using Int = std::integral_constant<int, N>;
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
      if (__builtin_expect(!full, 0)) {
        asm volatile("");
        const int* sg = (const int*)rv + 128;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
          const int lim = key_c[kb] - (q0_it + 4 * hh);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int4 g4 = *(const int4*)&sg[8 * i + 4 * hh];
            const int gs[4] = {g4.x, g4.y, g4.z, g4.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const bool ok = (8 * i + e >= lim) & (key_c[kb] >= gs[e]);
              s[kb][4 * i + e] = ok ? s[kb][4 * i + e] : -INFINITY;
            }
          }
        }
      }
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
      // dV^T += dO^T P; beside it dS = P (dP - Dsum), and the first operands of the next tile
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

}  // namespace pg

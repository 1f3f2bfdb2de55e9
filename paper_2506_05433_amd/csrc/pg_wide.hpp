// Building blocks of the kernels that run one wave per SIMD with all 512 registers (pg_bwd_wide.hpp): matrix
// products on pinned AGPRs, LDS copies that the compiler does not wait for.
#pragma once
#include <type_traits>

#include "pg_common.hpp"

namespace pg {

constexpr int kWideThreads = 256;

// Accumulators (and, in the query-stationary kernels, B operands) pinned in AGPRs. The products below
// name those registers themselves and declare every AGPR clobbered, so the compiler keeps nothing of
// its own there between them. R is the first register. The compiler knows neither that these are
// matrix instructions nor their hazards, so: FRESH puts the two wait states a vector write of an
// operand needs before the first product that reads it (later ones are further away); acc_settle()
// comes before the first acc_read(); and a result that a product leaves in VGPRs (mma_v) is read by
// vector code only after two further products or after settle(). tests/test_wide_codegen.py checks
// on every path of the generated code that the operands and VGPR results keep their wait states.
#define PG_AGPRS "a0", "a1", "a2", "a3", "a4", "a5", "a6", "a7", "a8", "a9", "a10", "a11", "a12", "a13", "a14", "a15", "a16", "a17", "a18", "a19", "a20", "a21", "a22", "a23", "a24", "a25", "a26", "a27", "a28", "a29", "a30", "a31", "a32", "a33", "a34", "a35", "a36", "a37", "a38", "a39", "a40", "a41", "a42", "a43", "a44", "a45", "a46", "a47", "a48", "a49", "a50", "a51", "a52", "a53", "a54", "a55", "a56", "a57", "a58", "a59", "a60", "a61", "a62", "a63", "a64", "a65", "a66", "a67", "a68", "a69", "a70", "a71", "a72", "a73", "a74", "a75", "a76", "a77", "a78", "a79", "a80", "a81", "a82", "a83", "a84", "a85", "a86", "a87", "a88", "a89", "a90", "a91", "a92", "a93", "a94", "a95", "a96", "a97", "a98", "a99", "a100", "a101", "a102", "a103", "a104", "a105", "a106", "a107", "a108", "a109", "a110", "a111", "a112", "a113", "a114", "a115", "a116", "a117", "a118", "a119", "a120", "a121", "a122", "a123", "a124", "a125", "a126", "a127", "a128", "a129", "a130", "a131", "a132", "a133", "a134", "a135", "a136", "a137", "a138", "a139", "a140", "a141", "a142", "a143", "a144", "a145", "a146", "a147", "a148", "a149", "a150", "a151", "a152", "a153", "a154", "a155", "a156", "a157", "a158", "a159", "a160", "a161", "a162", "a163", "a164", "a165", "a166", "a167", "a168", "a169", "a170", "a171", "a172", "a173", "a174", "a175", "a176", "a177", "a178", "a179", "a180", "a181", "a182", "a183", "a184", "a185", "a186", "a187", "a188", "a189", "a190", "a191", "a192", "a193", "a194", "a195", "a196", "a197", "a198", "a199", "a200", "a201", "a202", "a203", "a204", "a205", "a206", "a207", "a208", "a209", "a210", "a211", "a212", "a213", "a214", "a215", "a216", "a217", "a218", "a219", "a220", "a221", "a222", "a223", "a224", "a225", "a226", "a227", "a228", "a229", "a230", "a231", "a232", "a233", "a234", "a235", "a236", "a237", "a238", "a239", "a240", "a241", "a242", "a243", "a244", "a245", "a246", "a247", "a248", "a249", "a250", "a251", "a252", "a253", "a254", "a255"
template <int R, bool FRESH>
__device__ __forceinline__ void mma_acc(const bf16x8& a, const bf16x8& b) {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (FRESH)
    asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 a[%0:%1], %2, %3, a[%0:%1]" ::"n"(R), "n"(R + 15), "v"(a), "v"(b)
                 : PG_AGPRS);
  else
    asm volatile("v_mfma_f32_32x32x16_bf16 a[%0:%1], %2, %3, a[%0:%1]" ::"n"(R), "n"(R + 15), "v"(a), "v"(b)
                 : PG_AGPRS);
#endif
}
// d = a B (FIRST) or d += a B, with B in AGPRs R .. R + 3 and d in VGPRs. d is tied to its registers
// also where its old value is dead: loop-carried results then need no copies.
template <int R, bool FIRST>
__device__ __forceinline__ void mma_v(f32x16& d, const bf16x8& a) {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (FIRST)
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, a[%2:%3], 0" : "+v"(d) : "v"(a), "n"(R), "n"(R + 3));
  else
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, a[%2:%3], %0" : "+v"(d) : "v"(a), "n"(R), "n"(R + 3));
#endif
}
// d = a B + c
template <int R>
__device__ __forceinline__ void mma_v_from(f32x16& d, const bf16x8& a, const f32x16& c) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, a[%2:%3], %4" : "+v"(d) : "v"(a), "n"(R), "n"(R + 3), "v"(c));
#endif
}
__device__ __forceinline__ void settle(f32x16& x, f32x16& y) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_nop 15\n\ts_nop 3" : "+v"(x), "+v"(y));
#endif
}
template <int R>
__device__ __forceinline__ void acc_put(unsigned v) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("v_accvgpr_write_b32 a[%0], %1" ::"n"(R), "v"(v) : PG_AGPRS);
#endif
}
template <int R>
__device__ __forceinline__ void acc_put_frag(const bf16x8& f) {
  typedef unsigned u4 __attribute__((ext_vector_type(4)));
  const u4 u = __builtin_bit_cast(u4, f);
  acc_put<R>(u[0]);
  acc_put<R + 1>(u[1]);
  acc_put<R + 2>(u[2]);
  acc_put<R + 3>(u[3]);
}
template <int R>
__device__ __forceinline__ void acc_zero() {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("v_accvgpr_write_b32 a[%0], 0" ::"n"(R) : PG_AGPRS);
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
  asm volatile("s_nop 15\n\ts_nop 15" ::: PG_AGPRS);
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
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds), "v"(voff), "s"(rs) : "memory", "m0");
#endif
}
__device__ __forceinline__ void dma4(u32x4 rs, unsigned lds, int voff) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds" ::"s"(lds), "v"(voff), "s"(rs) : "memory", "m0");
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

template <int N>
using Int = std::integral_constant<int, N>;
constexpr int kWideBK = 32;   // keys per staged tile

// dq_wide_kernel's copies of 32-row K and V tiles into a ring of LDS stages: waves 0, 1 fill the K tile,
// waves 2, 3 the V tile. A workgroup walks one or two runs of keys (the
// prefix, then responses).
template <int D>
struct KvCopies {
  static constexpr int TILE = LdsTile<bf16, D>::bytes(kWideBK);
  static constexpr int STAGE = 2 * TILE;
  static constexpr int PW = TILE / 1024 / 2;  // copies per wave and tile
  static_assert(TILE % 2048 == 0, "copies split evenly over the waves");
  int voff[PW];
  unsigned lds;
  int left, row_bytes, next_rows;
  uint64_t next_src;
  u32x4 rs;
  __device__ __forceinline__ void move_to(uint64_t addr) {
    rs[0] = uniform((int)(unsigned)addr);
    rs[1] = uniform((int)(unsigned)(addr >> 32));
  }
  __device__ __forceinline__ void set_rows() { rs[2] = min(left, kWideBK) * row_bytes; }
  // first run: n0 rows from s0 (this wave's tensor), then n1 rows from s1; row stride in elements
  __device__ __forceinline__ void init(const char* stage, const bf16* s0, int n0, const bf16* s1, int n1, int stride,
                                       int wave, int lane) {
    using L = LdsTile<bf16, D>;
    row_bytes = stride * 2;
#pragma unroll
    for (int k = 0; k < PW; ++k) {
      const int p = 1024 * ((wave & 1) + 2 * k) + 16 * lane;
      const int row = p / L::kPitch, pc = (p % L::kPitch) / 16;
      voff[k] = pc < L::kChunks ? row * row_bytes + 16 * (pc ^ L::swz(row)) : 0x7ffffff0;
    }
    lds = lds_addr(stage) + TILE * (wave >> 1) + 1024 * (wave & 1);
    rs[3] = 0x00020000;
    left = n0 > 0 ? n0 : n1;
    move_to((uint64_t)(n0 > 0 ? s0 : s1));
    next_src = (uint64_t)s1;
    next_rows = n0 > 0 ? n1 : 0;
    set_rows();
  }
  __device__ __forceinline__ void next() {  // past the end a tile has no rows: zeros are stored
    move_to((rs[0] | (uint64_t)rs[1] << 32) + (unsigned)(kWideBK * row_bytes));
    left = max(left - kWideBK, 0);
    if (__builtin_expect(left == 0, 0)) {
      asm volatile("");
      left = next_rows;
      next_rows = 0;
      move_to(next_src);
    }
    set_rows();
  }
  __device__ __forceinline__ void part(int k, int off) const { dma16(rs, lds + off + 2048 * k, voff[k]); }
};

}  // namespace pg

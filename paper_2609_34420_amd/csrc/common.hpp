// Device-side building blocks shared by the gfx950 attention kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gt {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.69314718055994531f;

// 32x32x16 bf16 matrix-core product, fp32 accumulate (gfx950).
//   A operand: lane l supplies row (l & 31), k = (l >> 5) * 8 + [0, 8)
//   B operand: lane l supplies col (l & 31), k = (l >> 5) * 8 + [0, 8)
//   C/D:       lane l holds col (l & 31), rows 8u + 4 (l >> 5) + t in
//              register 4u + t (u, t in [0, 4))
__device__ __forceinline__ f32x16 mfma32(const bf16x8& a, const bf16x8& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// Index of the calling wave in its workgroup, as a wave-uniform (scalar)
// value: derived values such as buffer descriptors then stay in SGPRs.
__device__ __forceinline__ int wave_id() {
  return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
}

// Keep the compiler from moving instructions across this point (used after
// issuing prefetch loads, so no use of their results is hoisted next to
// them and forces an early wait).
__device__ __forceinline__ void sched_fence() { __builtin_amdgcn_sched_barrier(0); }

// Hide a loaded value from the optimiser until this point: nothing derived
// from it (e.g. the shifts that pack a transposed tile) can be computed
// earlier, next to the load, where it would force an early wait.
__device__ __forceinline__ void opaque(uint4& x) {
  asm volatile("" : "+v"(x.x), "+v"(x.y), "+v"(x.z), "+v"(x.w));
}
__device__ __forceinline__ void opaque(uint32_t& x) { asm volatile("" : "+v"(x)); }
__device__ __forceinline__ void opaque_f(float& x) { asm volatile("" : "+v"(x)); }

// Workgroup barrier that orders LDS accesses only: each wave waits for its
// own LDS operations (lgkmcnt), not for its global loads, so prefetches stay
// in flight across it. For kernels whose waves share nothing but LDS.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Wait for every outstanding vector-memory load (s_waitcnt vmcnt(0) with the
// other counters left free). Used once before a software-pipelined loop, so
// that values loaded ahead of it are not treated as pending inside the loop,
// where a conservative merge of the two loop entries would otherwise make the
// first use of the current tile also wait for the next tile's prefetch.
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// 2^x on the transcendental unit (v_exp_f32): exp2(-inf) = 0.
__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }

// Operand row permutation inside a 32-row block. If the A operand of a
// product loads block row perm32(m) into MFMA row m, then the C layout gives
// lane half g (lane >> 5) the 16 CONSECUTIVE block rows 16 g + r in its
// registers r = 0..15: C row 8u + 4g + t  <->  block row 16g + 4u + t.
// Consecutive rows per lane let one 16-byte load fetch the lane's spd bytes
// and let 8 consecutive registers feed the next product's operand.
__device__ __forceinline__ int perm32(int m) {
  return (((m >> 2) & 1) << 4) | ((m >> 3) << 2) | (m & 3);
}

__device__ __forceinline__ bf16x8 lds_b128(const uint16_t* p) {
  return *reinterpret_cast<const bf16x8*>(p);
}

__device__ __forceinline__ bf16x8 zero_bf16x8() {
  bf16x8 z;
#pragma unroll
  for (int i = 0; i < 8; ++i) z[i] = (__bf16)0.0f;
  return z;
}

__device__ __forceinline__ f32x16 zero_f32x16() {
  f32x16 z;
#pragma unroll
  for (int i = 0; i < 16; ++i) z[i] = 0.0f;
  return z;
}

__device__ __forceinline__ bf16x8 cvt_bf16x8(const float* x) {
  bf16x8 r;
#pragma unroll
  for (int i = 0; i < 8; ++i) r[i] = (__bf16)x[i];
  return r;
}

// Sum of the 8 bf16 values of v plus acc, by packed dot products with 1.
__device__ __forceinline__ float sum_bf16x8(const bf16x8& v, float acc) {
  const bf16x2 one = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
  for (int i = 0; i < 8; i += 2) {
    const bf16x2 pr = {v[i], v[i + 1]};
    acc = __builtin_amdgcn_fdot2_f32_bf16(pr, one, acc, false);
  }
  return acc;
}

// Weights of a pairwise LSE merge (Section III-A-1 part 3): a running state
// with log-sum-exp lo and a new block with lb combine to
// O = wo O_running + wb O_block, LSE = out. Two -inf inputs give weights 0 and
// out = -inf.
__device__ __forceinline__ void lse_merge_weights(float lo, float lb, float& wo, float& wb, float& out) {
  const float mx = fmaxf(lo, lb);
  if (mx == -INFINITY) {
    wo = 0.0f;
    wb = 0.0f;
    out = -INFINITY;
    return;
  }
  const float eo = expf(lo - mx), eb = expf(lb - mx);
  const float tot = eo + eb;
  wo = eo / tot;
  wb = eb / tot;
  out = mx + logf(tot);
}

__device__ __forceinline__ uint16_t f2bf(float x) {
  __bf16 b = (__bf16)x;
  return __builtin_bit_cast(uint16_t, b);
}

__device__ __forceinline__ float bf2f(uint16_t x) {
  return __uint_as_float(((uint32_t)x) << 16);
}

// Workgroup id -> logical id so that consecutive logical ids (the H heads of
// one row block, which share their spd tiles) land on the same XCD at about
// the same time. Workgroups are handed to the 8 XCDs round robin.
__device__ __forceinline__ int64_t xcd_remap(int64_t w, int64_t total) {
  if ((total & 7) != 0) return w;
  return (w & 7) * (total >> 3) + (w >> 3);
}

// Raw buffer resource over [base, base + 2 GiB): untyped loads, 32-bit data
// format (the gfx9-family descriptor word). Its loads are always inside the
// caller's buffer; the range field is not relied on.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, 0x7fffffff, 0x00020000);
}

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// Range check of a raw buffer load: only the lane offset (with the
// instruction's immediate) is counted on to be compared with the resource's
// end. A scalar offset is documented as left out of the comparison, and as
// subtracted from the end, which then goes negative for one past it; so where a
// load may lie past the end, the scalar part goes into the resource's start
// (make_rsrc_from in stage.hpp), and a scalar offset is given only to loads that are
// always inside.
__device__ __forceinline__ void buf_u128(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t w[4]) {
  const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, voff, 0, 0);
  w[0] = v[0]; w[1] = v[1]; w[2] = v[2]; w[3] = v[3];
}
// Of a load that is inside the caller's buffer whatever the lane.
__device__ __forceinline__ void buf_u128_inside(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff,
                                                uint32_t w[4]) {
  const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0);
  w[0] = v[0]; w[1] = v[1]; w[2] = v[2]; w[3] = v[3];
}

// A 16-byte spd group at any byte address, as the 5 dwords that hold it
// (voff4: its offset rounded down to a dword; dwords past the resource's end
// read 0). A load of 16 bytes from an odd address costs up to 1.4 times the
// whole forward (N = 16001 against 16004 at H = 8, d = 64: 936 and 659 us),
// one from a dword boundary costs no more than an aligned one.
__device__ __forceinline__ void load_spd5(__amdgpu_buffer_rsrc_t r, uint32_t voff4, uint32_t (&w)[5]) {
  const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, voff4, 0, 0);
  w[0] = v[0]; w[1] = v[1]; w[2] = v[2]; w[3] = v[3];
  w[4] = __builtin_amdgcn_raw_buffer_load_b32(r, voff4 + 16u, 0, 0);
}
// Its 16 bytes into w[0..3] (sh: its address mod 4).
__device__ __forceinline__ void align_spd5(uint32_t (&w)[5], uint32_t sh) {
#pragma unroll
  for (int i = 0; i < 4; ++i) w[i] = __builtin_amdgcn_alignbyte(w[i + 1], w[i], sh);
}

}  // namespace gt

// Device-side building blocks shared by the MomentKV kernels (gfx950 / CDNA4, wave64).
//
//   * element access for fp32 and bf16 (bf16 kept as uint16 bit patterns, RNE rounding)
//   * 8-element MFMA fragments: a lane holds 8 consecutive elements along the
//     contraction index, so fp32 and bf16 operands are loaded the same way
//   * 16x16 MFMA tile product for both element types
//   * 16-lane row reductions through DPP and 64-lane wave reductions
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mkv {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef uint16_t bf16_t;  // storage type of bf16 tensors

constexpr int kWave = 64;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

__device__ __forceinline__ float bf2f(bf16_t x) { return __uint_as_float((uint32_t)x << 16); }

__device__ __forceinline__ bf16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (bf16_t)((u >> 16) | 0x40u);  // quiet NaN
  u += 0x7fffu + ((u >> 16) & 1u);                                             // RNE
  return (bf16_t)(u >> 16);
}

template <class T> __device__ __forceinline__ float to_f(T x);
template <> __device__ __forceinline__ float to_f<float>(float x) { return x; }
template <> __device__ __forceinline__ float to_f<bf16_t>(bf16_t x) { return bf2f(x); }

template <class T> __device__ __forceinline__ T from_f(float x);
template <> __device__ __forceinline__ float from_f<float>(float x) { return x; }
template <> __device__ __forceinline__ bf16_t from_f<bf16_t>(float x) { return f2bf(x); }

// ---------------------------------------------------------------- MFMA fragments
template <class T> struct Frag;
template <> struct Frag<bf16_t> { typedef bf16x8 type; };
template <> struct Frag<float> { typedef f32x8 type; };

// 8 consecutive elements starting at p (16-byte aligned for bf16, 32-byte for fp32).
__device__ __forceinline__ bf16x8 load_frag(const bf16_t* p) {
  uint4 u = *reinterpret_cast<const uint4*>(p);
  return __builtin_bit_cast(bf16x8, u);
}
__device__ __forceinline__ f32x8 load_frag(const float* p) {
  float4 a = reinterpret_cast<const float4*>(p)[0];
  float4 b = reinterpret_cast<const float4*>(p)[1];
  f32x8 r;
  r[0] = a.x; r[1] = a.y; r[2] = a.z; r[3] = a.w;
  r[4] = b.x; r[5] = b.y; r[6] = b.z; r[7] = b.w;
  return r;
}

// The converse of load_frag.
__device__ __forceinline__ void store_frag(bf16_t* p, const bf16x8& f) {
  *reinterpret_cast<uint4*>(p) = __builtin_bit_cast(uint4, f);
}
__device__ __forceinline__ void store_frag(float* p, const f32x8& f) {
  reinterpret_cast<float4*>(p)[0] = make_float4(f[0], f[1], f[2], f[3]);
  reinterpret_cast<float4*>(p)[1] = make_float4(f[4], f[5], f[6], f[7]);
}

// Compile-time choice between two types.
template <bool C, class A, class B> struct Pick { typedef A type; };
template <class A, class B> struct Pick<false, A, B> { typedef B type; };

template <class T> __device__ __forceinline__ typename Frag<T>::type zero_frag();
template <> __device__ __forceinline__ bf16x8 zero_frag<bf16_t>() {
  return __builtin_bit_cast(bf16x8, make_uint4(0, 0, 0, 0));
}
template <> __device__ __forceinline__ f32x8 zero_frag<float>() {
  f32x8 r;
#pragma unroll
  for (int e = 0; e < 8; ++e) r[e] = 0.f;
  return r;
}

// Element access.  Elements of a bf16 fragment are read through a bit cast of the whole
// vector to 16-bit integers: a bit cast of a single __bf16 vector element does not select
// the element on this toolchain.
__device__ __forceinline__ bf16_t raw_elem(const bf16x8& f, int e) {
  const u16x8 u = __builtin_bit_cast(u16x8, f);
  return u[e];
}
__device__ __forceinline__ float raw_elem(const f32x8& f, int e) { return f[e]; }
__device__ __forceinline__ float elem_f(const bf16x8& f, int e) { return bf2f(raw_elem(f, e)); }
__device__ __forceinline__ float elem_f(const f32x8& f, int e) { return f[e]; }

// C(16x16) += A(16x32) * B(32x16).  Lane l supplies A[l%16][8*(l/16) + e] and
// B[8*(l/16) + e][l%16], e = 0..7, and holds C[4*(l/16) + i][l%16], i = 0..3.
// bf16: one v_mfma_f32_16x16x32_bf16.  fp32: eight v_mfma_f32_16x16x4f32, the e-th one
// pairing element e of every lane (the 32-long contraction is covered in another order,
// which only changes the summation order).
__device__ __forceinline__ void mma(f32x4& c, const bf16x8& a, const bf16x8& b) {
  c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ void mma(f32x4& c, const f32x8& a, const f32x8& b) {
#pragma unroll
  for (int e = 0; e < 8; ++e) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], c, 0, 0, 0);
}

// An MFMA operand fragment read transposed from a row-major bf16 tile in LDS whose rows
// run along the contraction: lane l receives tile[r0 + 8 (l / 16) + e][c0 + l % 16],
// e = 0..7 (the B layout above with the tile's columns as n; the A layout with them as
// m).  ds_read_b64_tr_b16 hands each group of 16 lanes a 4 x 16 block whose row m is read
// by lanes 4m .. 4m + 3 (eight bytes each) and gives lane j the block's column j; two
// such reads cover the eight rows.  ld (elements) and c0 keep every read 8-byte aligned.
__device__ __forceinline__ bf16x8 lds_frag_tr(const bf16_t* tile, int ld, int r0, int c0, int lane) {
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
  const int i = lane & 15;
  const bf16_t* p = tile + (r0 + 8 * (lane >> 4) + (i >> 2)) * ld + c0 + 4 * (i & 3);
  const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p);
  const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * ld));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

__device__ __forceinline__ f32x4 zero4() {
  f32x4 r;
  r[0] = r[1] = r[2] = r[3] = 0.f;
  return r;
}

// ---------------------------------------------------------------- lane reductions
// DPP row_ror:n rotates within each row of 16 lanes; the butterfly below leaves the
// same value in all 16 lanes of a row (every step combines a commutative pair).
template <int CTRL> __device__ __forceinline__ float dpp_f(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false));
}
template <int CTRL> __device__ __forceinline__ int dpp_i(int x) {
  return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xF, 0xF, false);
}
__device__ __forceinline__ float row16_sum(float x) {
  x += dpp_f<0x128>(x);
  x += dpp_f<0x124>(x);
  x += dpp_f<0x122>(x);
  x += dpp_f<0x121>(x);
  return x;
}
__device__ __forceinline__ float row16_max(float x) {
  x = fmaxf(x, dpp_f<0x128>(x));
  x = fmaxf(x, dpp_f<0x124>(x));
  x = fmaxf(x, dpp_f<0x122>(x));
  x = fmaxf(x, dpp_f<0x121>(x));
  return x;
}
// Sum over the lanes of a quad (4 consecutive lanes), same value in all four.
__device__ __forceinline__ float quad_sum(float x) {
  x += dpp_f<0xB1>(x);  // quad_perm [1,0,3,2]
  x += dpp_f<0x4E>(x);  // quad_perm [2,3,0,1]
  return x;
}
// Sum over lanes l, l^16, l^32, l^48 (the four 16-lane rows), same value in each.  The row
// and half swaps of gfx950 are vector instructions (a shuffle is an LDS round trip): of two
// copies of x, one ends with rows (0, 0, 2, 2), the other with rows (1, 1, 3, 3); the
// halves likewise.
template <class F>
__device__ __forceinline__ float cross_row(float x, F f) {
  const uint32_t u = __float_as_uint(x);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const uint32_t y = __float_as_uint(f(__uint_as_float(r[0]), __uint_as_float(r[1])));
  const auto h = __builtin_amdgcn_permlane32_swap(y, y, false, false);
  return f(__uint_as_float(h[0]), __uint_as_float(h[1]));
}
__device__ __forceinline__ float cross_row_sum(float x) {
  return cross_row(x, [](float p, float q) { return p + q; });
}
__device__ __forceinline__ float cross_row_max(float x) {
  return cross_row(x, [](float p, float q) { return fmaxf(p, q); });
}
__device__ __forceinline__ float wave_sum(float x) { return cross_row_sum(row16_sum(x)); }
__device__ __forceinline__ float wave_max(float x) { return cross_row_max(row16_max(x)); }

__device__ __forceinline__ float wave_min(float x) {
  x = fminf(x, dpp_f<0x128>(x));
  x = fminf(x, dpp_f<0x124>(x));
  x = fminf(x, dpp_f<0x122>(x));
  x = fminf(x, dpp_f<0x121>(x));
  return cross_row(x, [](float p, float q) { return fminf(p, q); });
}
__device__ __forceinline__ int wave_min_i(int x) {
  x = min(x, dpp_i<0x128>(x));
  x = min(x, dpp_i<0x124>(x));
  x = min(x, dpp_i<0x122>(x));
  x = min(x, dpp_i<0x121>(x));
  const auto r = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)x, false, false);
  x = min((int)r[0], (int)r[1]);
  const auto h = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)x, false, false);
  return min((int)h[0], (int)h[1]);
}

// Inclusive prefix sum over the 64 lanes through DPP (row shifts, then the row totals
// broadcast into the rows after): no LDS round trips.
template <int CTRL, int ROWS> __device__ __forceinline__ int dpp_rows_i(int x) {
  return __builtin_amdgcn_update_dpp(0, x, CTRL, ROWS, 0xF, false);
}
__device__ __forceinline__ int wave_incl_scan(int x) {
  x += dpp_rows_i<0x111, 0xF>(x);  // row_shr:1
  x += dpp_rows_i<0x112, 0xF>(x);  // row_shr:2
  x += dpp_rows_i<0x114, 0xF>(x);  // row_shr:4
  x += dpp_rows_i<0x118, 0xF>(x);  // row_shr:8
  x += dpp_rows_i<0x142, 0xA>(x);  // row_bcast:15 into rows 1 and 3
  x += dpp_rows_i<0x143, 0xC>(x);  // row_bcast:31 into rows 2 and 3
  return x;
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// ---------------------------------------------------------------- query rows
// Query g of a group sits in MFMA row (column) 4 (g % 4) + g / 4, so that a lane's result
// rows 4 (l / 16) + i hold queries 4 i + l / 16: with up to four queries per group only
// i = 0 is work (the online softmax of four rows per lane, three of them padding, was most
// of a block's vector instructions), with up to eight i = 0, 1.  The map is its own inverse.
__device__ __forceinline__ int query_of(int row) { return 4 * (row & 3) + (row >> 2); }

// ---------------------------------------------------------------- in-launch hand-off
// Results that one workgroup hands to another of the same launch go through agent-scope
// relaxed atomic stores and loads, which are not served from the per-XCD caches (those are
// not kept coherent with each other).  A writer waits until its own stores have completed
// (stores_complete) before it counts itself in, and the last to arrive reads only after the
// count (loads_after_count), so no device-scope fence is needed (on this part such a fence
// writes back and invalidates a whole L2).
// s_waitcnt with vmcnt = 0 and the other counters at their maximum: every vector memory
// operation of the wave issued so far (stores included) has completed.
constexpr int kWaitVmem = 0x0F70;
__device__ __forceinline__ void stores_complete() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_s_waitcnt(kWaitVmem);
}
__device__ __forceinline__ void loads_after_count() {
  __builtin_amdgcn_s_waitcnt(kWaitVmem);
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

__device__ __forceinline__ void st_agent_u32(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t ld_agent_u32(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_agent_u64(uint64_t* p, uint64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t ld_agent_u64(const uint64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Online (max, sum) pair in the base-2 domain: represents sum_i 2^(x_i) = l * 2^m.
__device__ __forceinline__ void ml_merge(float& m, float& l, float m2, float l2) {
  float mn = fmaxf(m, m2);
  if (mn == -INFINITY) return;  // both empty
  l = l * fast_exp2(m - mn) + l2 * fast_exp2(m2 - mn);
  m = mn;
}

}  // namespace mkv

// Device-side helpers shared by the HIP kernels: storage formats and wave-level reductions (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <hip/hip_ext.h>

namespace flk {

enum { DT_F32 = 0, DT_F16 = 1, DT_BF16 = 2 };

// Launch with optional timing: when ev0 / ev1 are given they take the start / end time stamps of this very dispatch
// (no extra packets on the stream, so a timed launch costs what an untimed one does and the elapsed time between the two
// is the kernel's own duration); without them a plain launch.
template <typename... KArgs, typename... Args>
inline void launch_timed(void (*kernel)(KArgs...), dim3 grid, dim3 block, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1,
                         Args... args) {
  if (ev0 || ev1) hipExtLaunchKernelGGL(kernel, grid, block, 0, st, ev0, ev1, 0, static_cast<KArgs>(args)...);
  else hipLaunchKernelGGL(kernel, grid, block, 0, st, static_cast<KArgs>(args)...);
}

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4_t;   // 16 bytes of storage
typedef u32x4_t u32x4_any __attribute__((aligned(2)));               // ... of 16-bit rows, or
typedef f32x4_t f32x4_any __attribute__((aligned(4)));               // fp32 rows, that a caller may start at any element

template <int DT> struct Store;          // storage element of a model dtype
template <> struct Store<DT_F32> { typedef float type; };
template <> struct Store<DT_F16> { typedef uint16_t type; };
template <> struct Store<DT_BF16> { typedef uint16_t type; };

__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }
__device__ __forceinline__ float f16_to_f32(uint16_t h) { return (float)__builtin_bit_cast(_Float16, h); }

// fp32 -> bf16, round to nearest even (NaN kept quiet).
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ uint16_t f32_to_f16(float f) { return __builtin_bit_cast(uint16_t, (_Float16)f); }

template <int DT> __device__ __forceinline__ float ld(const void* p, size_t i) {
  if constexpr (DT == DT_F32) return ((const float*)p)[i];
  else if constexpr (DT == DT_F16) return f16_to_f32(((const uint16_t*)p)[i]);
  else return bf16_to_f32(((const uint16_t*)p)[i]);
}
template <int DT> __device__ __forceinline__ void st(void* p, size_t i, float v) {
  if constexpr (DT == DT_F32) ((float*)p)[i] = v;
  else if constexpr (DT == DT_F16) ((uint16_t*)p)[i] = f32_to_f16(v);
  else ((uint16_t*)p)[i] = f32_to_bf16(v);
}
// value after rounding to the model dtype
template <int DT> __device__ __forceinline__ float rdt(float v) {
  if constexpr (DT == DT_F32) return v;
  else if constexpr (DT == DT_F16) return f16_to_f32(f32_to_f16(v));
  else return bf16_to_f32(f32_to_bf16(v));
}

// 16 bytes of storage -> fp32 lanes (8 values for the 16-bit dtypes, 4 for fp32)
template <int DT> __device__ __forceinline__ void unpack16(const u32x4_t& r, float* f) {
  if constexpr (DT == DT_F32) {
    f[0] = __uint_as_float(r.x); f[1] = __uint_as_float(r.y); f[2] = __uint_as_float(r.z); f[3] = __uint_as_float(r.w);
  } else if constexpr (DT == DT_BF16) {
    f[0] = __uint_as_float(r.x << 16); f[1] = __uint_as_float(r.x & 0xffff0000u);
    f[2] = __uint_as_float(r.y << 16); f[3] = __uint_as_float(r.y & 0xffff0000u);
    f[4] = __uint_as_float(r.z << 16); f[5] = __uint_as_float(r.z & 0xffff0000u);
    f[6] = __uint_as_float(r.w << 16); f[7] = __uint_as_float(r.w & 0xffff0000u);
  } else {
    f[0] = f16_to_f32((uint16_t)(r.x & 0xffffu)); f[1] = f16_to_f32((uint16_t)(r.x >> 16));
    f[2] = f16_to_f32((uint16_t)(r.y & 0xffffu)); f[3] = f16_to_f32((uint16_t)(r.y >> 16));
    f[4] = f16_to_f32((uint16_t)(r.z & 0xffffu)); f[5] = f16_to_f32((uint16_t)(r.z >> 16));
    f[6] = f16_to_f32((uint16_t)(r.w & 0xffffu)); f[7] = f16_to_f32((uint16_t)(r.w >> 16));
  }
}

// ---- layout of the 16-bit GEMM inputs (norm output, attention output, MLP activation) inside a pass
// "Fragment order": x[M][K] is kept as tiles of 16 rows x 32 k in the order the MFMA reads its row operand -- lane l
// of a tile holds x[16*mt + l%16][32*kb + 8*(l/16) .. +7] (16 bytes) -- tiles ordered [k-block][row tile], so one
// fragment load of a wave is 1 KiB contiguous and the row tiles of a k-block follow each other.  mtt = row tiles of the
// pass (ceil(M/16)); mtt == 0 means plain row-major with leading dimension ld.  k % 4 == 0 keeps 4 consecutive
// elements contiguous in both layouts.
__device__ __forceinline__ size_t xrow_index(int m, int k, int ld, int mtt) {
  if (mtt == 0) return (size_t)m * ld + k;
  return ((size_t)(k >> 5) * mtt + (m >> 4)) * 512 + ((((k & 31) >> 3) << 4) + (m & 15)) * 8 + (k & 7);
}

// ---- 4 consecutive elements at a time
__device__ __forceinline__ f32x4_t ld4(const float* p) { return *(const f32x4_t*)p; }
template <int DT> __device__ __forceinline__ f32x4_t ldv4(const void* p, size_t i) {   // 4 consecutive dtype elements
  if constexpr (DT == DT_F32) return *(const f32x4_t*)((const float*)p + i);
  else {
    const uint2 r = *(const uint2*)((const uint16_t*)p + i);
    if constexpr (DT == DT_BF16)
      return f32x4_t{__uint_as_float(r.x << 16), __uint_as_float(r.x & 0xffff0000u), __uint_as_float(r.y << 16),
                     __uint_as_float(r.y & 0xffff0000u)};
    else
      return f32x4_t{f16_to_f32((uint16_t)(r.x & 0xffffu)), f16_to_f32((uint16_t)(r.x >> 16)),
                     f16_to_f32((uint16_t)(r.y & 0xffffu)), f16_to_f32((uint16_t)(r.y >> 16))};
  }
}
template <int DT> __device__ __forceinline__ void stv4(void* p, size_t i, f32x4_t v) {
  if constexpr (DT == DT_F32) *(f32x4_t*)((float*)p + i) = v;
  else {
    uint2 r;
    if constexpr (DT == DT_BF16) {
      r.x = (uint32_t)f32_to_bf16(v[0]) | ((uint32_t)f32_to_bf16(v[1]) << 16);
      r.y = (uint32_t)f32_to_bf16(v[2]) | ((uint32_t)f32_to_bf16(v[3]) << 16);
    } else {
      r.x = (uint32_t)f32_to_f16(v[0]) | ((uint32_t)f32_to_f16(v[1]) << 16);
      r.y = (uint32_t)f32_to_f16(v[2]) | ((uint32_t)f32_to_f16(v[3]) << 16);
    }
    *(uint2*)((uint16_t*)p + i) = r;
  }
}

// ---- row-wise epilogue arithmetic shared by the stand-alone kernels and the GEMM kernels that fuse them
// Floating-point contraction is switched off inside, so that the same inputs give the same bits wherever the function
// is inlined (a request's result must not depend on which variant served it).
// Norm of a row: sums of four consecutive elements, and the normalised elements (layer norm, or RMS where mean and b are not used).
__device__ __forceinline__ float sum4(const f32x4_t& t) { return (t[0] + t[1]) + (t[2] + t[3]); }
__device__ __forceinline__ float square_sum4(const f32x4_t& t) {
#pragma clang fp contract(off)
  return fmaf(t[0], t[0], t[1] * t[1]) + fmaf(t[2], t[2], t[3] * t[3]);
}
template <bool RMS> __device__ __forceinline__ f32x4_t norm_value(const f32x4_t& v, float mean, float inv, const f32x4_t& g, const f32x4_t& b) {
#pragma clang fp contract(off)
  f32x4_t o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = RMS ? v[e] * inv * g[e] : fmaf((v[e] - mean) * inv, g[e], b[e]);
  return o;
}
// Rotary pair (a0, a1) = elements (i, i + d/2) of a head, (cs, sn) = cos/sin of pos * theta^(-2i/d).
__device__ __forceinline__ void rope_rotate(f32x4_t& a0, f32x4_t& a1, const f32x4_t& cs, const f32x4_t& sn) {
#pragma clang fp contract(off)
  const f32x4_t r0 = a0 * cs - a1 * sn, r1 = a1 * cs + a0 * sn;
  a0 = r0;
  a1 = r1;
}
__device__ __forceinline__ f32x4_t act_swiglu(const f32x4_t& g, const f32x4_t& u) {   // silu(g) * u
#pragma clang fp contract(off)
  f32x4_t o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = g[e] / (1.0f + expf(-g[e])) * u[e];
  return o;
}
// Tanh form of GELU.  16-bit results take 0.5 (1 + tanh v) as 1 / (1 + exp(-2v)), the same function: tanhf spelled out for every
// accumulator of a tile kernel is 15 to 63 KB of code that runs once and is fetched cold (8192 x 2048 at 138 / 287 / 436 rows: 23.2 /
// 26.9 / 28.4 -> 21.1 / 25.7 / 27.1 us), and where the tail cancels it loses all digits; fp32 keeps tanhf.  The quotient t / (1 + e) is
// taken with the rounding of 1 + e put back and one correction step, in place of a division.  2-norm of the error against 64 bits before the
// rounding to 16 bits, tanhf / plain quotient / this: t normal 3.8e-8 / 4.2e-8 / 2.8e-8, of deviation 0.1 3.8e-8 / 4.1e-8 / 2.9e-8, of 3
// 2.8e-8 / 3.3e-8 / 2.1e-8, uniform in -9..-5 0.44 / 8.8e-7 / 6.9e-7.
template <int DT> __device__ __forceinline__ float gelu(float t) {
#pragma clang fp contract(off)
  if constexpr (DT == DT_F32) return 0.5f * t * (1.0f + tanhf(0.7978845608028654f * (t + 0.044715f * t * t * t)));
  const float e = expf(-t * fmaf((float)(1.5957691216057308 * 0.044715), t * t, 1.5957691216057308f)), s = 1.0f + e, lost = e - (s - 1.0f);
  const float inv = __builtin_amdgcn_rcpf(s), q = t * inv, left = fmaf(-q, lost, fmaf(-q, s, t));
  // a remainder that is zero, infinite or no number corrects nothing: signed zeros, infinities and NaN stay what q is
  return __builtin_amdgcn_classf(left, 0x198) ? fmaf(left, inv, q) : q;
}
template <int DT> __device__ __forceinline__ f32x4_t act_gelu(const f32x4_t& t) {
  f32x4_t o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = gelu<DT>(t[e]);
  return o;
}

// ---- matrix core: D[16][16] += A[16][32] . B[32][16]
template <int DT> __device__ __forceinline__ f32x4_t mfma16(const u32x4_t& a, const u32x4_t& b, f32x4_t c) {
  if constexpr (DT == DT_BF16)
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b), c, 0, 0, 0);
}

// ---- asynchronous copies to LDS
// Barrier behind which at most N of this wave's copies are still in flight (none when `all`) and its LDS reads are done.
// The waits are builtins outside any branch, so that the compiler knows that the fragments read before have arrived.
template <int N> __device__ __forceinline__ void copies_barrier(bool all) {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((N & 15) | 7 << 4 | (N >> 4) << 14);        // vmcnt(N) lgkmcnt(0)
  if (all) __builtin_amdgcn_s_waitcnt(7 << 4 | 15 << 8);                 // vmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
// 64 lanes x 16 bytes, lane i from base + off (base is wave-uniform) to l[i].  The buffer form: after the global form the
// compiler counts later LDS reads and loads as out of order and waits for all of them.
__device__ __forceinline__ void copy_to_lds(const char* base, uint32_t off, u32x4_t* l) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, -1, 0x00020000),
                                           (__attribute__((address_space(3))) void*)l, 16, off, 0, 0, 0);
}

// ---- cross-lane: DPP within a row of 16 lanes, lane swaps beyond.  Every step is a fixed butterfly,
// so a reduction's result does not depend on anything but the values reduced.
template <int CTRL> __device__ __forceinline__ float dpp_f(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}
// xor-butterfly partner of `v` at distance DIST (1, 2, 4 or 8); valid when all lanes at smaller distances
// already agree for DIST in {4, 8} (mirror forms), which is how the reductions below use it.
template <int DIST> __device__ __forceinline__ float partner(float v) {
  if constexpr (DIST == 1) return dpp_f<0xB1>(v);        // quad_perm [1,0,3,2]
  else if constexpr (DIST == 2) return dpp_f<0x4E>(v);   // quad_perm [2,3,0,1]
  else if constexpr (DIST == 4) return dpp_f<0x141>(v);  // row_half_mirror
  else {
    static_assert(DIST == 8, "within a row of 16 lanes");
    return dpp_f<0x140>(v);                              // row_mirror
  }
}
// v + its partner, and the larger of the two; at distances 16 and 32 the lane swaps give both sides of the pair without a
// round through LDS (sums are the same bits: a + b = b + a).
template <int DIST> __device__ __forceinline__ float sum_partner(float v) {
  if constexpr (DIST < 16) {
    return v + partner<DIST>(v);
  } else {
    const auto r = DIST == 16 ? __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false)
                              : __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
}
template <int DIST> __device__ __forceinline__ float max_partner(float v) {
  if constexpr (DIST < 16) {
    return fmaxf(v, partner<DIST>(v));
  } else {
    const auto r = DIST == 16 ? __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false)
                              : __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  }
}
// all-reduce sum over aligned groups of W lanes (W = 2..64), every lane gets the total
template <int W> __device__ __forceinline__ float group_sum(float v) {
  if constexpr (W >= 2) v = sum_partner<1>(v);
  if constexpr (W >= 4) v = sum_partner<2>(v);
  if constexpr (W >= 8) v = sum_partner<4>(v);
  if constexpr (W >= 16) v = sum_partner<8>(v);
  if constexpr (W >= 32) v = sum_partner<16>(v);
  if constexpr (W >= 64) v = sum_partner<32>(v);
  return v;
}

}  // namespace flk

// Shared device helpers for the gfx950 kernels: bf16 bit conversion, vector
// types, wave reductions and the launch-check macro.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdlib.h>
#include <type_traits>
#include "../../include/distrifusion.h"

namespace df {

typedef unsigned short bf16_t;  // raw bfloat16 bits

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;

__device__ __forceinline__ float bf2f(bf16_t v) { return __uint_as_float(((unsigned int)v) << 16); }

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;

// float -> bf16, round to nearest even, in hardware (v_cvt_pk_bf16_f32 on gfx950)
__device__ __forceinline__ unsigned int pack_bf2(float lo, float hi) {
  const f32x2 v = {lo, hi};
  return __builtin_bit_cast(unsigned int, __builtin_convertvector(v, bf16x2));
}

__device__ __forceinline__ bf16_t f2bf(float f) { return (bf16_t)(pack_bf2(f, 0.f) & 0xffffu); }

// x * sigmoid(x); the hardware reciprocal (1 ulp) replaces the multi-instruction IEEE division
__device__ __forceinline__ float silu_f(float x) {
  return x * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * x));
}

// GELU in its exact (erf) form, 0.5 x (1 + erf(x / sqrt 2)) = max(x, 0) - |x| Q(|x|) for both signs, Q(a) = erfc(a / sqrt 2) / 2: for
// negative arguments nothing cancels.  log2 Q is so smooth that a polynomial of degree 8 in a holds it: fitted here by reweighted least
// squares on [0, 5.6] to |error of a Q| <= 1e-7 and |error of Q| <= 1e-4 Q (0.61 of either bound reached; Q < 1e-8 beyond, where the
// polynomial goes on falling to -infinity).  Against 64 bits the float function is off by 2.4e-7 at most and 4.1e-8 rms over N(0, 1)
// (Abramowitz & Stegun 7.1.26, with a reciprocal besides: 3.3e-7 and 5.4e-8), 6e-5 of the value at arguments around -5 (2.5e-3).
// Twelve instructions per value, one of them at a quarter of the rate: the GEGLU epilogues are bounded by them.
// The factor of Q is kept finite, so that +inf stays +inf (Q is 0 there).
__device__ __forceinline__ float gelu_erf(float x) {
  const float a = fabsf(x);
  float q = fmaf(-6.546825e-07f, a, 1.1150935e-05f);
  q = fmaf(q, a, -4.1239004e-05f);
  q = fmaf(q, a, -0.00051439233f);
  q = fmaf(q, a, 0.007592879f);
  q = fmaf(q, a, -0.05288758f);
  q = fmaf(q, a, -0.45907083f);
  q = fmaf(q, a, -1.1511227f);
  q = fmaf(q, a, -0.99999964f);
  return fmaf(-fabsf(fminf(x, 3.0e38f)), __builtin_amdgcn_exp2f(q), fmaxf(x, 0.f));
}

template <typename T> struct Elem;
template <> struct Elem<float> {
  static constexpr int kVec = 4;  // elements per 16-byte access
  __device__ static __forceinline__ float ld(const float* p) { return *p; }
  __device__ static __forceinline__ void st(float* p, float v) { *p = v; }
};
template <> struct Elem<bf16_t> {
  static constexpr int kVec = 8;
  __device__ static __forceinline__ float ld(const bf16_t* p) { return bf2f(*p); }
  __device__ static __forceinline__ void st(bf16_t* p, float v) { *p = f2bf(v); }
};

// 16-byte vector load/store of kVec elements to/from float registers
__device__ __forceinline__ void ld_vec(const float* p, float* v) {
  f32x4 t = *reinterpret_cast<const f32x4*>(p);
  v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
}
__device__ __forceinline__ void ld_vec(const bf16_t* p, float* v) {
  u32x4 t = *reinterpret_cast<const u32x4*>(p);
  v[0] = __uint_as_float(t.x << 16); v[1] = __uint_as_float(t.x & 0xffff0000u);
  v[2] = __uint_as_float(t.y << 16); v[3] = __uint_as_float(t.y & 0xffff0000u);
  v[4] = __uint_as_float(t.z << 16); v[5] = __uint_as_float(t.z & 0xffff0000u);
  v[6] = __uint_as_float(t.w << 16); v[7] = __uint_as_float(t.w & 0xffff0000u);
}
__device__ __forceinline__ void st_vec(float* p, const float* v) {
  f32x4 t = {v[0], v[1], v[2], v[3]};
  *reinterpret_cast<f32x4*>(p) = t;
}
__device__ __forceinline__ void st_vec(bf16_t* p, const float* v) {
  u32x4 t = {pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3]), pack_bf2(v[4], v[5]), pack_bf2(v[6], v[7])};
  *reinterpret_cast<u32x4*>(p) = t;
}

// Direct loads, memory -> LDS: lane i's 16 bytes go to dst + 16 i (`dst` the same for the whole wave).  They count in vmcnt, and
// the caller waits (s_waitcnt, then a barrier if other waves read).  Two forms, neither of them the compiler's global_load_lds
// builtin: it takes that for an access to LDS in flight and turns every wait for an LDS read behind one into lgkmcnt(0), so
// operands requested for the next matrix instructions were waited for at once.
//   - lds_load_buf: from base + sofs (uniform) + ofs bytes.  The form to use where 32-bit lane offsets do.
//   - lds_load16: from a lane's own pointer, or base (uniform) + ofs bytes, as instructions the compiler does not count: keep it
//     out of loops that are entered with other loads in flight (it waits for those with vmcnt(0) in every pass).  M0, which
//     holds the LDS address, is named as clobbered: the compiler warns that it is a reserved register, and orders its own writes
//     of M0 (for lds_load_buf) by it.
// 1800 x 1280 x 5120 on 128 x 128 tiles (bgemm.hip): 50 us with the global builtin, 52 - 54 with lds_load16 (the residual's
// loads are in flight there), 40.4 with lds_load_buf; attention 7200 x 57600 x 10 heads: 1227, 1194, 1215 us.
__device__ __forceinline__ unsigned int lds_offset(const void* p) {
  return (unsigned int)(uintptr_t)(__attribute__((address_space(3))) const void*)p;
}
__device__ __forceinline__ void lds_load_buf(const void* base, unsigned int ofs, unsigned int sofs, void* dst) {
  // raw buffer descriptor: stride 0, no bound, data format 32
  __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, -1, 0x00020000),
                                           (__attribute__((address_space(3))) void*)dst, 16, ofs, sofs, 0, 0);
}
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void lds_load16(const void* src, const void* dst) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(lds_offset(dst)) : "memory", "m0");
}
__device__ __forceinline__ void lds_load16(const void* base, unsigned int ofs, const void* dst) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(ofs), "s"(base), "s"(lds_offset(dst)) : "memory", "m0");
}
#pragma clang diagnostic pop

// x / d of 32 bits from the reciprocal of d rounded down, (2^32 - 1) / d: that is at most 1 less than 2^32 / d, so the product's upper half
// is the quotient or one less, for every x and d.
__host__ __device__ inline unsigned int reciprocal_u32(unsigned int d) { return 0xffffffffu / d; }
__host__ __device__ inline unsigned int quotient_u32(unsigned int x, unsigned int d, unsigned int reciprocal) {
  const unsigned int q = (unsigned int)(((unsigned long long)x * reciprocal) >> 32);
  return q + (x - q * d >= d ? 1u : 0u);
}

// A barrier that no memory access is moved across, without the wait for all of them that __syncthreads brings
__device__ __forceinline__ void block_sync() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// The wave's sum, the same for every lane, added in a fixed order: within rows of 16 lanes, then over the rows, by lane moves of the
// vector ALU (six of them; a step through LDS costs a round trip).
__device__ __forceinline__ float wave_total(float v) {
  auto add = [&](auto ctrl, auto rows) {
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), decltype(ctrl)::value, decltype(rows)::value, 0xf, true));
  };
  add(std::integral_constant<int, 0x111>{}, std::integral_constant<int, 0xf>{});   // row_shr:1, 2, 4, 8: lane 15 of a row has its sum
  add(std::integral_constant<int, 0x112>{}, std::integral_constant<int, 0xf>{});
  add(std::integral_constant<int, 0x114>{}, std::integral_constant<int, 0xf>{});
  add(std::integral_constant<int, 0x118>{}, std::integral_constant<int, 0xf>{});
  add(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{});   // row_bcast:15 into rows 1 and 3
  add(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{});   // row_bcast:31 into rows 2 and 3
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// Kernel-selection overrides from the environment (DF_TG, DF_TGS, DF_BGEMM, DF_PARTS, DF_ATTN_*) exist only in builds with
// -DDF_TUNING; in the library as shipped every choice is a function of the call's arguments alone.
#ifdef DF_TUNING
static inline const char* tune_env(const char* name) { return getenv(name); }
#else
static inline const char* tune_env(const char*) { return nullptr; }
#endif

// Position of row m (within its batch item) of a segmented GEMM output inside the destination buffer's batch item:
// identity, or - for a vertical strip of a token grid, pin > 0 - grid row m / pin, column m % pin of the strip, in a
// destination whose grid rows are pout tokens long (the caller's row offset selects the strip's first column).
__device__ __forceinline__ long long seg_pos(int m, int pin, int pout) {
  return pin > 0 ? (long long)(m / pin) * pout + (m % pin) : (long long)m;
}

// s / n where inv = 1 / n (rounded) is at hand: the product corrected by its remainder is the correctly rounded quotient (Markstein),
// in three dependent operations instead of some twenty.  An infinite product has no remainder.
__host__ __device__ inline double div_by(double s, double n, double inv) {
  const double q = s * inv, c = __builtin_fma(__builtin_fma(-q, n, s), inv, q);
  return __builtin_fabs(q) < __builtin_inf() ? c : q;
}

// 1 / sqrt(v) from a float estimate r: two Newton steps, the first leaves 3e-14, the second the rounding of double.
__host__ __device__ inline double rsqrt_from(double v, float est) {
  double r = (double)est;
  r = __builtin_fma(0.5 * r, __builtin_fma(-v * r, r, 1.0), r);
  return __builtin_fma(0.5 * r, __builtin_fma(-v * r, r, 1.0), r);
}

static inline int cdiv(long long a, long long b) { return (int)((a + b - 1) / b); }

}  // namespace df

#define DF_LAUNCH_CHECK()                          \
  do {                                             \
    if (hipGetLastError() != hipSuccess) return DF_EHIP; \
  } while (0)

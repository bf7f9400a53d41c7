// Small device helpers shared by the kernel files.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace d2o {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) double f64x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

// Storage element traits: float and bf16 (held as uint16_t).
template <typename T>
struct Elem;
template <>
struct Elem<float> {
  static __device__ __forceinline__ double to_f64(float x) { return double(x); }
  static __device__ __forceinline__ float to_f32(float x) { return x; }
  static __device__ __forceinline__ float from_f64(double x) { return float(x); }
  static __device__ __forceinline__ float from_f32(float x) { return x; }
};
template <>
struct Elem<uint16_t> {
  static __device__ __forceinline__ float to_f32(uint16_t x) { return __uint_as_float(uint32_t(x) << 16); }
  static __device__ __forceinline__ double to_f64(uint16_t x) { return double(to_f32(x)); }
  // fp64 -> bf16, round to nearest even, in one rounding (no detour through fp32 rounding):
  // bf16 keeps 7 of the 52 fraction bits; values are far from bf16's exponent limits.
  static __device__ __forceinline__ uint16_t from_f64(double x) {
    unsigned long long b = (unsigned long long)__double_as_longlong(x);
    const unsigned long long lsb = (b >> 45) & 1ull;
    b = (b + ((1ull << 44) - 1ull) + lsb) & ~((1ull << 45) - 1ull);
    const float f = float(__longlong_as_double((long long)b));  // exact: 8 significant bits
    return uint16_t(__float_as_uint(f) >> 16);
  }
  static __device__ __forceinline__ uint16_t from_f32(float x) {
    uint32_t b = __float_as_uint(x);
    b += 0x7FFFu + ((b >> 16) & 1u);
    return uint16_t(b >> 16);
  }
};

// ---- fp8 cache rows: d codes of the 8-bit format E4M3 (1 sign, 4 exponent bits with bias 7, 3
// fraction bits, subnormals, largest magnitude 448, no infinities) and one power of two per row;
// a row's values are code * 2^e.
template <>
struct Elem<uint8_t> {  // the code alone, without the row's power of two
  static __device__ __forceinline__ float to_f32(uint8_t x) { return __builtin_amdgcn_cvt_f32_fp8(int(x), 0); }
  static __device__ __forceinline__ double to_f64(uint8_t x) { return double(to_f32(x)); }
};
__device__ __forceinline__ double pow2_f64(int e) { return __hiloint2double((1023 + e) << 20, 0); }   // |e| < 1023
__device__ __forceinline__ float pow2_f32(int e) { return __uint_as_float(uint32_t(127 + e) << 23); }  // |e| < 127
// The row's exponent: the smallest e with amax * 2^-e <= 448 (448 = 0.875 * 2^9), not below -120
// (one signed byte holds it); 0 for an all-zero row.
__device__ __forceinline__ int fp8_row_exponent(double amax) {
  if (!(amax > 0.0)) return 0;
  int ex;
  const double fr = frexp(amax, &ex);
  return max((fr <= 0.875 ? ex - 9 : ex - 8), -120);
}
// y (|y| <= 448) to the nearest E4M3 value, ties to the even fraction; exact arithmetic throughout.
__device__ __forceinline__ uint8_t fp8_encode(double y) {
  const double ay = fabs(y);
  int ex;
  (void)frexp(ay, &ex);                       // ay in [2^(ex-1), 2^ex); ex = 0 for ay = 0
  const int E = max(ex - 1, -6);              // the subnormal range counts as binade -6
  const double q = ldexp(rint(ldexp(ay, 3 - E)), E - 3);
  if (q == 0.0) return 0;                     // (no negative zero)
  int eq;
  (void)frexp(q, &eq);
  const int Eq = eq - 1;                      // rounding may have carried into the next binade
  const uint32_t code = Eq < -6 ? uint32_t(ldexp(q, 9)) : (uint32_t(Eq + 7) << 3) | uint32_t(ldexp(q, 3 - Eq) - 8.0);
  return uint8_t(code | (y < 0.0 ? 0x80u : 0u));
}

// x / sqrt(D), rounded once: the product with the rounded reciprocal and one correction by its exact
// remainder (Markstein's theorem), with the instruction that ends a division for infinities and NaN: four instructions
// where the compiler's division, which does not use that the divisor is a constant, takes twelve.
template <int D>
__device__ __forceinline__ double div_root(double x) {
  const double root = sqrt(double(D)), inv = 1.0 / root;
  const double q = x * inv;
  return __builtin_amdgcn_div_fixup(fma(fma(-q, root, x), inv, q), root, x);
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ int wave_min(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o, 64));
  return v;
}

// Wavefront reductions on the data-parallel-primitive path (register-to-register lane
// permutations, no LDS round trip): four butterfly steps inside each row of 16 lanes, then the
// four row results are combined through scalar registers.  Every lane gets the result; the
// combination tree is fixed.
constexpr int kDppXor1 = 0xB1;         // quad_perm [1,0,3,2]
constexpr int kDppXor2 = 0x4E;         // quad_perm [2,3,0,1]
constexpr int kDppHalfMirror = 0x141;  // lane i <-> 7 - i within 8
constexpr int kDppMirror = 0x140;      // lane i <-> 15 - i within 16
constexpr int kDppRor4 = 0x124;        // lane i <- (i - 4) mod 16 within 16
constexpr int kDppRor8 = 0x128;        // lane i <-> i ^ 8 within 16
template <int CTRL>
__device__ __forceinline__ int dpp_i32(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true);
}
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const int lo = dpp_i32<CTRL>(__double2loint(v)), hi = dpp_i32<CTRL>(__double2hiint(v));
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double lane_f64(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                          __builtin_amdgcn_readlane(__double2loint(v), lane));
}
// The maximum as the instruction itself: fmax would first re-canonicalise values that were moved
// between lanes as bits (twice the instructions).  A NaN operand loses, as with fmax.
__device__ __forceinline__ double max_f64(double a, double b) {
  double r;
  asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
// Maximum over each row of 16 lanes; every lane of the row gets it.
__device__ __forceinline__ double row16_max(double v) {
  v = max_f64(v, dpp_f64<kDppXor1>(v));
  v = max_f64(v, dpp_f64<kDppXor2>(v));
  v = max_f64(v, dpp_f64<kDppHalfMirror>(v));
  return max_f64(v, dpp_f64<kDppMirror>(v));
}
// One lane's value to the next rows (0x142: lane 15 of a row to the row after it, 0x143: lane 31 to the upper
// half); lanes that receive nothing keep their own.
template <int CTRL>
__device__ __forceinline__ double row_bcast_f64(double v) {
  const int lo = __double2loint(v), hi = __double2hiint(v);
  return __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xF, 0xF, false),
                          __builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ double fast_wave_max(double v) {
  v = row16_max(v);
  v = max_f64(v, row_bcast_f64<0x142>(v));
  return lane_f64(max_f64(v, row_bcast_f64<0x143>(v)), 63);
}
__device__ __forceinline__ double fast_wave_sum(double v) {
  v += dpp_f64<kDppXor1>(v);
  v += dpp_f64<kDppXor2>(v);
  v += dpp_f64<kDppHalfMirror>(v);
  v += dpp_f64<kDppMirror>(v);
  return (lane_f64(v, 0) + lane_f64(v, 16)) + (lane_f64(v, 32) + lane_f64(v, 48));
}
__device__ __forceinline__ int fast_wave_min(int v) {
  v = min(v, dpp_i32<kDppXor1>(v));
  v = min(v, dpp_i32<kDppXor2>(v));
  v = min(v, dpp_i32<kDppHalfMirror>(v));
  v = min(v, dpp_i32<kDppMirror>(v));
  return min(min(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
             min(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

// Sum over each row of 16 lanes with the same four butterfly steps; every lane of the row gets
// the row's sum.
__device__ __forceinline__ double row16_sum(double v) {
  v += dpp_f64<kDppXor1>(v);
  v += dpp_f64<kDppXor2>(v);
  v += dpp_f64<kDppHalfMirror>(v);
  v += dpp_f64<kDppMirror>(v);
  return v;
}

// Sum over each half of the wavefront (32 lanes) by halves: lanes 16 apart first, then 8, 4, 2 and 1 apart
// (once lanes eight apart agree, a rotation by four reaches the lane four apart); every lane gets its half's sum.
template <typename F>
__device__ __forceinline__ F half_wave_sum(F v) {
  auto moved = [](auto ctrl, F x) {
    if constexpr (sizeof(F) == 8)
      return dpp_f64<decltype(ctrl)::value>(x);
    else
      return __int_as_float(dpp_i32<decltype(ctrl)::value>(__float_as_int(x)));
  };
  v += __shfl_xor(v, 16, 64);
  v += moved(std::integral_constant<int, kDppRor8>{}, v);
  v += moved(std::integral_constant<int, kDppRor4>{}, v);
  v += moved(std::integral_constant<int, kDppXor2>{}, v);
  v += moved(std::integral_constant<int, kDppXor1>{}, v);
  return v;
}

// v + the same of the lane 32 away (a register exchange between the halves, no LDS).
__device__ __forceinline__ double sum_halves(double v) {
  const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
  return __hiloint2double(int(hi[0]), int(lo[0])) + __hiloint2double(int(hi[1]), int(lo[1]));
}

// Workgroup barrier for exchanges through LDS only: it waits for the wavefront's LDS traffic,
// not for its outstanding global loads and stores (which __syncthreads would drain first).
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// A buffer descriptor over `bytes` bytes at p: a load through it whose lane offset is not below `bytes`
// touches no memory and returns zero.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* p, uint32_t bytes) {
  const uint64_t u = reinterpret_cast<uint64_t>(p);  // the same for all lanes, in scalar registers
  const uint64_t lo = uint32_t(__builtin_amdgcn_readfirstlane(int(uint32_t(u)))),
                 hi = uint32_t(__builtin_amdgcn_readfirstlane(int(uint32_t(u >> 32))));
  return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(lo | (hi << 32)), 0,
                                           __builtin_amdgcn_readfirstlane(int(bytes)), 0x00020000);
}
// 16 bytes per lane from memory straight into LDS: the wavefront's 64 chunks land at `dst` (the same
// for all lanes) one after the other, each lane choosing what it reads.  The whole displacement is
// the lane's: the instruction's scalar offset takes no part in the comparison with the buffer's size.
// Arrival is waited for with wait_vm<younger loads that may still be on their way>().
__device__ __forceinline__ void load_lds16(__amdgpu_buffer_rsrc_t src, uint32_t lane_off, uint16_t* dst) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(src, (__attribute__((address_space(3))) void*)dst, 16, int(lane_off), 0, 0, 0);
}
// The same from an address of each lane's own.
__device__ __forceinline__ void load_lds16(const void* src, uint16_t* dst) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                   (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
}
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "six bits");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// All LDS traffic of the wavefront done (as the intrinsic, so that the compiler knows it: vmcnt 63,
// expcnt 7, lgkmcnt 0).
__device__ __forceinline__ void wait_lgkm0() {
  __builtin_amdgcn_s_waitcnt(0xC07F);
  asm volatile("" ::: "memory");
}

// Deterministic block-wide sum (fixed tree): every thread gets the total.
// `buf` holds one double per wave; blockDim.x must be a multiple of 64 and <= 1024.
__device__ __forceinline__ double block_sum(double v, double* buf) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) buf[w] = v;
  __syncthreads();
  double t = 0.0;
  for (int i = 0; i < nw; ++i) t += buf[i];
  return t;
}

}  // namespace d2o

// Operands of the matrix-core kernels: FP32 values split into two FP16 numbers, packed in
// the lane order of v_mfma_f32_32x32x16_f16, and loads and stores of device memory.
#ifndef AIDG_MATRIX_COMMON_H
#define AIDG_MATRIX_COMMON_H

#include <hip/hip_runtime.h>

#include "device_common.h"
#include "subgrid_common.h"

namespace aidg {
namespace {

typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef _Float16 half8v __attribute__((ext_vector_type(8)));
typedef float acc16 __attribute__((ext_vector_type(16)));

// Eight FP16 values of one lane's matrix operand, as four packed pairs.
struct alignas(16) Frag {
  unsigned w[4];
};

__device__ __forceinline__ acc16 mfma(const Frag& a, const Frag& b, const acc16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8v, a), __builtin_bit_cast(half8v, b), c, 0,
                                                0, 0);
}
__device__ __forceinline__ unsigned pk_mul(unsigned a, unsigned b) {
  return __builtin_bit_cast(unsigned, __builtin_bit_cast(half2v, a) * __builtin_bit_cast(half2v, b));
}
__device__ __forceinline__ unsigned pk_mul_neg(unsigned a, unsigned b) {  // -a b
  return __builtin_bit_cast(unsigned, -__builtin_bit_cast(half2v, a) * __builtin_bit_cast(half2v, b));
}
// (x, y) -> (-y, x), and (x, y) -> (y b_low, x b_high): one packed multiplication each, which
// takes its operands' halves in any order (the compiler moves the swap behind it).
__device__ __forceinline__ unsigned swap_mul(unsigned p, unsigned b) {
  unsigned r;
  asm("v_pk_mul_f16 %0, %1, %2 op_sel:[1,0] op_sel_hi:[0,1]" : "=v"(r) : "v"(p), "v"(b));
  return r;
}
// The same, plus c, and minus c, fused.
__device__ __forceinline__ unsigned swap_fma(unsigned p, unsigned b, unsigned c) {
  unsigned r;
  asm("v_pk_fma_f16 %0, %1, %2, %3 op_sel:[1,0,0] op_sel_hi:[0,1,1]" : "=v"(r) : "v"(p), "v"(b), "v"(c));
  return r;
}
__device__ __forceinline__ unsigned swap_fma_sub(unsigned p, unsigned b, unsigned c) {
  unsigned r;
  asm("v_pk_fma_f16 %0, %1, %2, %3 op_sel:[1,0,0] op_sel_hi:[0,1,1] neg_lo:[0,0,1] neg_hi:[0,0,1]"
      : "=v"(r)
      : "v"(p), "v"(b), "v"(c));
  return r;
}
// (a + a_lo) (b + b_lo) as hi + lo: what rounding a b leaves is exact in FP16, and the two
// cross products are below 2^-11 of it.
__device__ __forceinline__ unsigned mul_rest(unsigned a, unsigned a_lo, unsigned b, unsigned b_lo, unsigned hi) {
  const half2v x = __builtin_bit_cast(half2v, a), y = __builtin_bit_cast(half2v, b);
  half2v r = __builtin_elementwise_fma(x, y, -__builtin_bit_cast(half2v, hi));
  r = __builtin_elementwise_fma(x, __builtin_bit_cast(half2v, b_lo), r);
  r = __builtin_elementwise_fma(__builtin_bit_cast(half2v, a_lo), y, r);
  return __builtin_bit_cast(unsigned, r);
}
__device__ __forceinline__ unsigned rot90(unsigned p) {
  unsigned r;
  asm("v_pk_mul_f16 %0, %1, %2 op_sel:[1,0] op_sel_hi:[0,1]" : "=v"(r) : "v"(p), "s"(0x3C00BC00u));  // (-1, 1)
  return r;
}
__device__ __forceinline__ Frag rot90(const Frag& f) {
  return {rot90(f.w[0]), rot90(f.w[1]), rot90(f.w[2]), rot90(f.w[3])};
}
constexpr unsigned kNegLow = 0x8000u;

// Loads and stores of device memory at a wave-uniform base and a lane's byte offset.  The
// pointers of a launch come out of memory, which leaves their address space unknown: without
// the casts these would be flat accesses, with 64-bit addresses per lane and an LDS wait each.
typedef float vec2 __attribute__((ext_vector_type(2)));
typedef float vec4 __attribute__((ext_vector_type(4)));
typedef vec4 vec4_of_2 __attribute__((aligned(8)));  // a caller's complex values: aligned as they are
#define AIDG_GLOBAL __attribute__((address_space(1)))
template <typename V>
__device__ __forceinline__ V gload(const void* base, unsigned off) {
  return *(const AIDG_GLOBAL V*)((const AIDG_GLOBAL char*)base + off);
}
template <typename V>
__device__ __forceinline__ void gstore(void* base, unsigned off, V v) {
  *(AIDG_GLOBAL V*)((AIDG_GLOBAL char*)base + off) = v;
}
// Byte offset of visibility (row, c) of a sub-table, whose rows are nc_total apart.  A
// sub-table of 2048 rows reaches 2^32 bytes from 65536 channels on, so it is 64 bits wide.
__device__ __forceinline__ int64_t vis_offset(int row, int c, int nc_total) {
  return ((int64_t)row * nc_total + c) * 32;
}

// (x, y) rounded to an FP16 pair (to nearest), and what it leaves of either (exact).
__device__ __forceinline__ unsigned cvt_pair(float x, float y) {
  const vec2 v = {x, y};
  unsigned r = __builtin_bit_cast(unsigned, __builtin_convertvector(v, half2v));
  asm("" : "+v"(r));  // one packed conversion: not formed again per element by what reads it
  return r;
}
// (v_fma_mix_f32, which the compiler does not form from the subtraction.  Its operand x may
// come from the transcendental unit, whose result a following instruction must not read at
// once; the conversion that made p has read it before.)
__device__ __forceinline__ float rest_low(float x, unsigned p) {
  float r;
  asm("v_fma_mix_f32 %0, -%1, 1.0, %2 op_sel_hi:[1,0,0]" : "=v"(r) : "v"(p), "v"(x));
  return r;
}
__device__ __forceinline__ float rest_high(float y, unsigned p) {
  float r;
  asm("v_fma_mix_f32 %0, -%1, 1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(p), "v"(y));
  return r;
}
// (x, y) as FP16 pairs hi + lo.
__device__ __forceinline__ void split(float x, float y, unsigned& hi, unsigned& lo) {
  hi = cvt_pair(x, y);
  lo = cvt_pair(rest_low(x, hi), rest_high(y, hi));
}
__device__ __forceinline__ unsigned pair_of(float x) {
  const half2v h = {(_Float16)x, (_Float16)x};
  return __builtin_bit_cast(unsigned, h);
}
__device__ __forceinline__ float pair_high(unsigned p) { return (float)__builtin_bit_cast(half2v, p).y; }

// Power of two that brings a largest component m to [2^9, 2^10), and its reciprocal (so
// that the low halves stay normal FP16 numbers down to 2^-23 of m); below 2^-117 to less, as
// the reciprocal is at least 2^-126: the smallest normal m to 1.  Infinities and NaNs stay
// what they are under either factor.
__device__ __forceinline__ void fit_scale(float m, float& scale, float& unscale) {
  int e = (int)((__float_as_uint(m) >> 23) & 255) - 127;
  e = max(-117, min(e, 127));
  scale = __uint_as_float((unsigned)(127 + 9 - e) << 23);
  unscale = __uint_as_float((unsigned)(127 - 9 + e) << 23);
}

__device__ __forceinline__ float inverse_power(float p) {  // of a power of two, 2^-126 to 2^126
  return __uint_as_float((254u << 23) - __float_as_uint(p));
}

// Largest of the wave's values (>= 0), by DPP: rotations within each row of 16 lanes, then
// the four rows.
__device__ __forceinline__ float wave_max(float m) {
  m = fmaxf(m, dpp<0x121>(m));
  m = fmaxf(m, dpp<0x122>(m));
  m = fmaxf(m, dpp<0x124>(m));
  m = fmaxf(m, dpp<0x128>(m));
  const int v = __float_as_int(m);
  return fmaxf(fmaxf(__int_as_float(__builtin_amdgcn_readlane(v, 0)), __int_as_float(__builtin_amdgcn_readlane(v, 16))),
               fmaxf(__int_as_float(__builtin_amdgcn_readlane(v, 32)), __int_as_float(__builtin_amdgcn_readlane(v, 48))));
}
// Largest of the values (>= 0) of the wave's lanes of the same parity, in each lane.
__device__ __forceinline__ float parity_max(float m) {
  m = fmaxf(m, dpp<0x122>(m));
  m = fmaxf(m, dpp<0x124>(m));
  m = fmaxf(m, dpp<0x128>(m));
  float n = m;
  swap16(m, n);
  m = n = fmaxf(m, n);
  swap32(m, n);
  return fmaxf(m, n);
}

// Visibilities per LDS block.
constexpr int kBlk = 32;

}  // namespace
}  // namespace aidg

#endif  // AIDG_MATRIX_COMMON_H

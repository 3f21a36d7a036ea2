// Vector types, matrix-core operand fragments and tile helpers shared by the
// kernels that build and use them (encode_kernels.hip, grad_kernels.hip).
#pragma once
#include "nfs_internal.h"

namespace nfs {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef __bf16 b8 __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef unsigned int u4 __attribute__((ext_vector_type(4)));

constexpr double kInv2Pi = 0.159154943091895335768883763372514362;

__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// e_b of the balancing power for term b, from the term maxima (identical on
// both sides and in every kernel that reads it)
__device__ __forceinline__ int term_shift(const unsigned* __restrict__ tmax, int b) {
  const float ma = __uint_as_float(tmax[b]) * (float)kInv2Pi;
  const float mh = __uint_as_float(tmax[kMaxTerms + b]);
  if (!(ma > 0.f) || !(mh > 0.f) || !isfinite(ma) || !isfinite(mh)) return 0;
  int ea, eh;
  frexpf(ma, &ea);
  frexpf(mh, &eh);
  return (ea - eh) / 2;
}

// One lane's 8 fragment values of (chunk ch, column block nb) in the layout
// of precision PREC (layouts: see pack_data in encode_kernels.hip).
template <int PREC>
__device__ __forceinline__ void store_fragment(const float (&vals)[8], void* __restrict__ out, int64_t ch, int nb,
                                               int NB, int lane) {
  if (PREC == PREC_FP32) {
    h8 hi, lo;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      hi[u] = (_Float16)vals[u];
      lo[u] = (_Float16)(vals[u] - (float)hi[u]);
    }
    ((h8*)out)[((ch * NB + nb) * 2 + 0) * 64 + lane] = hi;
    ((h8*)out)[((ch * NB + nb) * 2 + 1) * 64 + lane] = lo;
  } else if (PREC == PREC_FP16) {
    h8 h;
#pragma unroll
    for (int u = 0; u < 8; ++u) h[u] = (_Float16)vals[u];
    ((h8*)out)[(ch * NB + nb) * 64 + lane] = h;
  } else {
    b8 hi, lo;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      hi[u] = (__bf16)vals[u];
      lo[u] = (__bf16)(vals[u] - (float)hi[u]);
    }
    ((b8*)out)[((ch * NB + nb) * 2 + 0) * 64 + lane] = hi;
    ((b8*)out)[((ch * NB + nb) * 2 + 1) * 64 + lane] = lo;
  }
}

typedef __attribute__((address_space(3))) void lds_void;

// Phase tile on the f16 matrix cores: NQ chained 16x16x32 products.
template <int NQ>
__device__ __forceinline__ f4 phase_tile(const u4 (&ph)[NQ], const u4 (&hc)[NQ]) {
  f4 p = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int q = 0; q < NQ; ++q)
    p = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8, ph[q]), __builtin_bit_cast(h8, hc[q]), p, 0,
                                               0, 0);
  return p;
}

// Two-part f16 split of 8 float32 values: hi = f16(v), lo = f16(v - hi), the
// difference exact in one mixed-precision FMA that reads its half of the
// packed hi register.
__device__ __forceinline__ void split8(const float (&v)[8], h8& hi, h8& lo) {
  typedef _Float16 h2 __attribute__((ext_vector_type(2)));
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    h2 hp;
    hp[0] = (_Float16)v[2 * r];
    hp[1] = (_Float16)v[2 * r + 1];
    const unsigned hb = __builtin_bit_cast(unsigned, hp);
    float l0, l1;
    asm("v_fma_mix_f32 %0, -%1, 1.0, %2 op_sel_hi:[1,0,0]" : "=v"(l0) : "v"(hb), "v"(v[2 * r]));
    asm("v_fma_mix_f32 %0, -%1, 1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(l1) : "v"(hb), "v"(v[2 * r + 1]));
    hi[2 * r] = hp[0];
    hi[2 * r + 1] = hp[1];
    lo[2 * r] = (_Float16)l0;
    lo[2 * r + 1] = (_Float16)l1;
  }
}

// Whether the hardware sine and cosine take the phase directly: its bound
// sum_b max|a_b| max|h_b| (revolutions) stays below kRawPhaseBound; also
// false for NaN.  Whole waves.
__device__ __forceinline__ bool raw_phase(const unsigned* __restrict__ tmax, int T, int lane) {
  float bound = 0.f;
  if (lane < T) bound = __uint_as_float(tmax[lane]) * (float)kInv2Pi * __uint_as_float(tmax[kMaxTerms + lane]);
  for (int off = 32; off > 0; off >>= 1) bound += __shfl_xor(bound, off);
  return bound < kRawPhaseBound;
}

// XCD-aware order: block b of nblk goes to XCD b % 8 (round-robin dispatch);
// renumbering makes each XCD take a contiguous range of blocks, which share
// streamed chunks in that XCD's L2.
__device__ __forceinline__ int64_t xcd_order(int64_t b, int64_t nblk) {
  const int64_t per = nblk / 8;
  return b < per * 8 ? (b % 8) * per + b / 8 : b;
}

}  // namespace nfs

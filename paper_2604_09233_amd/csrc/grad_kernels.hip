// Gradient of the field coefficients in one pass (FP32 form).
//
// grad_kcoef[k][b] = Im sum_c G_c(k) conj((E (h_b o rho))_c(k)) needs E of P
// different images when the sum over coils is taken last.  Taking it first
// leaves one image-sized quantity per (sample, voxel) pair:
//   grad_kcoef[k][b] = sum_l h_b(l) w(k, l),
//   w(k, l) = Im(exp(-i phi(k, l)) D(k, l)),  D(k, l) = sum_c conj(S_c(l) rho(l)) G_c(k),
// so every pair is visited once: the phase tile and its sine and cosine as in
// the encode kernel, D as a contraction over the coils whose result has the
// phase tile's layout (streamed voxels x held samples), w on the VALU, and w
// (which is then the A operand of a product over voxels, in place) against
// the field values of 16 terms per column block.  All three products take
// two-part f16 operands, three matrix-core products each, like the FP32 form
// of the encode kernel; per 16 x 16 tile that is NQ + 6 NK + 1.5 NP
// matrix-core instructions and 8 transcendentals in place of P times the
// FP32 encode tile's NQ + 3 NB and 8.
#include <algorithm>

#include "fragment.h"

namespace nfs {

// Operand layouts (per lane g = lane / 16, n = lane % 16, slots e = 0..7,
// 16-byte vectors; part 0 = hi, 1 = lo; "kk" blocks of 16 coils):
//  voxels   q  [(chunk * NK + kk) * 2 + part][64]: voxel 16 chunk + n, coil
//           16 kk + 4 g + e / 2, re / im of S_c rho (e % 2), scaled per voxel;
//  samples  Gf [(tile * NK + kk) * 2 + part][64]: sample 16 tile + n, same
//           coils, (Gr, Gi), scaled per sample: the operand of Re D; that of
//           Im D, (Gi, -Gr), is the same words with their halves turned;
//  fields   hf [(pair * NP + np) * 2 + part][64]: term 16 np + n, voxel
//           32 pair + 16 (e / 4) + 4 g + e % 4, times the voxel's scale,
//           scaled per term.
// Every scale is a power of two that puts the largest magnitude just below
// 2^kTop.  The low f16 part ends at 2^-24, so values down to about 2^-16 of
// that largest one keep all their 22 bits: of the coils of one voxel, of the
// coils of one sample, and per term of h_b max_c |S_c rho|, which is what each
// term's image had when every term went through E by itself.  (One scale for
// the whole image and fields below 2 lost up to 10 bits of the high-order
// terms of an object near the centre, and of everything beside one bright
// voxel.)  w is scaled once more before its split: |D| <= 2 G 2^(2 kTop), so
// |w| 2^-(kTop + ceil(log2 G)) <= 2^(kTop + 1), half of f16's largest value.
// Sums over voxels stay below 2^(2 kTop + 1) L.
constexpr int kTop = 14;
constexpr int kNoExp = -(1 << 20);  // exponent of zero or of a value that is not finite
constexpr int kInfExp = 1 << 20;    // of a sample with an infinite gradient

__device__ __forceinline__ void store_split(const float (&v)[8], h8* out, int64_t block, int lane) {
  h8 hi, lo;
  split8(v, hi, lo);
  out[(block * 2 + 0) * 64 + lane] = hi;
  out[(block * 2 + 1) * 64 + lane] = lo;
}

__device__ __forceinline__ int top_exp(float mx) {  // mx < 2^top_exp
  if (!(mx > 0.f) || !isfinite(mx)) return kNoExp;
  int e;
  frexpf(mx, &e);
  return e;
}

__device__ __forceinline__ float pow2_below(float mx, int top) {  // largest 2^s with mx 2^s < 2^top
  const int e = top_exp(mx);
  if (e == kNoExp) return 1.f;
  const int s = top - e;
  return ldexpf(1.f, s > 100 ? 100 : (s < -100 ? -100 : s));
}

// largest |re|, |im| of S_c rho over the coils of voxel l
__device__ __forceinline__ float voxel_max(const float2* __restrict__ rho, const float2* __restrict__ sens, int64_t l,
                                           int64_t L, int G) {
  const float2 r = rho[l];
  float mx = 0.f;
#pragma unroll 8
  for (int c = 0; c < G; ++c) {
    const float2 v = cmul(sens[(int64_t)c * L + l], r);
    mx = fmaxf(mx, fmaxf(fabsf(v.x), fabsf(v.y)));
  }
  return mx;
}

// The samples' operand (i: lane index over tiles x NK x 64).
__device__ __forceinline__ void grad_pack_G(const float2* __restrict__ gm, int64_t K, int G, int NK, int64_t KC,
                                            int* __restrict__ ge, h8* __restrict__ out, int64_t i) {
  if (i >= KC * NK * 64) return;
  const int lane = (int)(i & 63), g = lane >> 4;
  const int64_t blk = i >> 6, k = blk / NK * kChunk + (lane & 15);
  const int kk = (int)(blk % NK);
  float mx = 0.f;
  if (k < K)
    for (int c = 0; c < G; ++c) {
      const float2 a = gm[(int64_t)c * K + k];
      mx = fmaxf(mx, fmaxf(fabsf(a.x), fabsf(a.y)));
    }
  // beside an infinite entry finite ones count for nothing: its sign goes
  // through (a split of infinity itself is not a number), the size is put back
  // at the end
  const bool inf = isinf(mx);
  const int e = inf ? kInfExp : top_exp(mx), s = inf || e == kNoExp ? 0 : kTop - e;
  auto entry = [&](float x) {
    return !inf || isnan(x) ? ldexpf(x, s) : isinf(x) ? copysignf(ldexpf(1.f, kTop - 1), x) : 0.f;
  };
  if (kk == 0 && g == 0) ge[k] = e;  // KC * 16 entries
  float v[8];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int c = kk * 16 + g * 4 + j;
    float2 a = make_float2(0.f, 0.f);
    if (k < K && c < G) a = gm[(int64_t)c * K + k];
    v[2 * j] = entry(a.x);
    v[2 * j + 1] = entry(a.y);
  }
  store_split(v, out, blk, lane);
}

// The first nem workgroups: ve[l] = exponent of max_c |S_c rho|; em[b][x] =
// workgroup x's largest exponent of |h_b| plus that of its voxel; the others
// pack the samples' operand, which needs none of it (4 us as a launch by
// itself).  Maxima in registers, reduced once: with an LDS atomic per voxel
// and term 36 us at 128x128, 16 coils, 16 terms, 11 now.
__global__ __launch_bounds__(256) void grad_range_pack_G_kernel(
    const float2* __restrict__ rho, const float2* __restrict__ sens, const float* __restrict__ fields, int64_t L, int G,
    int P, int nem, int* __restrict__ ve, int* __restrict__ em, const float2* __restrict__ gm, int64_t K, int NK,
    int64_t KC, int* __restrict__ ge, h8* __restrict__ gf) {
  if ((int)blockIdx.x >= nem) {
    grad_pack_G(gm, K, G, NK, KC, ge, gf, (int64_t)(blockIdx.x - nem) * 256 + threadIdx.x);
    return;
  }
  __shared__ int red[kWaves][kMaxTerms];
  int mx[kMaxTerms];
#pragma unroll
  for (int b = 0; b < kMaxTerms; ++b) mx[b] = kNoExp;
  for (int64_t l = (int64_t)blockIdx.x * 256 + threadIdx.x; l < L; l += (int64_t)nem * 256) {
    const int e = top_exp(voxel_max(rho, sens, l, L, G));
    ve[l] = e;
#pragma unroll
    for (int b = 0; b < kMaxTerms; ++b)
      if (b < P) {
        const int eh = top_exp(fabsf(fields[(int64_t)b * L + l]));
        mx[b] = max(mx[b], e == kNoExp || eh == kNoExp ? kNoExp : e + eh);
      }
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int b = 0; b < kMaxTerms; ++b)
    if (b < P) {
      for (int off = 32; off > 0; off >>= 1) mx[b] = max(mx[b], __shfl_xor(mx[b], off));
      if (lane == 0) red[wave][b] = mx[b];
    }
  __syncthreads();
  if ((int)threadIdx.x < P) {
    int m = red[0][threadIdx.x];
    for (int w = 1; w < kWaves; ++w) m = max(m, red[w][threadIdx.x]);
    em[threadIdx.x * nem + blockIdx.x] = m;
  }
}

// The voxels' operand (i: lane index over chunks x NK x 64).
__device__ __forceinline__ void grad_pack_q(const float2* __restrict__ rho, const float2* __restrict__ sens, int64_t L,
                                            int G, int NK, int64_t LC, const int* __restrict__ ve,
                                            h8* __restrict__ out, int64_t i) {
  if (i >= LC * NK * 64) return;
  const int lane = (int)(i & 63), g = lane >> 4;
  const int64_t blk = i >> 6, l = blk / NK * kChunk + (lane & 15);
  const int kk = (int)(blk % NK);
  const int e = l < L ? ve[l] : kNoExp, s = e == kNoExp ? 0 : kTop - e;
  float v[8];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int c = kk * 16 + g * 4 + j;
    float2 q = make_float2(0.f, 0.f);
    if (l < L && c < G) q = cmul(sens[(int64_t)c * L + l], rho[l]);
    v[2 * j] = ldexpf(q.x, s);
    v[2 * j + 1] = ldexpf(q.y, s);
  }
  store_split(v, out, blk, lane);
}

// The fields' operand (i: lane index over pairs x NP x 64); eb[b]: the
// exponent of term b's largest field value times voxel magnitude.
__device__ __forceinline__ void grad_pack_h(const float* __restrict__ fields, int64_t L, int P, int NP, int64_t npair,
                                            const int* __restrict__ ve, const int* eb, h8* __restrict__ out,
                                            int64_t i) {
  if (i >= npair * NP * 64) return;
  const int lane = (int)(i & 63), g = lane >> 4;
  const int64_t blk = i >> 6, pair = blk / NP;
  const int b = (int)(blk % NP) * 16 + (lane & 15);
  const int top = b < P ? eb[b] : kNoExp;
  float v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int64_t l = pair * 32 + (e >> 2) * 16 + g * 4 + (e & 3);
    const int s = l < L && top != kNoExp ? ve[l] : kNoExp;  // none: w is zero there, or nothing is finite
    v[e] = s == kNoExp ? 0.f : ldexpf(fields[(int64_t)b * L + l], s + kTop - top);
  }
  store_split(v, out, blk, lane);
}

// The first nh workgroups pack the fields, each with its own maxima of em (a
// few kB from the L2, against a launch that forms eb before this one), the
// others the voxels; the first one keeps eb for the finish.
__global__ __launch_bounds__(256) void grad_pack_hq_kernel(
    const float2* __restrict__ rho, const float2* __restrict__ sens, const float* __restrict__ fields, int64_t L, int G,
    int P, int NK, int NP, int64_t LC, int64_t npair, const int* __restrict__ ve, const int* __restrict__ em, int nem,
    int64_t nh, int* __restrict__ eb, h8* __restrict__ q, h8* __restrict__ hf) {
  if ((int64_t)blockIdx.x >= nh) {
    grad_pack_q(rho, sens, L, G, NK, LC, ve, q, (blockIdx.x - nh) * 256 + threadIdx.x);
    return;
  }
  __shared__ int top[kMaxTerms];
  for (int b = threadIdx.x >> 6; b < P; b += kWaves) {
    int mx = kNoExp;
    for (int x = threadIdx.x & 63; x < nem; x += 64) mx = max(mx, em[b * nem + x]);
    for (int off = 32; off > 0; off >>= 1) mx = max(mx, __shfl_xor(mx, off));
    if ((threadIdx.x & 63) == 0) {
      top[b] = mx;
      if (blockIdx.x == 0) eb[b] = mx;
    }
  }
  __syncthreads();
  grad_pack_h(fields, L, P, NP, npair, ve, top, hf, (int64_t)blockIdx.x * 256 + threadIdx.x);
}

// Grid (ceil(HC / (kWaves MT)), nsplit), held samples x streamed pairs of
// voxel chunks, staged through LDS and remapped to XCDs as in encode_kernel.
// 128x128, 60 000 samples, 16 coils, 16 terms: 553 us, matrix cores 43 %
// (1082 TFLOP/s), sines and cosines 18 % and the other VALU work 43 % of their
// peaks; no LDS conflicts.  They share the issue slots; w's factor is one of
// about eight VALU operations per value and is not seen in the time.
template <int NQ, int NK, int NP, int MT, bool FRACT>
__device__ __forceinline__ void grad_stream(const u4* __restrict__ strmcoef, const u4* __restrict__ q,
                                            const u4* __restrict__ hf, float wscale, int64_t p0, int64_t p1, int64_t LC,
                                            const u4 (&hc)[MT][NQ], const u4 (&gb)[MT][NK][2][2], f4 (&acc)[MT][NP],
                                            u4 (*stage)[(2 * NQ + 4 * NK + 2 * NP) * 64], int wave, int lane) {
  constexpr int kPh = 2 * NQ, kQ = 4 * NK, kBlk = kPh + kQ + 2 * NP;
  // a pair's blocks: phase parts of both chunks, q of both, field values; the
  // second chunk of the last pair may not exist and repeats the first (its
  // field values are zero)
  auto load = [&](int64_t pair, u4* dst) {
#pragma unroll
    for (int blk = wave; blk < kBlk; blk += kWaves) {
      const u4* src;
      if (blk < kPh) {
        const int64_t ch = 2 * pair + blk / NQ;
        src = strmcoef + ((ch < LC ? ch : LC - 1) * NQ + blk % NQ) * 64;
      } else if (blk < kPh + kQ) {
        const int64_t ch = 2 * pair + (blk - kPh) / (2 * NK);
        src = q + ((ch < LC ? ch : LC - 1) * (2 * NK) + (blk - kPh) % (2 * NK)) * 64;
      } else {
        src = hf + (pair * (2 * NP) + (blk - kPh - kQ)) * 64;
      }
      __builtin_amdgcn_global_load_lds((const void*)(src + lane), (lds_void*)(dst + blk * 64), 16, 0, 0);
    }
  };
  auto h = [](u4 v) { return __builtin_bit_cast(h8, v); };
  if (p0 < p1) load(p0, stage[0]);
  int buf = 0;
  for (int64_t pair = p0; pair < p1; ++pair) {
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (pair + 1 < p1) load(pair + 1, stage[buf ^ 1]);
    const u4* st = stage[buf];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      float w[8];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        u4 ph[NQ];
#pragma unroll
        for (int i = 0; i < NQ; ++i) ph[i] = st[(u * NQ + i) * 64 + lane];
        const f4 p = phase_tile<NQ>(ph, hc[mt]);
        f4 dr = {0.f, 0.f, 0.f, 0.f}, di = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < NK; ++kk) {
          const h8 qh = h(st[(kPh + (u * NK + kk) * 2) * 64 + lane]), ql = h(st[(kPh + (u * NK + kk) * 2 + 1) * 64 + lane]);
          dr = __builtin_amdgcn_mfma_f32_16x16x32_f16(ql, h(gb[mt][kk][0][0]), dr, 0, 0, 0);
          di = __builtin_amdgcn_mfma_f32_16x16x32_f16(ql, h(gb[mt][kk][1][0]), di, 0, 0, 0);
          dr = __builtin_amdgcn_mfma_f32_16x16x32_f16(qh, h(gb[mt][kk][0][1]), dr, 0, 0, 0);
          di = __builtin_amdgcn_mfma_f32_16x16x32_f16(qh, h(gb[mt][kk][1][1]), di, 0, 0, 0);
          dr = __builtin_amdgcn_mfma_f32_16x16x32_f16(qh, h(gb[mt][kk][0][0]), dr, 0, 0, 0);
          di = __builtin_amdgcn_mfma_f32_16x16x32_f16(qh, h(gb[mt][kk][1][0]), di, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float x = FRACT ? __builtin_amdgcn_fractf(p[r]) : p[r];
          w[4 * u + r] = (__builtin_amdgcn_cosf(x) * di[r] - __builtin_amdgcn_sinf(x) * dr[r]) * wscale;
        }
      }
      h8 wh, wl;
      split8(w, wh, wl);
#pragma unroll
      for (int np = 0; np < NP; ++np) {
        const h8 fh = h(st[(kPh + kQ + 2 * np) * 64 + lane]), fl = h(st[(kPh + kQ + 2 * np + 1) * 64 + lane]);
        f4 t = {0.f, 0.f, 0.f, 0.f};
        t = __builtin_amdgcn_mfma_f32_16x16x32_f16(wl, fh, t, 0, 0, 0);
        t = __builtin_amdgcn_mfma_f32_16x16x32_f16(wh, fl, t, 0, 0, 0);
        t = __builtin_amdgcn_mfma_f32_16x16x32_f16(wh, fh, t, 0, 0, 0);
        acc[mt][np] += t;
      }
    }
    buf ^= 1;
  }
}

template <int NQ, int NK, int NP, int MT>
__global__ __launch_bounds__(256) void grad_kcoef_fused_kernel(const u4* __restrict__ heldcoef,
                                                               const u4* __restrict__ strmcoef,
                                                               const u4* __restrict__ q, const u4* __restrict__ gf,
                                                               const u4* __restrict__ hf, float wscale, int64_t HC,
                                                               int64_t LC, int64_t npair, int64_t pps,
                                                               float* __restrict__ part,
                                                               const unsigned* __restrict__ tmax, int T) {
  __shared__ u4 stage[2][(2 * NQ + 4 * NK + 2 * NP) * 64];
  const int64_t b = xcd_order(blockIdx.x + (int64_t)gridDim.x * blockIdx.y, (int64_t)gridDim.x * gridDim.y);
  const int64_t bx = b % gridDim.x, split = b / gridDim.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t tile0 = (bx * kWaves + wave) * MT;
  const bool raw = raw_phase(tmax, T, lane);
  u4 hc[MT][NQ], gb[MT][NK][2][2];
  f4 acc[MT][NP];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int64_t tile = tile0 + mt < HC ? tile0 + mt : HC - 1;  // past the end: not written
#pragma unroll
    for (int i = 0; i < NQ; ++i) hc[mt][i] = heldcoef[(tile * NQ + i) * 64 + lane];
#pragma unroll
    for (int kk = 0; kk < NK; ++kk)
#pragma unroll
      for (int part = 0; part < 2; ++part) {
        const u4 v = gf[((tile * NK + kk) * 2 + part) * 64 + lane];
        gb[mt][kk][0][part] = v;
        gb[mt][kk][1][part] = ((v >> 16) | (v << 16)) ^ 0x80000000u;
      }
#pragma unroll
    for (int np = 0; np < NP; ++np) acc[mt][np] = f4{0.f, 0.f, 0.f, 0.f};
  }
  const int64_t p0 = split * pps, p1 = p0 + pps < npair ? p0 + pps : npair;
  if (raw) grad_stream<NQ, NK, NP, MT, false>(strmcoef, q, hf, wscale, p0, p1, LC, hc, gb, acc, stage, wave, lane);
  else grad_stream<NQ, NK, NP, MT, true>(strmcoef, q, hf, wscale, p0, p1, LC, hc, gb, acc, stage, wave, lane);
  const int g = lane >> 4, n = lane & 15;
  float* o = part + (size_t)split * (size_t)HC * 16 * (NP * 16);
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    if (tile0 + mt >= HC) continue;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int np = 0; np < NP; ++np)
        o[((tile0 + mt) * 16 + g * 4 + r) * (NP * 16) + np * 16 + n] = acc[mt][np][r];
  }
}

// out[k][b] = the split sums, unscaled: 2^sh carries w's factor and the three
// operands' kTop
__global__ __launch_bounds__(256) void grad_kcoef_finish_kernel(const float* __restrict__ part, int nsplit,
                                                                int64_t HC16, int NP, int sh,
                                                                const int* __restrict__ ge, const int* __restrict__ eb,
                                                                int64_t K, int P, float* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= K * P) return;
  const int64_t k = i / P;
  const int b = (int)(i - k * P), ncol = NP * 16;
  float v = 0.f;
  for (int s = 0; s < nsplit; ++s) v += part[((size_t)s * HC16 + k) * ncol + b];
  out[i] = ge[k] == kInfExp ? v * INFINITY : ldexpf(v, ge[k] + eb[b] + sh);
}

// ---------------------------------------------------------------------------
static int grad_nk(int G) { return G <= 16 ? 1 : G <= 32 ? 2 : 4; }
static int grad_np(int P) { return P <= 16 ? 1 : 2; }
// workgroups that take the voxels in grad_range_pack_G_kernel
static int grad_range_blocks(int64_t L) { return (int)std::min<int64_t>(cdiv(L, 256), kBmaxBlocks); }
// held tiles per wave: the samples' operands take 16 NK registers a tile
static int grad_mt(int G) { return grad_nk(G) <= 2 ? 2 : 1; }

GradShape grad_shape(int64_t K, int64_t L, int G, int P, int n_cu, size_t avail) {
  GradShape g{};
  const int64_t KC = cdiv(K, kChunk), LC = cdiv(L, kChunk);
  g.NK = grad_nk(G);
  g.NP = grad_np(P);
  g.npair = cdiv(LC, 2);
  auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
  g.o_q = 0;
  g.o_G = g.o_q + al((size_t)LC * g.NK * 2 * 1024);
  g.o_h = g.o_G + al((size_t)KC * g.NK * 2 * 1024);
  g.o_gs = g.o_h + al((size_t)g.npair * g.NP * 2 * 1024);
  g.o_ve = g.o_gs + al((size_t)KC * kChunk * 4);
  g.o_eb = g.o_ve + al((size_t)L * 4);
  g.o_em = g.o_eb + al(kMaxTerms * 4);
  g.o_part = g.o_em + al((size_t)P * grad_range_blocks(L) * 4);
  const size_t one = (size_t)KC * kChunk * g.NP * 16 * 4;  // a multiple of 256
  // about four workgroups per CU, at least 8 pairs each, inside the space the
  // E^H E workspace has anyway
  const int64_t gx = cdiv(KC, (int64_t)kWaves * grad_mt(G));
  const int64_t fit = avail > g.o_part && one ? (int64_t)((avail - g.o_part) / one) : 1;
  int64_t ns = gx > 0 ? cdiv((int64_t)4 * n_cu, gx) : 1;
  ns = std::max<int64_t>(1, std::min<int64_t>({ns, g.npair / 8, 64, fit}));
  g.pps = cdiv(g.npair, ns);
  g.nsplit = (int)std::max<int64_t>(1, g.pps > 0 ? cdiv(g.npair, g.pps) : 1);
  g.total = g.o_part + g.nsplit * one;
  return g;
}

template <int NQ>
static hipError_t launch_fused_nq(const GradShape& g, int G, const u4* held, const u4* strm, const char* ws, float wscale,
                                  int64_t KC, int64_t LC, float* part, const unsigned* tmax, int T, hipStream_t s) {
  const dim3 gr((unsigned)cdiv(KC, (int64_t)kWaves * grad_mt(G)), (unsigned)g.nsplit), bl(64 * kWaves);
  const u4 *q = (const u4*)(ws + g.o_q), *gf = (const u4*)(ws + g.o_G), *hf = (const u4*)(ws + g.o_h);
  switch (g.NK * 4 + g.NP) {
#define NFS_GRAD(nk, np, mt)                                                                                       \
  case nk * 4 + np:                                                                                                \
    hipLaunchKernelGGL((grad_kcoef_fused_kernel<NQ, nk, np, mt>), gr, bl, 0, s, held, strm, q, gf, hf, wscale, KC, LC, \
                       g.npair, g.pps, part, tmax, T);                                                              \
    break;
    NFS_GRAD(1, 1, 2)
    NFS_GRAD(1, 2, 2)
    NFS_GRAD(2, 1, 2)
    NFS_GRAD(2, 2, 2)
    NFS_GRAD(4, 1, 1)
    NFS_GRAD(4, 2, 1)
#undef NFS_GRAD
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_grad_kcoef_fused(const GradShape& g, const void* heldcoef, const void* strmcoef, const float2* rho,
                                   const float2* sens, const float* fields, const float2* grad_m, int64_t K, int64_t L,
                                   int G, int P, int NQ, const unsigned* tmax, void* ws, float* out, hipStream_t s) {
  if (K == 0 || P == 0) return hipSuccess;
  if (L == 0) return launch_fill_zero(out, K * P, s);
  const int64_t KC = cdiv(K, kChunk), LC = cdiv(L, kChunk);
  char* w = (char*)ws;
  int lg = 0;
  while ((1 << lg) < G) ++lg;
  const int wsh = kTop + lg;
  const float wscale = ldexpf(1.f, -wsh);
  int *ve = (int*)(w + g.o_ve), *em = (int*)(w + g.o_em), *eb = (int*)(w + g.o_eb), *ge = (int*)(w + g.o_gs);
  const int nem = grad_range_blocks(L);
  auto blocks = [](int64_t n) { return dim3((unsigned)cdiv(n, 256)); };
  hipLaunchKernelGGL(grad_range_pack_G_kernel, dim3((unsigned)(nem + cdiv(KC * g.NK * 64, 256))), dim3(256), 0, s, rho,
                     sens, fields, L, G, P, nem, ve, em, grad_m, K, g.NK, KC, ge, (h8*)(w + g.o_G));
  const int64_t nh = cdiv(g.npair * g.NP * 64, 256);
  hipLaunchKernelGGL(grad_pack_hq_kernel, dim3((unsigned)(nh + cdiv(LC * g.NK * 64, 256))), dim3(256), 0, s, rho, sens,
                     fields, L, G, P, g.NK, g.NP, LC, g.npair, ve, em, nem, nh, eb, (h8*)(w + g.o_q), (h8*)(w + g.o_h));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  float* part = (float*)(w + g.o_part);
  const u4 *held = (const u4*)heldcoef, *strm = (const u4*)strmcoef;
  e = NQ == 1   ? launch_fused_nq<1>(g, G, held, strm, w, wscale, KC, LC, part, tmax, P + 1, s)
      : NQ == 2 ? launch_fused_nq<2>(g, G, held, strm, w, wscale, KC, LC, part, tmax, P + 1, s)
      : NQ == 3 ? launch_fused_nq<3>(g, G, held, strm, w, wscale, KC, LC, part, tmax, P + 1, s)
                : hipErrorInvalidValue;
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(grad_kcoef_finish_kernel, blocks(K * P), dim3(256), 0, s, part, g.nsplit, KC * kChunk, g.NP,
                     wsh - 3 * kTop, ge, eb, K, P, out);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Several field terms per E launch (FP16 and BF16 forms).  The images
// h_b o rho of a group of terms go through E together as terms x coils
// virtual coils: the phase tiles and their sine and cosine, most of an E
// launch at up to 16 coils, are then shared by the group.  Every term keeps
// the operand it has alone (its own scale included).

// bmax[b][x] = workgroup x's maximum of |h_b| max_c |re|, |im| of S_c rho
__global__ __launch_bounds__(256) void grad_terms_absmax_kernel(const float2* __restrict__ rho,
                                                                const float2* __restrict__ sens,
                                                                const float* __restrict__ fields, int64_t L, int G,
                                                                int P, float* __restrict__ bmax) {
  __shared__ unsigned red[kMaxTerms];
  if (threadIdx.x < kMaxTerms) red[threadIdx.x] = 0u;
  __syncthreads();
  for (int64_t l = (int64_t)blockIdx.x * 256 + threadIdx.x; l < L; l += (int64_t)gridDim.x * 256) {
    const float mx = voxel_max(rho, sens, l, L, G);
    for (int b = 0; b < P; ++b) {
      const float v = fabsf(fields[(int64_t)b * L + l]) * mx;
      if (v > 0.f) atomicMax(&red[b], __float_as_uint(v));
    }
  }
  __syncthreads();
  if ((int)threadIdx.x < P) bmax[threadIdx.x * kBmaxBlocks + blockIdx.x] = __uint_as_float(red[threadIdx.x]);
}

// E operand (layout of pack_data, NB column blocks) of terms b0 .. b0 + n - 1:
// virtual coil j G + c holds S_c rho h_{b0 + j}
template <int PREC>
__global__ __launch_bounds__(256) void grad_terms_pack_kernel(const float2* __restrict__ rho,
                                                              const float2* __restrict__ sens,
                                                              const float* __restrict__ fields, int64_t L, int G,
                                                              int b0, int n, int NB, int64_t LC,
                                                              const float* __restrict__ bmax,
                                                              float* __restrict__ unscale, void* __restrict__ out) {
  __shared__ float scale[kMaxTerms];
  if (threadIdx.x < kMaxTerms) scale[threadIdx.x] = 1.f;
  if (PREC != PREC_BF16) {
    const int lane = threadIdx.x & 63;
    for (int j = threadIdx.x >> 6; j < n; j += kWaves) {
      float mx = 0.f;
      for (int x = lane; x < kBmaxBlocks; x += 64) mx = fmaxf(mx, bmax[(b0 + j) * kBmaxBlocks + x]);
      for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
      if (lane == 0) {
        scale[j] = pow2_below(mx, 14);
        if (blockIdx.x == 0) unscale[j] = 1.f / scale[j];
      }
    }
  }
  __syncthreads();
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= LC * NB * 64) return;
  const int lane = (int)(i & 63), g = lane >> 4;
  const int64_t q = i >> 6, ch = q / NB;
  const int nb = (int)(q % NB), N = nb * 16 + (lane & 15), v = N >> 1, reim = N & 1;
  const int j = v / G, c = v - j * G;
  float vals[8];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int64_t l = ch * kChunk + g * 4 + k;
    float2 x = make_float2(0.f, 0.f);
    if (l < L && j < n) {
      x = cmul(sens[(int64_t)c * L + l], rho[l]);
      const float w = fields[(int64_t)(b0 + j) * L + l] * scale[j];
      x.x *= w;
      x.y *= w;
    }
    vals[2 * k] = reim ? x.y : x.x;
    vals[2 * k + 1] = reim ? x.x : -x.y;
  }
  store_fragment<PREC>(vals, out, ch, nb, NB, lane);
}

// out[k][b0 + j] = Im sum_c G_c(k) conj(Z_jc(k)) from the group's E partials
// (16 samples per workgroup, turned through LDS; coils added in order)
__global__ __launch_bounds__(256) void grad_terms_finish_kernel(const float* __restrict__ epart, int nsplit,
                                                                int64_t HC16, int NB, const float* __restrict__ unscale,
                                                                const float2* __restrict__ grad_m, int64_t K, int G,
                                                                int P, int b0, int n, float* __restrict__ out) {
  constexpr int kRows = 16;
  __shared__ float tile[64][kRows + 1];
  const int64_t k0 = (int64_t)blockIdx.x * kRows;
  const int nc = NB * 8;
  for (int i = threadIdx.x; i < kRows * nc; i += 256) {
    const int r = i / nc, v = i - r * nc;
    if (v >= n * G || k0 + r >= K) continue;
    const float2 z = sum_strided((const float2*)epart + (k0 + r) * nc + v, nsplit, HC16 * nc);
    const float2 g = grad_m[(int64_t)(v % G) * K + k0 + r];
    tile[v][r] = g.y * z.x - g.x * z.y;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kRows * n; i += 256) {
    const int r = i / n, j = i - r * n;
    if (k0 + r >= K) continue;
    float acc = 0.f;
    for (int c = 0; c < G; ++c) acc += tile[j * G + c][r];
    out[(k0 + r) * P + b0 + j] = acc * (unscale ? unscale[j] : 1.f);
  }
}

GradTerms grad_terms(int prec, int64_t KC, int64_t LC, int G, int P, int nsplit, int n_cu, size_t avail) {
  GradTerms t{};
  auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
  for (int n = std::min(64 / G, P); n > 1; --n) {
    t.n = n;
    t.NB = col_blocks(n * G);
    t.MT = t.NB <= 4 ? 4 : 2;
    t.o_bmax = 0;
    t.o_unscale = al((size_t)kMaxTerms * kBmaxBlocks * 4);
    t.o_data = t.o_unscale + 256;
    t.o_part = t.o_data + al((size_t)LC * t.NB * data_chunk_bytes(prec));
    const size_t one = (size_t)KC * kChunk * t.NB * 16 * 4;
    if (avail < t.o_part + one) continue;
    // as many splits as a single term's launch where they fit; fewer are
    // fine while there are four workgroups per CU
    const int64_t gx = cdiv(KC, (int64_t)kWaves * t.MT);
    const int64_t fit = (int64_t)((avail - t.o_part) / one);
    t.nsplit = (int)std::min<int64_t>(nsplit, fit);
    if (t.nsplit < nsplit && gx * t.nsplit < 4LL * n_cu) continue;
    return t;
  }
  t.n = 1;
  return t;
}

hipError_t launch_grad_terms_absmax(const GradTerms& t, const float2* rho, const float2* sens, const float* fields,
                                    int64_t L, int G, int P, char* ws, hipStream_t s) {
  hipLaunchKernelGGL(grad_terms_absmax_kernel, dim3(kBmaxBlocks), dim3(256), 0, s, rho, sens, fields, L, G, P,
                     (float*)(ws + t.o_bmax));
  return hipGetLastError();
}

hipError_t launch_grad_terms_pack(int prec, const GradTerms& t, const float2* rho, const float2* sens,
                                  const float* fields, int64_t L, int G, int b0, int n, char* ws, hipStream_t s) {
  const int64_t LC = cdiv(L, kChunk);
  const dim3 gr((unsigned)cdiv(LC * t.NB * 64, 256)), bl(256);
  const float* bmax = (const float*)(ws + t.o_bmax);
  float* un = (float*)(ws + t.o_unscale);
  if (prec == PREC_BF16)
    hipLaunchKernelGGL(grad_terms_pack_kernel<PREC_BF16>, gr, bl, 0, s, rho, sens, fields, L, G, b0, n, t.NB, LC, bmax,
                       un, ws + t.o_data);
  else
    hipLaunchKernelGGL(grad_terms_pack_kernel<PREC_FP16>, gr, bl, 0, s, rho, sens, fields, L, G, b0, n, t.NB, LC, bmax,
                       un, ws + t.o_data);
  return hipGetLastError();
}

hipError_t launch_grad_terms_finish(int prec, const GradTerms& t, const float2* grad_m, int64_t K, int G, int P, int b0,
                                    int n, char* ws, float* out, hipStream_t s) {
  const int64_t KC = cdiv(K, kChunk);
  hipLaunchKernelGGL(grad_terms_finish_kernel, dim3((unsigned)KC), dim3(256), 0, s, (const float*)(ws + t.o_part),
                     t.nsplit, KC * kChunk, t.NB, prec == PREC_BF16 ? nullptr : (const float*)(ws + t.o_unscale), grad_m,
                     K, G, P, b0, n, out);
  return hipGetLastError();
}

}  // namespace nfs

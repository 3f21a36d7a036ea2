// k-space filter of the reconstructed image (Methods, "Computation of
// k-space filters"; last line of both reconstruction listings):
// rho_f = IFFT(FFT(rho) o f).  The multidimensional DFT is separable, so it
// is applied one axis at a time: a pass along an axis of length n maps every
// line of the grid along that axis through the n-point DFT, n complex
// multiply-adds per output.  Forward passes over all axes, the filter (and
// 1/L) with the last forward pass, then the inverse passes.  L (nx + ny + nz)
// multiply-adds per direction instead of the L^2 of the grid's full DFT
// matrix.
#include <algorithm>

#include "nfs_internal.h"

namespace nfs {

// One DFT pass along one axis of a complex array viewed as [outer][n][inner]
// (inner = 1: the axis is the contiguous one):
//   out[o][j][i] = scale * g[o][j][i] * sum_k in[o][k][i] exp(sign 2 pi i j k / n)
// with g = f (the filter, [L] in the array's own index order) or 1.
// A workgroup takes W columns (W consecutive inner indices of one o, or W
// consecutive lines when inner = 1) and J output rows j0 .. j0 + J - 1
// (blockIdx.y), stages the columns' n x W input block in LDS with loads that
// are contiguous across the columns (strided axes) or along each line
// (contiguous axis), and the n twiddle factors, computed in double
// precision.  Thread (j, c) forms one output with consecutive threads on
// consecutive columns, summing in float32 in order of k.
__global__ __launch_bounds__(256) void dft_axis_kernel(const float2* __restrict__ in, float2* __restrict__ out,
                                                       int64_t outer, int n, int64_t inner, int W, int J, int sign,
                                                       float scale, const float* __restrict__ f) {
  extern __shared__ float2 lds[];
  float2* tw = lds;                  // [n]
  float2* blk = lds + n;             // [n][W] inputs
  float2* ob = blk + (size_t)n * W;  // contiguous axis only: [J][W + 1] results
  for (int k = threadIdx.x; k < n; k += blockDim.x) {
    double s, c;
    sincospi(2.0 * (double)k / (double)n, &s, &c);
    tw[k] = make_float2((float)c, (float)(sign * s));
  }
  // columns of this workgroup: W lines from c0 (contiguous axis) or W inner
  // indices from c0 of line group o (strided axes)
  int64_t o = 0, c0, ncol;
  if (inner == 1) {
    c0 = (int64_t)blockIdx.x * W;
    ncol = outer - c0 < W ? outer - c0 : W;
  } else {
    const int64_t per = (inner + W - 1) / W;
    o = (int64_t)blockIdx.x / per;
    c0 = ((int64_t)blockIdx.x % per) * W;
    ncol = inner - c0 < W ? inner - c0 : W;
  }
  const int j0 = blockIdx.y * J;
  const int nj = n - j0 < J ? n - j0 : J;
  auto addr = [&](int k, int c) -> int64_t {
    return inner == 1 ? (c0 + c) * (int64_t)n + k : (o * (int64_t)n + k) * inner + c0 + c;
  };
  // loads: consecutive threads along each line (contiguous axis) or across
  // the columns (strided axes), i.e. contiguous in memory either way
  const int total = n * W;
  for (int e = threadIdx.x; e < total; e += blockDim.x) {
    int k, c;
    if (inner == 1) {
      c = e / n;
      k = e - c * n;
    } else {
      k = e / W;
      c = e - k * W;
    }
    blk[k * W + c] = c < ncol ? in[addr(k, c)] : make_float2(0.f, 0.f);
  }
  __syncthreads();
  const int nout = J * W;
  for (int e = threadIdx.x; e < nout; e += blockDim.x) {
    const int jj = e / W, c = e - jj * W;
    if (c >= ncol || jj >= nj) continue;
    const int j = j0 + jj;
    float re = 0.f, im = 0.f;
    int idx = 0;  // (j k) mod n
    for (int k = 0; k < n; ++k) {
      const float2 x = blk[k * W + c], w = tw[idx];
      re = fmaf(x.x, w.x, re);
      re = fmaf(-x.y, w.y, re);
      im = fmaf(x.x, w.y, im);
      im = fmaf(x.y, w.x, im);
      idx += j;
      if (idx >= n) idx -= n;
    }
    if (inner == 1) {
      ob[jj * (W + 1) + c] = make_float2(re, im);
    } else {
      const int64_t a = addr(j, c);
      const float g = f ? f[a] * scale : scale;
      out[a] = make_float2(re * g, im * g);
    }
  }
  if (inner != 1) return;
  // contiguous axis: results leave along each line, as they came in
  __syncthreads();
  for (int e = threadIdx.x; e < nout; e += blockDim.x) {
    const int c = e / J, jj = e - c * J;
    if (c >= ncol || jj >= nj) continue;
    const int64_t a = addr(j0 + jj, c);
    const float g = f ? f[a] * scale : scale;
    const float2 v = ob[jj * (W + 1) + c];
    out[a] = make_float2(v.x * g, v.y * g);
  }
}

// The same pass for n = n1 n2 as two short sums per output, and (MID) the
// forward pass of the last axis, the filter and the inverse pass of the same
// axis in one: with k = k1 n2 + k2 and j = j1 + n1 j2
//   A[j1][k2] = w^(j1 k2) sum_k1 x[k1 n2 + k2] w^(n2 j1 k1),
//   X[j] = sum_k2 A[j1][k2] w^(n1 j2 k2),   w = exp(sign 2 pi i / n).
// A workgroup holds all n rows of its W = 2^lw columns, twice, in LDS, rows
// apart by an odd number of values, so that loads along a line (contiguous
// axis) meet no bank conflict; A's groups of n2 rows are p.pitch rows apart, so
// that the second sum's do not either (n = 2048 = 32 x 64, one column a
// workgroup: a call on 4x2048x4 169 -> 81 us, direct sums 180; on 2048x4x4
// 169 -> 79, direct 152).  The direct sums above read LDS 2 n times per
// output, which bounds them; these read it 2 (n1 + n2) times.  All reads of a
// workgroup's columns come before its writes: in == out is allowed.
// 96 x 96 x 48: the call 80 -> 45.5 us, error against 64 bits 5.7e-7 ->
// 2.6e-7, a pass 14.9 -> 9.6 us (the middle two together 12.6; both at half
// as many workgroups as now).  Its 7 MB take 1.5 us at the rate of a copy; the
// rest is the chain of load, two sums and store.  Loads before the twiddles
// rather than after them: 50.0 -> 47.5 us.
// magic m of d: x / d = (x m) >> 32 for x < 2^16 (x m of 64 bits).
__device__ __forceinline__ int div_magic(int x, unsigned m, int d) { return d == 1 ? x : (int)__umulhi((unsigned)x, m); }

__device__ __forceinline__ void dft_two_factors(const float2* tw, float2* a, float2* b, const DftPlan& p, int S,
                                                float sg) {
  const int n = p.n, n1 = p.n1, n2 = p.n2, pad = p.pitch - n2, nout = n << p.lw, cm = (1 << p.lw) - 1;
  for (int e = threadIdx.x; e < nout; e += blockDim.x) {
    const int c = e & cm, r = e >> p.lw, j1 = div_magic(r, p.m2, n2), k2 = r - j1 * n2;
    float re = 0.f, im = 0.f;
    int idx = 0;
    const float2* x = a + k2 * S + c;
#pragma unroll 4
    for (int k1 = 0; k1 < n1; ++k1) {
      const float2 v = x[k1 * n2 * S], w = tw[idx];
      const float wy = sg * w.y;
      re = fmaf(v.x, w.x, re);
      re = fmaf(-v.y, wy, re);
      im = fmaf(v.x, wy, im);
      im = fmaf(v.y, w.x, im);
      idx += n2 * j1;
      if (idx >= n) idx -= n;
    }
    const float2 w = tw[j1 * k2];
    const float wy = sg * w.y;
    b[(r + j1 * pad) * S + c] = make_float2(fmaf(re, w.x, -im * wy), fmaf(re, wy, im * w.x));
  }
  __syncthreads();
  for (int e = threadIdx.x; e < nout; e += blockDim.x) {
    const int c = e & cm, r = e >> p.lw, j2 = div_magic(r, p.m1, n1), j1 = r - j2 * n1;
    float re = 0.f, im = 0.f;
    int idx = 0;
    const float2* x = b + j1 * p.pitch * S + c;
#pragma unroll 4
    for (int k2 = 0; k2 < n2; ++k2) {
      const float2 v = x[k2 * S], w = tw[idx];
      const float wy = sg * w.y;
      re = fmaf(v.x, w.x, re);
      re = fmaf(-v.y, wy, re);
      im = fmaf(v.x, wy, im);
      im = fmaf(v.y, w.x, im);
      idx += n1 * j2;
      if (idx >= n) idx -= n;
    }
    a[r * S + c] = make_float2(re, im);
  }
  __syncthreads();
}

template <bool MID>
__global__ __launch_bounds__(256) void dft_two_kernel(const float2* in, float2* out, int64_t outer, int64_t inner,
                                                      DftPlan p, int sign, float scale,
                                                      const float* __restrict__ f) {
  extern __shared__ float2 lds[];
  const int n = p.n, W = 1 << p.lw, S = W | 1;
  float2* tw = lds;             // [n]
  float2* a = lds + n;          // [n][S]
  float2* b = a + (size_t)n * S;  // [n1][pitch][S]
  int64_t base, ncol;
  if (inner == 1) {
    base = (int64_t)blockIdx.x * W;
    ncol = outer - base < W ? outer - base : W;
    base *= n;
  } else {
    const int64_t per = (inner + W - 1) / W, o = (int64_t)blockIdx.x / per;
    const int64_t c0 = ((int64_t)blockIdx.x - o * per) * W;
    ncol = inner - c0 < W ? inner - c0 : W;
    base = o * (int64_t)n * inner + c0;
  }
  // element e of the block, in memory order -> row k, column c
  auto place = [&](int e, int& k, int& c) -> int64_t {
    if (inner == 1) {
      c = div_magic(e, p.m, n);
      k = e - c * n;
      return base + e;
    }
    k = e >> p.lw;
    c = e & (W - 1);
    return base + (int64_t)k * inner + c;
  };
  const int total = n << p.lw;
  // the twiddle factors (double precision) are formed while the first four
  // loads of each thread are under way
  float2 first[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int e = threadIdx.x + u * 256;
    int k, c;
    const int64_t at = place(e, k, c);
    first[u] = e < total && c < ncol ? in[at] : make_float2(0.f, 0.f);
  }
  for (int k = threadIdx.x; k < n; k += blockDim.x) {
    double s, c;
    sincospi(2.0 * (double)k / (double)n, &s, &c);
    tw[k] = make_float2((float)c, (float)s);
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int e = threadIdx.x + u * 256;
    int k, c;
    place(e, k, c);
    if (e < total) a[k * S + c] = first[u];
  }
  for (int e = threadIdx.x + 1024; e < total; e += 256) {
    int k, c;
    const int64_t at = place(e, k, c);
    a[k * S + c] = c < ncol ? in[at] : make_float2(0.f, 0.f);
  }
  __syncthreads();
  dft_two_factors(tw, a, b, p, S, (float)sign);
  if (MID) {
    for (int e = threadIdx.x; e < total; e += blockDim.x) {
      int k, c;
      const int64_t at = place(e, k, c);
      if (c >= ncol) continue;
      const float g = f[at] * scale;
      a[k * S + c].x *= g;
      a[k * S + c].y *= g;
    }
    __syncthreads();
    dft_two_factors(tw, a, b, p, S, -(float)sign);
  }
  for (int e = threadIdx.x; e < total; e += blockDim.x) {
    int k, c;
    const int64_t at = place(e, k, c);
    if (c < ncol) out[at] = a[k * S + c];
  }
}

// out = rho * f * scale elementwise (the filter of a single-bin grid)
__global__ void filter_scale_kernel(const float2* __restrict__ in, float2* __restrict__ out, const float* f,
                                    float scale, int64_t L) {
  const int64_t l = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (l >= L) return;
  const float g = f[l] * scale;
  out[l] = make_float2(in[l].x * g, in[l].y * g);
}

// Tiling of a pass: J output rows (32, or n if shorter) times W columns per
// workgroup, W * J <= 256 (one output per thread), W limited so that the
// twiddles, the n x W input block and, for the contiguous axis, the
// J x (W + 1) results fit in 64 KiB of LDS (n <= kMaxDftAxis = 2048).
static void dft_axis_tiling(int n, bool contiguous, int* W, int* J) {
  const int j = n < 32 ? n : 32;
  int w = 256 / j;
  const int slots = 65536 / 8 - n;  // float2 slots left after the twiddles
  while (w > 1 && n * w + (contiguous ? j * (w + 1) : 0) > slots) --w;
  *W = w;
  *J = j;
}

hipError_t launch_dft_axis(const float2* in, float2* out, int64_t outer, int n, int64_t inner, int sign, float scale,
                           const float* f, hipStream_t s) {
  const bool contiguous = inner == 1;
  int W, J;
  dft_axis_tiling(n, contiguous, &W, &J);
  const int64_t blocks = contiguous ? cdiv(outer, W) : outer * cdiv(inner, W);
  if (blocks == 0) return hipSuccess;
  const size_t lds = ((size_t)n + (size_t)n * W + (contiguous ? (size_t)J * (W + 1) : 0)) * sizeof(float2);
  hipLaunchKernelGGL(dft_axis_kernel, dim3((unsigned)blocks, (unsigned)cdiv(n, J)), dim3(256), lds, s, in, out, outer,
                     n, inner, W, J, sign, scale, f);
  return hipGetLastError();
}

// Two factors nearest the root of n, and the columns of a workgroup: 16, fewer
// until the pass has 1024 workgroups (calls of 96x96x48 / 219x219x22 at 256,
// 512, 1024 and 2048: 57.9, 47.3, 46.0, 49.8 / 242, 166, 144, 142 us), but no
// fewer than leave half the threads an output.
// The rule: they are taken where they save half the direct sum's terms and one column's outputs,
// in turns of a workgroup's 256 threads, take no more terms than the direct
// kernel's one output per thread (few columns and a long axis such as 3 x 677).
DftPlan dft_plan(int n, int64_t outer, int64_t inner) {
  DftPlan p{};
  p.n = n;
  p.n1 = 1;
  for (int d = 2; d * d <= n; ++d)
    if (n % d == 0) p.n1 = d;
  p.n2 = n / p.n1;
  const int64_t sum = p.n1 + p.n2;
  p.two = 2 * sum <= n && cdiv(n, 256) * sum <= n;
  auto blocks = [&] { return inner == 1 ? cdiv(outer, (int64_t)1 << p.lw) : outer * cdiv(inner, (int64_t)1 << p.lw); };
  auto slots = [&](int pitch) { return n + (n + (int64_t)p.n1 * pitch) * ((1 << p.lw) | 1); };
  constexpr int kSlots = 65536 / 8;
  p.lw = 4;
  while (p.lw > 0 && (slots(p.n2) > kSlots || (blocks() < 1024 && (n << p.lw) > 256))) --p.lw;
  // rows between the groups of A: up to three more than n2, the fewest with the
  // least 8-byte reads of 32 lanes (columns, then j1) on one of 32 banks
  p.pitch = p.n2;
  for (int q = p.n2, least = 33; p.two && q < p.n2 + 4 && slots(q) <= kSlots && least > 1; ++q) {
    int hits[32] = {}, worst = 0;
    for (int i = 0; i < 32 && (i >> p.lw) < p.n1; ++i)
      worst = std::max(worst, ++hits[((i >> p.lw) * q * ((1 << p.lw) | 1) + (i & ((1 << p.lw) - 1))) % 32]);
    if (worst < least) {
      least = worst;
      p.pitch = q;
    }
  }
  auto magic = [](int d) { return (unsigned)((((uint64_t)1 << 32) + d - 1) / d); };  // d >= 2 where used
  p.m = magic(n);
  p.m1 = magic(p.n1);
  p.m2 = magic(p.n2);
  p.blocks = blocks();
  p.lds = (size_t)slots(p.pitch) * 8;
  return p;
}

hipError_t launch_dft_two(const float2* in, float2* out, int64_t outer, int64_t inner, const DftPlan& p, int sign,
                          float scale, const float* f, hipStream_t s) {
  if (p.blocks == 0) return hipSuccess;
  const dim3 gr((unsigned)p.blocks), bl(256);
  if (f) hipLaunchKernelGGL(dft_two_kernel<true>, gr, bl, p.lds, s, in, out, outer, inner, p, sign, scale, f);
  else hipLaunchKernelGGL(dft_two_kernel<false>, gr, bl, p.lds, s, in, out, outer, inner, p, sign, scale, f);
  return hipGetLastError();
}

hipError_t launch_filter_scale(const float2* in, float2* out, const float* f, float scale, int64_t L, hipStream_t s) {
  if (L == 0) return hipSuccess;
  hipLaunchKernelGGL(filter_scale_kernel, dim3((unsigned)cdiv(L, 256)), dim3(256), 0, s, in, out, f, scale, L);
  return hipGetLastError();
}

}  // namespace nfs

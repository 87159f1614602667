// Optional per-step diagnostics of the Orth-Dion step and the rank-change helper, as HIP
// kernels for gfx950.  All of them are bandwidth-trivial next to the step itself; they favour
// accuracy (fp64 accumulation of sums of squares) and determinism (fixed reduction trees).
//
// Quantities (paper notation in brackets):
//   ||B||_F, ||G||_F, ||M_prev||_F      buffer, gradient, residual norms     (App. J)
//   ||R||_F = ||P^T B||_F               captured energy                      (Alg. 1 line 3)
//   tracking error                      sqrt(||B||^2 - ||R||^2) / ||B||      (Sec. 4.3; P orthonormal)
//   residual ratio                      ||M_prev|| / ||G||   [R-norm ratio]  (Sec. 6.3)
//   inner product <B, P Q^T>            trace of the triangular factor of R (QR, Lemma 4.2),
//                                       sum of column lengths of R (ColNorm)
//   nu = sigma_1(Q)                     dual-norm factor                     (Prop. 3.1, Lemma 4.1)
//   estimated effective rank            exp(entropy of normalised column lengths of R)  (App. B.2)
#include "od_kernels.h"

#include "od_common.h"
#include "od_gemm.h"

namespace od {

#define OD_CHECK_LAUNCH()                       \
  do {                                          \
    hipError_t e_ = hipGetLastError();          \
    if (e_ != hipSuccess) return e_;            \
  } while (0)

// Sum over the workgroup (256 threads) of one double per thread; result valid in thread 0.
OD_DEV double block_sum_256(double v, double* red) {
  const int tid = threadIdx.x;
  __syncthreads();
  red[tid] = v;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (tid < w) red[tid] += red[tid + w];
    __syncthreads();
  }
  return red[0];
}

// ------------------------------------------------------------------------------------
// sums of squares of M_prev, G and B = M_prev + G, one partial triple per workgroup
// ------------------------------------------------------------------------------------
// One wave per row at a time, four rows per workgroup: addresses advance without a division, and up to
// kDiagBlocks workgroups keep enough loads in flight for the memory system (2048 x 5632: 44 us with a 64-bit division per four
// elements and 128 workgroups, 15 us like this: 4.8 TB/s, the rate of a large copy).
template <bool GBF>
__global__ __launch_bounds__(256) void k_diag_norms(ClassDims d, const MatEntry* mats, double* dpart) {
  const int z = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
  double sm = 0.0, sg = 0.0, sb = 0.0;
  for (int i = (int)blockIdx.x * 4 + (tid >> 6); i < d.m; i += (int)gridDim.x * 4) {
    const float* mp = mats[z].M + (int64_t)i * d.ldm;
    const char* gp = reinterpret_cast<const char*>(mats[z].G) + (int64_t)i * d.ldg * (GBF ? 2 : 4);
#pragma unroll 2
    for (int j = lane * 4; j < d.n; j += 256) {
      const f32x4 mv = *reinterpret_cast<const f32x4*>(mp + j);
      float g[4];
      if constexpr (GBF) {
        const u32x2 raw = *reinterpret_cast<const u32x2*>(gp + j * 2);
        g[0] = bf16_lo(raw[0]); g[1] = bf16_hi(raw[0]); g[2] = bf16_lo(raw[1]); g[3] = bf16_hi(raw[1]);
      } else {
        const f32x4 raw = *reinterpret_cast<const f32x4*>(gp + j * 4);
        g[0] = raw[0]; g[1] = raw[1]; g[2] = raw[2]; g[3] = raw[3];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const double a = (double)mv[e], b = (double)g[e], c = a + b;
        sm += a * a;
        sg += b * b;
        sb += c * c;
      }
    }
  }
  __shared__ double red[256];
  const double tm = block_sum_256(sm, red);
  const double tg = block_sum_256(sg, red);
  const double tb = block_sum_256(sb, red);
  if (tid == 0) {
    double* o = dpart + ((int64_t)z * gridDim.x + blockIdx.x) * 4;
    o[0] = tm; o[1] = tg; o[2] = tb; o[3] = 0.0;
  }
}

// ------------------------------------------------------------------------------------
// column sums of squares of R: partials over slabs of rows, then lengths and their sums
// ------------------------------------------------------------------------------------
// Four columns per thread and as many rows side by side as a workgroup has threads for (5632 x 256: 9.6 us with one column
// and one row per thread, 4.9 so; the sum over the slabs stays at one thread per column: 7.7 us, 15.8 with four).
__global__ __launch_bounds__(256) void k_diag_colsq(int n, int r, WsArr rr, WsArr part, int slabs) {
  const int z = blockIdx.z, slab = blockIdx.y, tid = threadIdx.x;
  const int cols4 = min(64, (r - (int)blockIdx.x * 256) / 4), groups = 256 / cols4;
  const int g = tid / cols4, c = (int)blockIdx.x * 256 + 4 * (tid - g * cols4);
  const int per = (n + slabs - 1) / slabs;
  const int r0 = slab * per, r1 = (r0 + per) < n ? (r0 + per) : n;
  const float* src = rr.base + (int64_t)z * rr.stride + c;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  if (g < groups) {
#pragma unroll 4
    for (int i = r0 + g; i < r1; i += groups) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(src + (int64_t)i * r);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] += (double)v[e] * (double)v[e];
    }
  }
  __shared__ double red[256][4];
#pragma unroll
  for (int e = 0; e < 4; ++e) red[tid][e] = acc[e];
  __syncthreads();
  if (g != 0) return;
  for (int k = 1; k < groups; ++k)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] += red[tid + k * cols4][e];
  *reinterpret_cast<f32x4*>(part.base + (int64_t)z * part.stride + (int64_t)slab * r + c) = f32x4{(float)acc[0], (float)acc[1], (float)acc[2], (float)acc[3]};
}

__global__ __launch_bounds__(256) void k_diag_cols_final(int r, WsArr part, int slabs, double* dacc) {
  const int z = blockIdx.x, tid = threadIdx.x;
  double s2 = 0.0, sl = 0.0, sll = 0.0;
  for (int c = tid; c < r; c += 256) {
    double s = 0.0;
#pragma unroll 16
    for (int k = 0; k < slabs; ++k) s += (double)part.base[(int64_t)z * part.stride + (int64_t)k * r + c];
    s2 += s;
    const double len = sqrt(s);
    sl += len;
    if (len > 0.0) sll += len * log(len);
  }
  __shared__ double red[256];
  const double t2 = block_sum_256(s2, red);
  const double tl = block_sum_256(sl, red);
  const double tll = block_sum_256(sll, red);
  if (tid == 0) {
    double* o = dacc + (int64_t)z * kDaccPerMat;
    o[3] = t2; o[4] = tl; o[5] = tll;
  }
}

// copy of the callers' Q (n x r, ld r) into a workspace array
__global__ __launch_bounds__(256) void k_gather_q(int n, int r, const MatEntry* mats, WsArr out) {
  const int z = blockIdx.y;
  const f32x4* src = reinterpret_cast<const f32x4*>(mats[z].Q);
  f32x4* dst = reinterpret_cast<f32x4*>(out.base + (int64_t)z * out.stride);
  const int64_t n4 = (int64_t)n * r / 4;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += (int64_t)gridDim.x * 256) dst[i] = src[i];
}

// ------------------------------------------------------------------------------------
// largest eigenvalue of the r x r Gram matrix G of Q; nu = sqrt of it.  Up to r = 256 by Lanczos in one
// workgroup (below), above by power iteration.
// ||G v|| / ||v|| with v = G^(2^kPowerSquarings) x0 estimates the eigenvalue from below with
// relative error O((lambda_2 / lambda_1)^(2^(kPowerSquarings + 1))).  The power is formed by
// squaring: 7 symmetric r x r products on the matrix cores instead of 128 dependent
// matrix-vector products, one launch each above r = 512.  Each square is taken of the matrix divided by its
// largest diagonal entry - for a positive semidefinite matrix the largest entry - so that nothing
// leaves the range of fp32 on the way.
// ------------------------------------------------------------------------------------
constexpr int kPowerThreads = 1024;
constexpr int kPowerMaxR = 2048;          // x kept in LDS
constexpr int kPowerSquarings = 7;
constexpr int kPowerRowsPerWg = 16;

OD_DEV float power_start(int i) { return 1.f + 0.5f * __sinf(0.7f * (float)i); }

// out = (a / max diagonal of a)^2 for symmetric a: row i of the left and row j of the right operand
// are both read along k.  UPPER: only the tiles on and above the diagonal are computed, and stored a second
// time, transposed.  That is for grids that fill the chip, where the products count: what the diagnostics add
// to a step of six matrices of r = 2048 is 3.6 ms with 128 matrix-vector products in place of the squares, 5.4 with
// all tiles of the squares, 4.0 with half of them (one matrix 1.5, 1.06, 1.02; 24 of r = 1024 3.3, 3.1, 2.4).  A
// grid that leaves part of the chip idle is all latency, to which the second store adds (r = 256: 5 us per step).
template <class T, bool UPPER>
__global__ __launch_bounds__(T::THREADS) void k_power_square(int r, WsArr a, WsArr out) {
  typedef NumBF<3> Num;
  extern __shared__ __align__(16) char lds[];
  __shared__ float red[T::THREADS / 64];
  const int z = blockIdx.z, tid = threadIdx.x;
  const int tiles = (r + T::NT - 1) / T::NT;
  int tn = blockIdx.x % tiles, tm = blockIdx.x / tiles;
  if constexpr (UPPER) {
    tm = 0;
    tn = blockIdx.x;
    while (tn >= tiles - tm) { tn -= tiles - tm; ++tm; }
    tn += tm;
  }
  const SrcF32 s{a.base + (int64_t)z * a.stride, r, r, r};
  float md = 0.f;
  for (int i = tid; i < r; i += T::THREADS) md = fmaxf(md, s.p[(int64_t)i * r + i]);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) md = fmaxf(md, __shfl_xor(md, off, 64));
  if ((tid & 63) == 0) red[tid >> 6] = md;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < T::THREADS / 64; ++w) md = fmaxf(md, red[w]);
  const float inv = md > 0.f ? 1.f / md : 0.f;
  f32x16 acc[T::FM][T::FN];
  zero_acc<T>(acc);
  gemm_mainloop_deep<T, Num, KC, SrcF32, KC, SrcF32, 3>(s, s, tm * T::MT, tn * T::NT, 0, r, 1.f, 1.f, lds, acc);
  float* o = out.base + (int64_t)z * out.stride;
  for_each_acc<T>(acc, tm * T::MT, tn * T::NT, [&](int row, int col, float v) {
    if (row < r && col < r) o[(int64_t)row * r + col] = v * inv * inv;
  });
  if (UPPER && tm != tn) {
    // lane (c, h) holds rows 8q + 4h .. 8q + 4h + 3 of column c: four consecutive entries of row c of the
    // transposed tile (r is a multiple of 8, so they are inside or outside together)
    const int lane = tid & 63, wave = tid >> 6, wm = wave / T::WN, wn = wave % T::WN;
#pragma unroll
    for (int fm = 0; fm < T::FM; ++fm)
#pragma unroll
      for (int fn = 0; fn < T::FN; ++fn) {
        const int col = tn * T::NT + wn * T::WTN + fn * 32 + (lane & 31);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int row0 = tm * T::MT + wm * T::WTM + fm * 32 + 8 * q + 4 * (lane >> 5);
          if (col < r && row0 < r) {
            f32x4 v4;
#pragma unroll
            for (int e = 0; e < 4; ++e) v4[e] = acc[fm][fn][4 * q + e] * inv * inv;
            *reinterpret_cast<f32x4*>(o + (int64_t)col * r + row0) = v4;
          }
        }
      }
  }
}

// y[i] = scale * sum_j g[i][j] x[j], row0 <= i < row1: four consecutive rows per wave and turn, so that
// their loads are in flight together
OD_DEV void power_rows(const float* g, const float* x_lds, int r, int row0, int row1, float scale, float* y) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  for (int i = row0 + 4 * wave; i < row1; i += 4 * nw) {
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    for (int j = lane * 4; j < r; j += 256) {
      const f32x4 b = *reinterpret_cast<const f32x4*>(x_lds + j);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 a = *reinterpret_cast<const f32x4*>(g + (int64_t)min(i + q, row1 - 1) * r + j);
        acc[q] += a[0] * b[0] + a[1] * b[1] + a[2] * b[2] + a[3] * b[3];
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) acc[q] += __shfl_xor(acc[q], off, 64);
      if (lane == 0 && i + q < row1) y[i + q] = acc[q] * scale;
    }
  }
}

OD_DEV float block_sumsq(const float* v, int r, float* red) {
  const int tid = threadIdx.x;
  float s = 0.f;
  for (int i = tid; i < r; i += blockDim.x) s += v[i] * v[i];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  __syncthreads();
  if ((tid & 63) == 0) red[tid >> 6] = s;
  __syncthreads();
  float t = 0.f;
  for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += red[w];
  return t;
}

// ------------------------------------------------------------------------------------
// r <= 256: the matrix fits the registers of one workgroup (64 entries per thread), which takes kLanczosSteps steps of
// the Lanczos iteration from the same start vector and reports the largest Ritz value.  Like the power it approaches
// the eigenvalue from below, and closer: over random factors of 8 to 256 columns the largest error of nu is 3e-3 where the
// power's is 7e-3 (their means 2e-4 and 1e-3 at 256 columns, 4e-6 and 4e-4 at 136), and no larger than the power's over
// sixteen kinds of spectra (even, dense at the top, one value above a cluster, geometric ...: 7e-3 | 1.5e-2), without the
// seven dependent squarings.  The relative error of the eigenvalue is at most d + tan(t)^2 / T_23((1 + d) / (1 - d))^2
// for every d, t the angle between start vector and leading eigenvector: the Rayleigh quotient of T_23, the Chebyshev
// polynomial of [0, (1 - d) lambda_1], applied to the start vector (Saad, SIAM J. Numer. Anal. 17, 1980); the power's is
// d + tan(t)^2 (1 - d)^256.  2.2 and 4.6 % at tan(t)^2 = 256.  Ghost copies from lost orthogonality repeat Ritz values and
// raise the largest by rounding only (nu by up to 2e-5, with two different eigenvalues).
// What bounds it: 64 fma per thread and step at four waves per SIMD, two sums over the workgroup.
// r = 256: 86 us (seven squarings of 10 us, two products) -> 35 us; a 2048 x 5632 step with diagnostics, r = 256,
// 512 -> 462 us.
// ------------------------------------------------------------------------------------
constexpr int kLanczosMaxR = 256, kLanczosSteps = 24;

template <int CTRL>
OD_DEV float dpp_add(float x) { return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true)); }
OD_DEV float row16_sum(float x) {      // over the 16 lanes of a row, in every lane
  x = dpp_add<0x128>(x);               // row_ror:8, 4, 2, 1
  x = dpp_add<0x124>(x);
  x = dpp_add<0x122>(x);
  return dpp_add<0x121>(x);
}

__global__ __launch_bounds__(kPowerThreads) void k_lanczos(int r, WsArr gram, double* dacc) {
  __shared__ __align__(16) float x[kLanczosMaxR];
  __shared__ __align__(16) float red[2][kPowerThreads / 64];
  __shared__ float alphas[kLanczosSteps], betas2[kLanczosSteps];
  const int z = blockIdx.x, tid = threadIdx.x, lane = tid & 63, c = tid & 15, row0 = 4 * (tid >> 4);
  const float* g = gram.base + (int64_t)z * gram.stride;
  // rows row0 .. row0 + 3, columns 4 c + 64 q .. + 3 (orders are multiples of 8: four columns are in or out together)
  f32x4 a[4][4];
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      a[e][q] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (row0 + e < r && 4 * c + 64 * q < r) a[e][q] = *reinterpret_cast<const f32x4*>(g + (int64_t)(row0 + e) * r + 4 * c + 64 * q);
    }
  // sum over all rows of a value that the 16 lanes of a row group share
  auto total = [&](float v, int buf) {
    const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(p[0]) + __uint_as_float(p[1]);
    const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(h[0]) + __uint_as_float(h[1]);
    if (lane == 0) red[buf][tid >> 6] = v;
    __syncthreads();
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < kPowerThreads / 256; ++w) s += *reinterpret_cast<const f32x4*>(&red[buf][4 * w]);
    return (s[0] + s[1]) + (s[2] + s[3]);
  };
  f32x4 v, prev = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = row0 + e < r ? power_start(row0 + e) : 0.f;
  float beta = 0.f;
  {
    const float n2 = total(v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3], 0);
    v *= rsqrtf(n2);
  }
  for (int k = 0; k < kLanczosSteps; ++k) {
    if (c == 0) *reinterpret_cast<f32x4*>(x + row0) = v;
    __syncthreads();
    f32x4 w = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 b = *reinterpret_cast<const f32x4*>(x + 4 * c + 64 * q);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < 4; ++i) w[e] = fmaf(a[e][q][i], b[i], w[e]);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = row16_sum(w[e]);
    const float alpha = total(v[0] * w[0] + v[1] * w[1] + v[2] * w[2] + v[3] * w[3], 1);
    w -= alpha * v + beta * prev;
    const float b2 = total(w[0] * w[0] + w[1] * w[1] + w[2] * w[2] + w[3] * w[3], 0);
    if (tid == 0) {
      alphas[k] = alpha;
      betas2[k] = b2;
    }
    beta = sqrtf(b2);
    prev = v;
    v = w * (b2 > 0.f ? 1.f / beta : 0.f);        // an invariant subspace: zero rows from here on
  }
  __syncthreads();
  if (tid >= 64) return;
  // Largest eigenvalue of the tridiagonal matrix: x lies above it where all pivots of T - x are negative.
  // 64 points at a time between the largest diagonal entry and the Gershgorin bound.
  float al[kLanczosSteps], b2[kLanczosSteps];
#pragma unroll
  for (int k = 0; k < kLanczosSteps; ++k) {
    al[k] = alphas[k];
    b2[k] = betas2[k];
  }
  const float mine = lane < kLanczosSteps ? alphas[lane] : alphas[0];
  float lo = mine, hi = mine + (lane > 0 && lane < kLanczosSteps ? sqrtf(betas2[lane - 1]) : 0.f) + (lane + 1 < kLanczosSteps ? sqrtf(betas2[lane]) : 0.f);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    lo = fmaxf(lo, __shfl_xor(lo, off, 64));
    hi = fmaxf(hi, __shfl_xor(hi, off, 64));
  }
#pragma unroll 1
  for (int round = 0; round < 5; ++round) {
    const float p = lo + (hi - lo) * ((float)(lane + 1) * (1.f / 64.f));
    float d = al[0] - p;
    bool above = d < 0.f;
#pragma unroll
    for (int k = 1; k < kLanczosSteps; ++k) {
      d = al[k] - p - (b2[k - 1] > 0.f ? b2[k - 1] * __builtin_amdgcn_rcpf(d) : 0.f);
      above = above && d < 0.f;
    }
    const uint64_t m = __ballot(above);
    const int first = m != 0 ? __ffsll((unsigned long long)m) - 1 : 63;      // the bound itself, but for rounding
    hi = __shfl(p, first, 64);
    lo = first > 0 ? __shfl(p, first > 0 ? first - 1 : 0, 64) : lo;
  }
  if (tid == 0) dacc[(int64_t)z * kDaccPerMat + 7] = (double)lo;
}

// The two matrix-vector products after the squarings, v = P x0 and G v / ||v||.  Up to r = 512 one
// workgroup per matrix does both.
__global__ __launch_bounds__(kPowerThreads) void k_power_estimate(int r, WsArr power, WsArr gram, double* dacc) {
  __shared__ __align__(16) float x[kPowerMaxR];
  __shared__ __align__(16) float y[kPowerMaxR];
  __shared__ float red[kPowerThreads / 64];
  const int z = blockIdx.x, tid = threadIdx.x;
  for (int i = tid; i < r; i += kPowerThreads) x[i] = power_start(i);
  __syncthreads();
  power_rows(power.base + (int64_t)z * power.stride, x, r, 0, r, 1.f, y);
  __syncthreads();
  const float s = block_sumsq(y, r, red);
  const float inv = s > 0.f ? rsqrtf(s) : 0.f;
  power_rows(gram.base + (int64_t)z * gram.stride, y, r, 0, r, inv, x);
  __syncthreads();
  const float lam = sqrtf(block_sumsq(x, r, red));
  if (tid == 0) dacc[(int64_t)z * kDaccPerMat + 7] = (double)lam;
}

// Larger r: rows spread over workgroups, one launch per product; `first` starts from x0
__global__ __launch_bounds__(256) void k_power_step(int r, WsArr mat, WsArr xbuf, int first) {
  __shared__ __align__(16) float x[kPowerMaxR];
  __shared__ float red[4];
  const int z = blockIdx.y, tid = threadIdx.x;
  const float* g = mat.base + (int64_t)z * mat.stride;
  float* xb = xbuf.base + (int64_t)z * xbuf.stride;
  for (int i = tid; i < r; i += 256) x[i] = first ? power_start(i) : xb[i];
  __syncthreads();
  float inv = 1.f;
  if (!first) {
    const float s = block_sumsq(x, r, red);
    inv = s > 0.f ? rsqrtf(s) : 0.f;
  }
  const int row0 = blockIdx.x * kPowerRowsPerWg;
  const int row1 = (row0 + kPowerRowsPerWg) < r ? (row0 + kPowerRowsPerWg) : r;
  power_rows(g, x, r, row0, row1, inv, first ? xb : xb + r);
}
__global__ __launch_bounds__(256) void k_power_final(int r, WsArr xbuf, double* dacc) {
  __shared__ float red[4];
  const int z = blockIdx.x;
  const float* x = xbuf.base + (int64_t)z * xbuf.stride + r;
  const float s = block_sumsq(x, r, red);
  if (threadIdx.x == 0) dacc[(int64_t)z * kDaccPerMat + 7] = (double)sqrtf(s);
}

// ------------------------------------------------------------------------------------
// the reported scalars, one workgroup per matrix; QR variant: also the trace of T2 T1 (both upper
// triangular: the sum of products of the diagonals), which is <B, P Q^T>
// ------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_diag_final(int r, const double* dpart, int blocks, const double* dacc, WsArr t1, WsArr t2, int colnorm, float* diag) {
  const int z = blockIdx.x, tid = threadIdx.x;
  __shared__ double red[256];
  double sm = 0.0, sg = 0.0, sb = 0.0, tr = 0.0;
  for (int k = tid; k < blocks; k += 256) {
    const double* p = dpart + ((int64_t)z * blocks + k) * 4;
    sm += p[0]; sg += p[1]; sb += p[2];
  }
  if (!colnorm) {
    const float* a1 = t1.base + (int64_t)z * t1.stride;
    const float* a2 = t2.base + (int64_t)z * t2.stride;
    for (int i = tid; i < r; i += 256) tr += (double)a1[(int64_t)i * r + i] * (double)a2[(int64_t)i * r + i];
  }
  sm = block_sum_256(sm, red);
  sg = block_sum_256(sg, red);
  sb = block_sum_256(sb, red);
  tr = block_sum_256(tr, red);
  if (tid != 0) return;
  const double* a = dacc + (int64_t)z * kDaccPerMat;
  const double r2 = a[3], sl = a[4], sll = a[5];
  float* o = diag + (int64_t)z * kDiagPerMat;
  const double gap = sb - r2;
  o[0] = (float)sqrt(sb);
  o[1] = (float)sqrt(r2);
  o[2] = sb > 0.0 ? (float)sqrt((gap > 0.0 ? gap : 0.0) / sb) : 0.f;
  o[3] = sg > 0.0 ? (float)sqrt(sm / sg) : 0.f;
  o[4] = (float)(colnorm ? sl : tr);
  o[5] = (float)sqrt(a[7]);
  o[6] = sl > 0.0 ? (float)exp(log(sl) - sll / sl) : 0.f;
  o[7] = (float)sqrt(sg);
}

// ------------------------------------------------------------------------------------
// rank change of the warm-start factor: keep the leading columns, append caller-supplied ones
// ------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_resize_q(const float* q_old, int64_t n, int r_old, float* q_new, int r_new,
                                                  const float* pad) {
  const int64_t total = n * r_new;
  const int keep = r_old < r_new ? r_old : r_new;
  const int extra = r_new - keep;
  for (int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x; idx < total; idx += (int64_t)gridDim.x * 256) {
    const int64_t i = idx / r_new;
    const int c = (int)(idx - i * r_new);
    q_new[idx] = c < keep ? q_old[i * r_old + c] : pad[i * extra + (c - keep)];
  }
}

// ------------------------------------------------------------------------------------
// launchers
// ------------------------------------------------------------------------------------
hipError_t launch_diag_norms(const ClassDims& d, const MatEntry* mats, double* dpart, int blocks, hipStream_t st) {
  if (d.g_bf16) hipLaunchKernelGGL(k_diag_norms<true>, dim3(blocks, d.nb), dim3(256), 0, st, d, mats, dpart);
  else hipLaunchKernelGGL(k_diag_norms<false>, dim3(blocks, d.nb), dim3(256), 0, st, d, mats, dpart);
  OD_CHECK_LAUNCH();
  return hipSuccess;
}

hipError_t launch_diag_cols(int nb, int n, int r, WsArr rr, WsArr part, int slabs, double* dacc, hipStream_t st) {
  hipLaunchKernelGGL(k_diag_colsq, dim3((r + 255) / 256, slabs, nb), dim3(256), 0, st, n, r, rr, part, slabs);
  OD_CHECK_LAUNCH();
  hipLaunchKernelGGL(k_diag_cols_final, dim3(nb), dim3(256), 0, st, r, part, slabs, dacc);
  OD_CHECK_LAUNCH();
  return hipSuccess;
}

hipError_t launch_gather_q(int nb, int n, int r, const MatEntry* mats, WsArr out, hipStream_t st) {
  int64_t n4 = (int64_t)n * r / 4;
  int blocks = (int)((n4 + 255) / 256);
  if (blocks > 2048) blocks = 2048;
  hipLaunchKernelGGL(k_gather_q, dim3(blocks, nb), dim3(256), 0, st, n, r, mats, out);
  OD_CHECK_LAUNCH();
  return hipSuccess;
}

template <class T, bool UPPER>
static hipError_t power_square(int nb, int r, WsArr a, WsArr out, hipStream_t st) {
  constexpr int lds = T::template lds_bytes<NumBF<3>>();
  const hipError_t e = lds > 64 * 1024
      ? hipFuncSetAttribute(reinterpret_cast<const void*>(k_power_square<T, UPPER>), hipFuncAttributeMaxDynamicSharedMemorySize, lds) : hipSuccess;
  if (e != hipSuccess) return e;
  const int tiles = (r + T::NT - 1) / T::NT;
  hipLaunchKernelGGL((k_power_square<T, UPPER>), dim3(UPPER ? tiles * (tiles + 1) / 2 : tiles * tiles, 1, nb), dim3(T::THREADS), lds, st, r, a, out);
  OD_CHECK_LAUNCH();
  return hipSuccess;
}

hipError_t launch_power(int nb, int r, WsArr gram, WsArr tmp1, WsArr tmp2, WsArr xbuf, double* dacc, hipStream_t st) {
  if (r > kPowerMaxR || xbuf.stride < 2 * (int64_t)r) return hipErrorInvalidValue;
  if (r <= kLanczosMaxR) {
    hipLaunchKernelGGL(k_lanczos, dim3(nb), dim3(kPowerThreads), 0, st, r, gram, dacc);
    OD_CHECK_LAUNCH();
    return hipSuccess;
  }
  // 64 x 64 tiles until 128 x 128 ones fill the chip by themselves
  const bool big = (int64_t)((r + 127) / 128) * ((r + 127) / 128) * nb >= 256;
  WsArr cur = gram, nxt = tmp1;
  for (int i = 0; i < kPowerSquarings; ++i) {
    const hipError_t e = big ? power_square<Tile<128, 128, 32, 2, 2>, true>(nb, r, cur, nxt, st) : power_square<Tile<64, 64, 64, 2, 2>, false>(nb, r, cur, nxt, st);
    if (e != hipSuccess) return e;
    cur = nxt;
    nxt = cur.base == tmp1.base ? tmp2 : tmp1;
  }
  if (r <= 512) {
    hipLaunchKernelGGL(k_power_estimate, dim3(nb), dim3(kPowerThreads), 0, st, r, cur, gram, dacc);
    OD_CHECK_LAUNCH();
    return hipSuccess;
  }
  const dim3 grid((r + kPowerRowsPerWg - 1) / kPowerRowsPerWg, nb);
  hipLaunchKernelGGL(k_power_step, grid, dim3(256), 0, st, r, cur, xbuf, 1);
  OD_CHECK_LAUNCH();
  hipLaunchKernelGGL(k_power_step, grid, dim3(256), 0, st, r, gram, xbuf, 0);
  OD_CHECK_LAUNCH();
  hipLaunchKernelGGL(k_power_final, dim3(nb), dim3(256), 0, st, r, xbuf, dacc);
  OD_CHECK_LAUNCH();
  return hipSuccess;
}

hipError_t launch_diag_final(int nb, int r, const double* dpart, int blocks, const double* dacc, WsArr t1, WsArr t2, int colnorm, float* diag, hipStream_t st) {
  hipLaunchKernelGGL(k_diag_final, dim3(nb), dim3(256), 0, st, r, dpart, blocks, dacc, t1, t2, colnorm, diag);
  OD_CHECK_LAUNCH();
  return hipSuccess;
}

hipError_t launch_resize_q(const float* q_old, int64_t n, int r_old, float* q_new, int r_new, const float* pad, hipStream_t st) {
  int64_t total = n * r_new;
  int blocks = (int)((total + 255) / 256);
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_resize_q, dim3(blocks), dim3(256), 0, st, q_old, n, r_old, q_new, r_new, pad);
  OD_CHECK_LAUNCH();
  return hipSuccess;
}

}  // namespace od

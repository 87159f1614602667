// HIP kernels of the Orth-Dion optimizer step for gfx950 (CDNA4) and their launchers.
//
// Notation follows the library interface: B = M + G (paper Alg. 1 line 1, never stored),
// P_raw = B Q (line 2), P = orth(P_raw) (line 2), R = B^T P (line 3), Q = orth(R) or
// ColNorm(R) (line 4), X -= lr P Q^T (lines 5-6), M = a B - b P R^T (line 7).
#include "od_kernels.h"

#include <hip/hip_ext.h>

#include "od_chol.h"
#include "od_dma.h"
#include "od_gemm.h"

namespace od {

// ------------------------------------------------------------------------------------
// One launch for several batches.  A step over matrices of different shapes is a chain of short
// kernels, each a few microseconds of launch and latency; batches that take the same kernel share
// its launch, one segment of the grid each (five small matrices of four shapes and ranks: 503 -> 250 us;
// 126 matrices of three shapes, r = 192: 1950 -> 1715 us).
// The grid is one-dimensional; a segment starts at a multiple of 8 workgroups, so that the XCD a
// workgroup lands on (round robin by its index) follows from its index in the segment.
// A launch of a single segment takes its arguments as One<A> and an ordinary three-dimensional
// grid: indexing a table of segments costs a second round of argument loads before a workgroup can
// start (0.4 us per kernel in a chain of short ones).
// ------------------------------------------------------------------------------------
constexpr int kMaxSeg = 8;
struct SegGrid { int x, y, z; };              // the segment's own grid, x fastest
template <class A>
struct Segs {
  int n;
  int first[kMaxSeg];                         // first workgroup of segment i
  SegGrid grid[kMaxSeg];
  A seg[kMaxSeg];
};
template <class A>
struct One {
  A seg[1];
};
struct SegBlock {
  int flat, x, y, z;                          // position in the segment
  SegGrid grid;
};
// The segment of workgroup `bid`, or -1 for the padding between segments.
template <class A>
OD_DEV int seg_locate(const Segs<A>& g, SegBlock& b, int bid) {
  int s = 0;
#pragma unroll
  for (int i = 1; i < kMaxSeg; ++i)
    if (i < g.n && bid >= g.first[i]) s = i;
  b.grid = g.grid[s];
  b.flat = bid - g.first[s];
  const int plane = b.grid.x * b.grid.y;
  if (b.flat >= plane * b.grid.z) return -1;
  b.z = 0;
  int rest = b.flat;
  if (b.grid.z > 1) { b.z = rest / plane; rest -= b.z * plane; }
  b.y = 0;
  if (b.grid.y > 1) { b.y = rest / b.grid.x; rest -= b.y * b.grid.x; }
  b.x = rest;
  return s;
}
template <class A>
OD_DEV int seg_locate(const Segs<A>& g, SegBlock& b) { return seg_locate(g, b, (int)blockIdx.x); }
template <class A>
OD_DEV int seg_locate(const One<A>&, SegBlock& b) {
  b.grid = SegGrid{(int)gridDim.x, (int)gridDim.y, (int)gridDim.z};
  b.x = (int)blockIdx.x;
  b.y = (int)blockIdx.y;
  b.z = (int)blockIdx.z;
  b.flat = b.x + b.grid.x * (b.y + b.grid.y * b.z);
  return 0;
}
#define OD_SEGMENT(Args)                      \
  SegBlock blk;                               \
  const int seg_ = seg_locate(segs, blk);     \
  if (seg_ < 0) return;                       \
  const Args& a_ = segs.seg[seg_]
// The caller's buffers of matrix z: from the table, or from the arguments when the batch has one matrix
#define OD_MATRIX(z) (a_.d.nb == 1 ? a_.only : a_.mats[z])

// ------------------------------------------------------------------------------------
// tile shapes
// ------------------------------------------------------------------------------------
typedef Tile<128, 256, 32, 2, 2> TileWide;     // r > 128: wave tile 64 x 128
typedef Tile<128, 128, 32, 2, 2> TileSquare;   // wave tile 64 x 64
// The same on eight waves (wave tile 32 x 64): half the registers, twice the waves per CU at the same LDS, so that
// the operand conversions of one wave run beside the products of another.  A W of 96 matrices of rank 512:
// 2.44 -> 2.39 ms by the kernel trace, its correction 1.55 -> 1.50, Gram matrices 2.40 -> 2.37; 126 matrices of rank 192:
// 1668 -> 1629 us per step; the three-part operands of a 1024-wide fp32 model: 338 -> 329 us.
typedef Tile<128, 128, 32, 4, 2> TileSquare8;
typedef Tile<128, 64, 32, 4, 1> TileNarrow;    // r <= 64: wave tile 32 x 64
typedef Tile<64, 256, 32, 2, 2> TileFlat;      // projection, r > 128: twice the row panels, half the splits (wave tile 32 x 128)
typedef Tile<256, 256, 32, 2, 2> TileHuge;    // back-projection, r > 256: wave tile 128 x 128, one workgroup per CU
typedef Tile<128, 128, 64, 4, 2> TileSquareDeepK;   // single-part operands: half the k steps at the same LDS footprint
typedef Tile<64, 64, 64, 2, 2> TileSmall;      // wave tile 32 x 32: small problems that need many workgroups

typedef short s16x4 __attribute__((ext_vector_type(4)));    // result of the LDS transpose read
constexpr float kUnitScale = 1024.f;           // scale of orthonormal / unit-column factors in fp16

OD_DEV bool pred_on(const Pred& p, int z) {
  if (p.scal == nullptr) return true;
  return (p.scal[z * kScalPerMat + p.slot] > p.thr) == (p.want != 0);
}

OD_DEV int split_begin(int K, int splits, int KT, int s, int* kend) {
  int per = ((K + splits - 1) / splits + KT - 1) / KT * KT;
  int kb = s * per;
  int ke = kb + per;
  *kend = ke < K ? ke : K;
  return kb;
}

template <class GSrc>
OD_DEV SrcSum<GSrc> make_b_source(const ClassDims& d, const MatEntry& e) {
  SrcSum<GSrc> s;
  s.m = SrcF32{e.M, d.m, d.n, d.ldm};
  s.g = GSrc{reinterpret_cast<decltype(GSrc::p)>(e.G), d.m, d.n, d.ldg};
  return s;
}

// ------------------------------------------------------------------------------------
// sampled power-of-two scale of B for the fp16 operand format
// ------------------------------------------------------------------------------------
OD_DEV float pow2_scale_for_rms(float ms) {
  if (ms > 0.f && ms < 3.0e38f) return ldexpf(1.f, -ilogbf(sqrtf(ms)));
  return 1.f;
}

constexpr int kStatRows = 32;      // sampled rows per matrix, one workgroup each

template <class GSrc>
OD_DEV void stats_block(const ClassDims& d, const MatEntry& e, float* scal, int z, int row_index) {
  const int tid = threadIdx.x;
  SrcSum<GSrc> b = make_b_source<GSrc>(d, e);
  const int nrows = d.m < kStatRows ? d.m : kStatRows;
  float acc = 0.f;
  const int groups = d.n / 8;
  if (row_index < nrows)
  for (int idx = tid; idx < groups; idx += 256) {
    int s = row_index, c = idx * 8;
    int row = (int)(((int64_t)s * d.m) / nrows);
    float x[8];
    SrcSum<GSrc>::unpack8(b.load8(row, c), x);
#pragma unroll
    for (int i = 0; i < 8; ++i) acc += x[i] * x[i];
  }
  __shared__ float red[256];
  red[tid] = acc;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (tid < w) red[tid] += red[tid + w];
    __syncthreads();
  }
  if (tid == 0) scal[z * kScalPerMat + kScalSample + row_index] = red[0];
}

// Q (n x r fp32, the caller's state) -> pre-scaled fp16, transposed to [r][n]
OD_DEV void prep_q_block(const ClassDims& d, const float* q, HalfArr qht, int z, int bx, int by) {
  __shared__ uint16_t tile[64][66];
  const int tid = threadIdx.x;
  const int k0 = bx * 64, c0 = by * 64;       // k over n, c over r
  uint16_t* out = qht.base + (int64_t)z * qht.stride;
  for (int idx = tid; idx < 64 * 16; idx += 256) {            // 64 rows (k) x 16 groups of 4 columns
    const int kk = idx / 16, cg = (idx % 16) * 4;
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (k0 + kk < d.n && c0 + cg < d.r) v = *reinterpret_cast<const f32x4*>(q + (int64_t)(k0 + kk) * d.r + c0 + cg);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      _Float16 x = (_Float16)__builtin_amdgcn_fmed3f(v[e] * kUnitScale, -65504.f, 65504.f);
      tile[cg + e][kk] = __builtin_bit_cast(uint16_t, x);
    }
  }
  __syncthreads();
  for (int idx = tid; idx < 64 * 16; idx += 256) {            // 64 rows (c) x 16 groups of 4 k
    const int cc = idx / 16, kg = (idx % 16) * 4;
    if (c0 + cc < d.r && k0 + kg < d.n) {
      u32x2 h = {(uint32_t)tile[cc][kg] | ((uint32_t)tile[cc][kg + 1] << 16),
                 (uint32_t)tile[cc][kg + 2] | ((uint32_t)tile[cc][kg + 3] << 16)};
      *reinterpret_cast<u32x2*>(out + (int64_t)(c0 + cc) * d.n + k0 + kg) = h;
    }
  }
}

// First kernel of a step.  The caller's buffers arrive as kernel arguments, kMatChunk matrices at a
// time, and go to the table in the workspace that every later kernel reads (those can then take any
// number of matrices).  Workgroup 0 of a matrix writes its entry and clears its flag and scale words;
// in fast precision workgroups 0 .. kStatRows-1 also sample the scale of B and the others convert Q.
constexpr int kMatChunk = 64;
struct BeginArgs {
  ClassDims d;
  MatEntry* table;      // entries of this segment's matrices
  int chunk0;           // first of them in the launch's chunk
  float* scal;
  int* info;
  HalfArr qht;
};
struct MatChunk { MatEntry e[kMatChunk]; };

template <class GSrc, bool FAST, class SegsT>
__global__ __launch_bounds__(256) void k_begin(SegsT segs, MatChunk chunk) {
  OD_SEGMENT(BeginArgs);
  const int z = blk.z, bx = blk.x;
  const MatEntry e = chunk.e[a_.chunk0 + z];
  if (bx == 0) {
    if (threadIdx.x == 0) a_.table[z] = e;
    if (threadIdx.x < kScalSample) a_.scal[z * kScalPerMat + threadIdx.x] = 0.f;
    if (threadIdx.x < kInfoPerMat) a_.info[z * kInfoPerMat + threadIdx.x] = 0;
  }
  if constexpr (FAST) {
    if (bx < kStatRows) {
      stats_block<GSrc>(a_.d, e, a_.scal, z, bx);
    } else {
      const int t = bx - kStatRows, tiles_k = (a_.d.n + 63) / 64;
      prep_q_block(a_.d, e.Q, a_.qht, z, t % tiles_k, t / tiles_k);
    }
  }
}

// scale of B from the sampled row sums of squares (same value in every consumer)
OD_DEV float b_scale(const ClassDims& d, const float* scal, int z) {
  const int nrows = d.m < kStatRows ? d.m : kStatRows;
  // all kStatRows slots are written (zero beyond nrows): fixed-size vector loads, no loop-carried latency
  const f32x4* p = reinterpret_cast<const f32x4*>(scal + z * kScalPerMat + kScalSample);
  f32x4 acc4 = p[0];
#pragma unroll
  for (int i = 1; i < kStatRows / 4; ++i) acc4 += p[i];
  const float tot = (acc4[0] + acc4[1]) + (acc4[2] + acc4[3]);
  return pow2_scale_for_rms(tot / ((float)nrows * (float)d.n));
}

// ------------------------------------------------------------------------------------
// P_raw = B Q  (split over n)                                       Alg. 1 line 2
// ------------------------------------------------------------------------------------
// scale of R = B^T P in fp16: P is orthonormal, so rms(R) <= rms(B) sqrt(m / r); a power of
// two derived from the scale of B alone, known before R exists
OD_DEV float r_scale(const ClassDims& d, const float* scal, int z) {
  return ldexpf(b_scale(d, scal, z), -(ilogbf((float)d.m / (float)d.r) / 2));
}

// Second argument of __launch_bounds__ (waves per SIMD the register allocation must allow;
// with 4-wave workgroups that is workgroups per CU).  Register stages of a deep prefetch on
// top of 8 accumulator tiles, or 16 accumulator tiles alone, need more than 256 registers.
template <class T, int PF>
constexpr int min_waves_per_simd() { return ((PF > 1 && T::FM * T::FN >= 8) || T::FM * T::FN >= 16) ? 1 : 2; }

// Arguments of the projection and the back-projection (one segment).
struct StreamArgs {
  ClassDims d;
  const MatEntry* mats;
  MatEntry only;        // the one matrix of a batch of one
  const float* scal;
  int* info;
  WsArr factor;         // back-projection, exact precision: P in fp32
  HalfArr fh;           // fast precision: the factor operand as fp16, [r][contracted dimension]
  WsArr part;
  HalfArr rh;           // direct-to-LDS back-projection with one split: fp16 copy of R
  int splits, rotate;
};

template <class T, class Num, class GSrc, int PF, class SegsT>
__global__ __launch_bounds__(T::THREADS, (min_waves_per_simd<T, PF>())) void k_proj(SegsT segs) {
  extern __shared__ __align__(16) char lds[];
  OD_SEGMENT(StreamArgs);
  const ClassDims& d = a_.d;
  const float* scal = a_.scal;
  const int splits = a_.splits, rotate = a_.rotate;
  const int tiles_n = (d.r + T::NT - 1) / T::NT;
  // the column tiles of one row panel read the same part of B: keep them on one XCD
  const int bid = tiles_n > 1 ? xcd_contiguous(blk.x, blk.grid.x) : blk.x;
  const int tn = bid % tiles_n, tm = bid / tiles_n;
  const int split = blk.y, z = blk.z;
  const MatEntry mat = OD_MATRIX(z);
  SrcSum<GSrc> a = make_b_source<GSrc>(d, mat);
  SrcF32 b{mat.Q, d.n, d.r, d.r};
  int kend;
  const int kbeg = split_begin(d.n, splits, T::KT, split, &kend);
  const float sa = Num::F16 ? b_scale(d, scal, z) : 1.f;
  const float sb = Num::F16 ? kUnitScale : 1.f;
  f32x16 acc[T::FM][T::FN];
  zero_acc<T>(acc);
  if constexpr (Num::F16) {
    // Q as pre-scaled fp16, transposed to [r][n] so that k is contiguous
    SrcH16 bh{a_.fh.base + (int64_t)z * a_.fh.stride, d.r, d.n, d.n};
    // Row panels of one matrix read the same columns of B at the same time, and with a row
    // stride that is a multiple of the memory-channel interleave they all land on the same
    // channels: start every panel at a different k step then.
    if constexpr (PF > 1)
      gemm_mainloop_deep<T, Num, KC, SrcSum<GSrc>, KC, SrcH16, PF>(a, bh, tm * T::MT, tn * T::NT, kbeg, kend, sa, sb, lds, acc, rotate ? tm : 0);
    else
      gemm_mainloop<T, Num, KC, SrcSum<GSrc>, KC, SrcH16>(a, bh, tm * T::MT, tn * T::NT, kbeg, kend, sa, sb, lds, acc, rotate ? tm : 0);
  } else {
    gemm_mainloop<T, Num, KC, SrcSum<GSrc>, KS, SrcF32>(a, b, tm * T::MT, tn * T::NT, kbeg, kend, sa, sb, lds, acc);
  }
  const float inv = 1.f / (sa * sb);
  float* out = a_.part.base + (int64_t)z * a_.part.stride + (int64_t)split * d.m * d.r;
  for_each_acc<T>(acc, tm * T::MT, tn * T::NT, [&](int row, int col, float v) {
    if (row < d.m && col < d.r) out[(int64_t)row * d.r + col] = v * inv;
  });
}

// ------------------------------------------------------------------------------------
// R = B^T P  (split over m)                                         Alg. 1 line 3
// ------------------------------------------------------------------------------------
template <class T, class Num, class GSrc, int PF, class SegsT>
__global__ __launch_bounds__(T::THREADS, (min_waves_per_simd<T, PF>())) void k_back(SegsT segs) {
  extern __shared__ __align__(16) char lds[];
  OD_SEGMENT(StreamArgs);
  const ClassDims& d = a_.d;
  const float* scal = a_.scal;
  const int splits = a_.splits;
  const int tiles_n = (d.r + T::NT - 1) / T::NT;
  // as in the projection: the column tiles of one panel of B share an XCD's L2
  const int bid = tiles_n > 1 ? xcd_contiguous(blk.x, blk.grid.x) : blk.x;
  const int tn = bid % tiles_n, tm = bid / tiles_n;
  const int split = blk.y, z = blk.z;
  const MatEntry mat = OD_MATRIX(z);
  SrcSum<GSrc> a = make_b_source<GSrc>(d, mat);           // read as [k = row i][operand row = column j]
  SrcF32 b{a_.factor.base + (int64_t)z * a_.factor.stride, d.m, d.r, d.r};
  int kend;
  const int kbeg = split_begin(d.m, splits, T::KT, split, &kend);
  const float sa = Num::F16 ? b_scale(d, scal, z) : 1.f;
  const float sb = Num::F16 ? kUnitScale : 1.f;
  f32x16 acc[T::FM][T::FN];
  zero_acc<T>(acc);
  if constexpr (Num::F16) {
    SrcH16 bh{a_.fh.base + (int64_t)z * a_.fh.stride, d.r, d.m, d.m};  // P^T as fp16, [r][m]
    if constexpr (PF > 1)
      gemm_mainloop_deep<T, Num, KS, SrcSum<GSrc>, KC, SrcH16, PF>(a, bh, tm * T::MT, tn * T::NT, kbeg, kend, sa, sb, lds, acc);
    else
      gemm_mainloop<T, Num, KS, SrcSum<GSrc>, KC, SrcH16>(a, bh, tm * T::MT, tn * T::NT, kbeg, kend, sa, sb, lds, acc);
  } else {
    gemm_mainloop<T, Num, KS, SrcSum<GSrc>, KS, SrcF32>(a, b, tm * T::MT, tn * T::NT, kbeg, kend, sa, sb, lds, acc);
  }
  const float inv = 1.f / (sa * sb);
  float* out = a_.part.base + (int64_t)z * a_.part.stride + (int64_t)split * d.n * d.r;
  for_each_acc<T>(acc, tm * T::MT, tn * T::NT, [&](int row, int col, float v) {
    if (row < d.n && col < d.r) out[(int64_t)row * d.r + col] = v * inv;
  });
}

// ------------------------------------------------------------------------------------
// deterministic second stage of the split contractions
// ------------------------------------------------------------------------------------
struct ReduceArgs {
  WsArr part, out;
  int64_t count;
  int splits;
  Pred pred;
};
template <class SegsT>
__global__ __launch_bounds__(256) void k_reduce(SegsT segs) {
  OD_SEGMENT(ReduceArgs);
  const int z = blk.z, splits = a_.splits;
  if (!pred_on(a_.pred, z)) return;
  const int64_t count = a_.count;
  const float* src = a_.part.base + (int64_t)z * a_.part.stride;
  float* dst = a_.out.base + (int64_t)z * a_.out.stride;
  const int64_t n4 = count / 4;
  for (int64_t i = (int64_t)blk.x * 256 + threadIdx.x; i < n4; i += (int64_t)blk.grid.x * 256) {
    f32x4 s = reinterpret_cast<const f32x4*>(src)[i];
#pragma unroll 8
    for (int k = 1; k < splits; ++k) {       // unrolled: the loads of eight partials are in flight together
      f32x4 v = reinterpret_cast<const f32x4*>(src + (int64_t)k * count)[i];
      s += v;
    }
    reinterpret_cast<f32x4*>(dst)[i] = s;
  }
}

// the same for R, which is also stored as pre-scaled fp16 for the error-feedback kernel
struct ReduceRArgs {
  ClassDims d;
  WsArr part, out;
  int splits;
  HalfArr rh;
  const float* scal;
  int* info;
};
template <class SegsT>
__global__ __launch_bounds__(256) void k_reduce_r(SegsT segs) {
  OD_SEGMENT(ReduceRArgs);
  const int z = blk.z, splits = a_.splits;
  const ClassDims& d = a_.d;
  int* info = a_.info;
  const float* src = a_.part.base + (int64_t)z * a_.part.stride;
  float* dst = a_.out.base + (int64_t)z * a_.out.stride;
  uint16_t* dh = a_.rh.base + (int64_t)z * a_.rh.stride;
  const int64_t count = (int64_t)d.n * d.r, n4 = count / 4;
  const float sr = r_scale(d, a_.scal, z);
  float rmax = 0.f;
  for (int64_t i = (int64_t)blk.x * 256 + threadIdx.x; i < n4; i += (int64_t)blk.grid.x * 256) {
    f32x4 s = reinterpret_cast<const f32x4*>(src)[i];
#pragma unroll 8
    for (int k = 1; k < splits; ++k) s += reinterpret_cast<const f32x4*>(src + (int64_t)k * count)[i];
    if (dst != src) reinterpret_cast<f32x4*>(dst)[i] = s;     // in place (one split): only the fp16 copy is new
    u32x2 h = {pack_f16_sat(s[0] * sr, s[1] * sr), pack_f16_sat(s[2] * sr, s[3] * sr)};
    reinterpret_cast<u32x2*>(dh)[i] = h;
    rmax = fmaxf(rmax, fmaxf(fmaxf(fabsf(s[0]), fabsf(s[1])), fmaxf(fabsf(s[2]), fabsf(s[3]))));
  }
  // a clipped entry (or a NaN) is reported, not hidden
  if (!(rmax * sr <= 65504.f)) atomicOr(&info[z * kInfoPerMat + kWarnSlot], kWarnRClipped);
}

// ------------------------------------------------------------------------------------
// Gram matrix A^T A (split over rows)                 CholeskyQR for orth(), Alg. 1 l. 2, 4
// ------------------------------------------------------------------------------------
// Power-of-two scale of a Gram operand in the two-term fp16 format.  side 0: P_raw = B Q, whose
// rms is at most rms(B) sqrt(n / r) for an orthonormal Q; side 1: R = B^T P, at most
// rms(B) sqrt(m / r); both brought to about 2^6 .. 2^7, which leaves 2^9 of headroom for
// entries above the rms and saturates beyond.  side 2: a nearly orthonormal factor (entries
// at most about one): 2^12.
constexpr float kGramUnitScale = 4096.f;
OD_DEV float gram_operand_scale(const ClassDims& d, const float* scal, int side, int z) {
  if (side == 2) return kGramUnitScale;
  const float sb = b_scale(d, scal, z);
  const float ratio = side == 0 ? (float)d.n / (float)d.r : (float)d.m / (float)d.r;
  return ldexpf(sb, 6 - ilogbf(ratio) / 2);
}

// waves per SIMD the eight-wave tiles of the r-column products are meant for: two workgroups per CU
template <class T>
constexpr int product_waves() { return T::THREADS == 512 ? 4 : 1; }

struct GramArgs {
  ClassDims d;            // for the operand scale of sides 0 and 1
  const float* scal;
  int rows, r, splits, side;
  WsArr a, part;
};
template <class T, class Num>
OD_DEV void gram_tile(const GramArgs& a_, const SegBlock& blk, char* lds) {
  static_assert(T::MT == T::NT, "the tile grid of a symmetric result must be symmetric");
  const int rows = a_.rows, r = a_.r, splits = a_.splits;
  const int tiles = (r + T::NT - 1) / T::NT;
  // The result is symmetric: only the tiles (tm, tn) with tm <= tn are computed, row by row
  // of the tile grid, and an off-diagonal tile is stored a second time, transposed.
  // All tiles of one row split read the same rows of A.  Workgroups go to the 8 XCDs round robin
  // by their flattened index; each XCD gets one contiguous range of the order (matrix, split,
  // tile), so those tiles run under one L2 and A comes from HBM once.  (Taken per matrix, 20
  // workgroups spread over all XCDs: the counters showed three times the input fetched.)
  const int per_z = blk.grid.x * blk.grid.y;
  const int flat = xcd_contiguous(blk.flat, per_z * blk.grid.z);
  const int z = flat / per_z, logical = flat - z * per_z;
  int tm = 0, tn = logical % blk.grid.x;
  while (tn >= tiles - tm) { tn -= tiles - tm; ++tm; }
  tn += tm;
  const int split = logical / blk.grid.x;
  SrcF32 s{a_.a.base + (int64_t)z * a_.a.stride, rows, r, r};
  int kend;
  const int kbeg = split_begin(rows, splits, T::KT, split, &kend);
  f32x16 acc[T::FM][T::FN];
  zero_acc<T>(acc);
  const float sc = Num::F16 ? gram_operand_scale(a_.d, a_.scal, a_.side, z) : 1.f;
  gemm_mainloop_deep<T, Num, KSF, SrcF32, KSF, SrcF32, (T::THREADS == 512 ? 2 : 3)>(s, s, tm * T::MT, tn * T::NT, kbeg, kend, sc, sc, lds, acc);
  if constexpr (Num::F16) {
    const float inv = 1.f / (sc * sc);
#pragma unroll
    for (int fm = 0; fm < T::FM; ++fm)
#pragma unroll
      for (int fn = 0; fn < T::FN; ++fn)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[fm][fn][v] *= inv;
  }
  float* out = a_.part.base + (int64_t)z * a_.part.stride + (int64_t)split * r * r;
  for_each_acc<T>(acc, tm * T::MT, tn * T::NT, [&](int row, int col, float v) {
    if (row < r && col < r) out[(int64_t)row * r + col] = v;
  });
  if (tm != tn) {
    // lane (c, h) holds rows 8q + 4h .. 8q + 4h + 3 of column c: four consecutive entries of
    // row c of the transposed tile (r is a multiple of 8, so they are inside or outside together)
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave / T::WN, wn = wave % T::WN;
#pragma unroll
    for (int fm = 0; fm < T::FM; ++fm)
#pragma unroll
      for (int fn = 0; fn < T::FN; ++fn) {
        const int col = tn * T::NT + wn * T::WTN + fn * 32 + (lane & 31);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int row0 = tm * T::MT + wm * T::WTM + fm * 32 + 8 * q + 4 * (lane >> 5);
          if (col < r && row0 < r) {
            const f32x4 v4 = {acc[fm][fn][4 * q], acc[fm][fn][4 * q + 1], acc[fm][fn][4 * q + 2], acc[fm][fn][4 * q + 3]};
            *reinterpret_cast<f32x4*>(out + (int64_t)col * r + row0) = v4;
          }
        }
      }
  }
}
template <class T, class Num, class SegsT>
__global__ __launch_bounds__(T::THREADS, product_waves<T>()) void k_gram(SegsT segs) {
  extern __shared__ __align__(16) char lds[];
  OD_SEGMENT(GramArgs);
  gram_tile<T, Num>(a_, blk, lds);
}

// ------------------------------------------------------------------------------------
// out = A W with W upper triangular (the triangular solve of CholeskyQR as a product
// with the explicit inverse factor)
//
// CORR: the second pass of CholeskyQR2 in correction form.  `w` holds Phi(E) (entries far
// below one) and the result is A - A Phi: the product is a small correction of A, so one fp16
// product (A scaled by 2^10, Phi by 2^13: relative error 2^-11 of a term of size |E|) is
// enough, and A itself enters in full fp32 precision.
// ------------------------------------------------------------------------------------
constexpr float kPhiScale = 8192.f;
struct ApplyArgs {
  int rows, r;
  WsArr a, w, out;
  HalfArr wh, hn, ht;
  const MatEntry* q_mats;       // the result goes to these matrices' Q, or to `out` when null
  float* only_q;                // Q of the one matrix of a batch of one
  Pred pred;
};
template <class T, class Num, bool DEEP, bool CORR>
OD_DEV void apply_tile(const ApplyArgs& a_, const SegBlock& blk, char* lds) {
  const int rows = a_.rows, r = a_.r, z = blk.z;
  const HalfArr &hn = a_.hn, &ht = a_.ht, &wh = a_.wh;
  const int tiles_n = (r + T::NT - 1) / T::NT;
  // the column tiles of one row panel of A share an XCD's L2
  const int bid = tiles_n > 1 ? xcd_contiguous(blk.x, blk.grid.x) : blk.x;
  const int tn = bid % tiles_n, tm = bid / tiles_n;
  SrcF32 sa{a_.a.base + (int64_t)z * a_.a.stride, rows, r, r};
  SrcF32 sw{a_.w.base + (int64_t)z * a_.w.stride, r, r, r};
  int kend = (tn + 1) * T::NT;          // W[k][j] = 0 for k > j
  if (kend > r) kend = r;
  f32x16 acc[T::FM][T::FN];
  zero_acc<T>(acc);
  if constexpr (CORR) {
    // Phi arrives as ready operand words (fp16, scaled, transposed to [column][k]): its tiles go
    // to LDS as they are, without the transposition and conversion a fp32 source needs
    SrcH16 swh{wh.base + (int64_t)z * wh.stride, r, r, r};
    if constexpr (DEEP) gemm_mainloop_deep<T, Num, KC, SrcF32, KC, SrcH16, 3>(sa, swh, tm * T::MT, tn * T::NT, 0, kend, kUnitScale, 1.f, lds, acc);
    else gemm_mainloop<T, Num, KC, SrcF32, KC, SrcH16>(sa, swh, tm * T::MT, tn * T::NT, 0, kend, kUnitScale, 1.f, lds, acc);
  } else {
    if constexpr (DEEP) gemm_mainloop_deep<T, Num, KC, SrcF32, KS, SrcF32, 3>(sa, sw, tm * T::MT, tn * T::NT, 0, kend, 1.f, 1.f, lds, acc);
    else gemm_mainloop<T, Num, KC, SrcF32, KS, SrcF32>(sa, sw, tm * T::MT, tn * T::NT, 0, kend, 1.f, 1.f, lds, acc);
  }
  if constexpr (CORR) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave / T::WN, wn = wave % T::WN;
    constexpr float inv = 1.f / (kUnitScale * kPhiScale);
#pragma unroll
    for (int fm = 0; fm < T::FM; ++fm)
#pragma unroll
      for (int fn = 0; fn < T::FN; ++fn)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int row = tm * T::MT + wm * T::WTM + fm * 32 + acc_row(v, lane);
          const int col = tn * T::NT + wn * T::WTN + fn * 32 + acc_col(lane);
          const float a1 = (row < rows && col < r) ? sa.p[(int64_t)row * r + col] : 0.f;
          acc[fm][fn][v] = a1 - inv * acc[fm][fn][v];
        }
  }
  float* dst = a_.only_q != nullptr ? a_.only_q : a_.q_mats != nullptr ? a_.q_mats[z].Q : a_.out.base + (int64_t)z * a_.out.stride;
  for_each_acc<T>(acc, tm * T::MT, tn * T::NT, [&](int row, int col, float v) {
    if (row < rows && col < r) dst[(int64_t)row * r + col] = v;
  });
  // pre-scaled fp16 copies of the (orthonormal) result for the large contractions
  if (hn.base != nullptr) {
    uint16_t* h = hn.base + (int64_t)z * hn.stride;
    for_each_acc<T>(acc, tm * T::MT, tn * T::NT, [&](int row, int col, float v) {
      if (row < rows && col < r) {
        _Float16 x = (_Float16)__builtin_amdgcn_fmed3f(v * kUnitScale, -65504.f, 65504.f);
        h[(int64_t)row * r + col] = __builtin_bit_cast(uint16_t, x);
      }
    });
  }
  if (ht.base != nullptr) {     // transposed [r][rows]: 4 consecutive rows of one column per store
    uint16_t* h = ht.base + (int64_t)z * ht.stride;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / T::WN, wn = wave % T::WN;
#pragma unroll
    for (int fm = 0; fm < T::FM; ++fm)
#pragma unroll
      for (int fn = 0; fn < T::FN; ++fn) {
        const int col = tn * T::NT + wn * T::WTN + fn * 32 + (lane & 31);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int row = tm * T::MT + wm * T::WTM + fm * 32 + 8 * q + 4 * (lane >> 5);
          if (col < r && row < rows) {
            u32x2 hv = {pack_f16_sat(acc[fm][fn][4 * q] * kUnitScale, acc[fm][fn][4 * q + 1] * kUnitScale),
                        pack_f16_sat(acc[fm][fn][4 * q + 2] * kUnitScale, acc[fm][fn][4 * q + 3] * kUnitScale)};
            *reinterpret_cast<u32x2*>(h + (int64_t)col * rows + row) = hv;
          }
        }
      }
  }
}

template <class T, class Num, bool DEEP, bool CORR, class SegsT>
__global__ __launch_bounds__(T::THREADS, product_waves<T>()) void k_apply(SegsT segs) {
  extern __shared__ __align__(16) char lds[];
  OD_SEGMENT(ApplyArgs);
  if (!pred_on(a_.pred, blk.z)) return;
  apply_tile<T, Num, DEEP, CORR>(a_, blk, lds);
}
// The result of the second pass in one launch: the correction where the predicate holds, the full product A W2
// elsewhere (rare; 32-deep steps, so that it needs no more LDS).  For small grids: two launches of which one
// returns at once cost 4 to 5 us more (five small matrices of ranks 24 to 72: 201 -> 197.5 us a step, 2048 x 5632,
// r = 256 with diagnostics 543 -> 539 us).
typedef Tile<64, 64, 32, 2, 2> TileSmallFlat;
OD_DEV void apply_result_tile(const ApplyArgs& a_, const SegBlock& blk, char* lds) {
  if (pred_on(a_.pred, blk.z)) apply_tile<TileSmall, NumF16, true, true>(a_, blk, lds);
  else apply_tile<TileSmallFlat, NumBF<2>, false, false>(a_, blk, lds);
}
template <class SegsT>
__global__ __launch_bounds__(TileSmall::THREADS) void k_apply_result(SegsT segs) {
  extern __shared__ __align__(16) char lds[];
  OD_SEGMENT(ApplyArgs);
  apply_result_tile(a_, blk, lds);
}

// ------------------------------------------------------------------------------------
// r <= 32: the first CholeskyQR pass in one launch.  At this size every kernel of the pass is
// a few microseconds of latency, so three of them become one: every workgroup adds the partials of
// the Gram matrix and factors it for itself in its first wave (one 32 x 32 tile, padded with the
// identity), applies W = T^-1 to its share of the rows in plain fp32 and leaves the Gram
// partial of the rows it has just produced for the second pass.  Workgroup 0 of a matrix also
// writes T1.  One thread per row; `part` receives `splits` partial sums of r x r.
// ------------------------------------------------------------------------------------
// (second launch bound: up to 256 registers, which keeps the matrix-core accumulators in ordinary ones; in the
// others every group of pivots copied them back and forth)
// LDS: S, the rows of one pass ([kSmallRows][kSmallPitch]), then Wl ([32][kSmallPitch])
constexpr int kSmallRows = 256, kSmallPitch = 36;
constexpr int kSmallLds = (kSmallRows + 32) * kSmallPitch * (int)sizeof(float);

// Sum of a^T a over the 64 rows a wave owns of the tile S ([rows][kSmallPitch], 32 columns) on
// the matrix cores: fp32 32x32x2 products with both operands the same register (lane (c, h)
// feeds row 2i + h, column c).
OD_DEV f32x16 small_gram_rows(const float* S, int wave, int lane, f32x16 acc) {
  const float* sw = S + (wave * 64 + (lane >> 5)) * kSmallPitch + (lane & 31);
#pragma unroll 8
  for (int i = 0; i < 32; ++i) {
    const float a = sw[2 * i * kSmallPitch];
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a, a, acc, 0, 0, 0);
  }
  return acc;
}
// The four waves' tiles summed through S (then [wave][32][kSmallPitch]) and stored as r x r.
OD_DEV void small_gram_store(float* S, const f32x16& acc, int r, float* out, int tid) {
  const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
  for (int v = 0; v < 16; ++v) S[(wave * 32 + acc_row(v, lane)) * kSmallPitch + (lane & 31)] = acc[v];
  __syncthreads();
  const int gi = tid >> 3, gj = 4 * (tid & 7);
  f32x4 g = *reinterpret_cast<const f32x4*>(S + gi * kSmallPitch + gj);
#pragma unroll
  for (int w = 1; w < 4; ++w) g += *reinterpret_cast<const f32x4*>(S + (w * 32 + gi) * kSmallPitch + gj);
  if (gi < r && gj < r) *reinterpret_cast<f32x4*>(out + (int64_t)gi * r + gj) = g;
}

// The r x r sum of `splits` Gram partials (r * r apart, added in order) into `S` ([row][kSmallPitch],
// 32 x 32, the identity beyond r): one thread per four entries, so that all partials are in flight
// together; a single wave that added them row block by row block spent 8 round trips to memory on it.
OD_DEV void small_sum_partials(const float* G, int splits, int r, float* S, int tid) {
  const int gi = tid >> 3, gj = 4 * (tid & 7);
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if (gi < r && gj < r) {
    const f32x4* p = reinterpret_cast<const f32x4*>(G + gi * r + gj);
    const int step = r * r / 4;
#pragma unroll 16
    for (int sp = 0; sp < splits; ++sp) v += p[(int64_t)sp * step];
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = gi == gj + e ? 1.f : 0.f;
  }
  *reinterpret_cast<f32x4*>(S + gi * kSmallPitch + gj) = v;
}
// ... and from there to accumulator layout (lane = column c, registers = rows), read through the
// mirrored element of the symmetric matrix
OD_DEV f32x16 small_acc_tile(const float* S, int lane) {
  const int c = lane & 31, h = lane >> 5;
  f32x16 d;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const f32x4 v4 = *reinterpret_cast<const f32x4*>(S + c * kSmallPitch + 8 * q + 4 * h);
#pragma unroll
    for (int e = 0; e < 4; ++e) d[4 * q + e] = v4[e];
  }
  return d;
}
// o = x W for the row x in `xs` (LDS), W upper triangular in `Wl` (zero below the diagonal): column
// block jb takes k <= 4 jb + 3.  Four k per turn of a loop that stays rolled: unrolled, all 144 reads of W
// were issued ahead of the arithmetic and a quarter of them spilled to scratch memory.
OD_DEV void small_row_product(const float* xs, const float* Wl, int r, f32x4* o) {
#pragma unroll
  for (int jb = 0; jb < 8; ++jb) o[jb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
  for (int kb = 0; kb < r / 4; ++kb) {
    const f32x4 x4 = *reinterpret_cast<const f32x4*>(xs + 4 * kb);
#pragma unroll
    for (int jb = 0; jb < 8; ++jb) {
      if (jb >= kb) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const f32x4 w4 = *reinterpret_cast<const f32x4*>(Wl + (4 * kb + i) * kSmallPitch + 4 * jb);
#pragma unroll
          for (int e = 0; e < 4; ++e) o[jb][e] = fmaf(x4[i], w4[e], o[jb][e]);
        }
      }
    }
  }
}

// r <= 32: Gram partials A^T A of `splits` row ranges, one thread per row, in plain fp32.
struct SmallArgs {
  int rows, r, splits, side;
  WsArr a0, a1;
  WsArr gram;                   // `splits` Gram partials of a0, r x r each
  WsArr part;                   // the same of a1
  WsArr t1, t2;
  WsArr w;                      // W1, where the factorisation has run beside that of larger ranks (T1 is written then), or null
  const MatEntry* q_mats;       // the result goes to these matrices' Q, or to a0 when null
  float* only_q;                // Q of the one matrix of a batch of one
  HalfArr hn, ht;               // fp16 copies of the result ([rows][r] and [r][rows]), or null
  float* scal;
  int* info;
};
OD_DEV void small_gram(const SmallArgs& a_, const SegBlock& blk, char* lds) {
  float* S = reinterpret_cast<float*>(lds);
  const int rows = a_.rows, r = a_.r, splits = a_.splits;
  const int z = blk.z, split = blk.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int kend;
  const int kbeg = split_begin(rows, splits, 8, split, &kend);
  const float* A = a_.a0.base + (int64_t)z * a_.a0.stride;
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  for (int base = kbeg; base < kend; base += kSmallRows) {
    const int row = base + tid;
#pragma unroll
    for (int j4 = 0; j4 < 8; ++j4) {
      f32x4 v4 = {0.f, 0.f, 0.f, 0.f};
      if (row < kend && 4 * j4 < r) v4 = *reinterpret_cast<const f32x4*>(A + (int64_t)row * r + 4 * j4);
      *reinterpret_cast<f32x4*>(S + tid * kSmallPitch + 4 * j4) = v4;
    }
    __syncthreads();
    acc = small_gram_rows(S, wave, lane, acc);
    __syncthreads();
  }
  small_gram_store(S, acc, r, a_.gram.base + (int64_t)z * a_.gram.stride + (int64_t)split * r * r, tid);
}

// T1 and W = T1^-1 of the sum in `Wl`, which W replaces (one wave); workgroup 0 of a matrix writes T1
OD_DEV void small_factor(const SmallArgs& a_, float* Wl, int z, int split, int lane) {
  const int r = a_.r;
  const int c = lane & 31, h = lane >> 5;
  f32x16 d = small_acc_tile(Wl, lane), zt;
  const int bad = diag_tile_factor(d, zt, lane, r);
  if (bad != 0 && lane == 0) atomicCAS(&a_.info[z * kInfoPerMat + a_.side], 0, bad);
  // zt = M with W = M^T: lane c holds row c of W
#pragma unroll
  for (int v = 0; v < 16; ++v) Wl[c * kSmallPitch + acc_row(v, lane)] = zt[v];
  if (split == 0 && c < r) {
    float* tp = a_.t1.base + (int64_t)z * a_.t1.stride;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int gi = 8 * q + 4 * h;
      if (gi < r) {
#pragma unroll
        for (int e = 0; e < 4; ++e) tp[(int64_t)(gi + e) * r + c] = d[4 * q + e];
      }
    }
  }
}
OD_DEV void small_first_pass(const SmallArgs& a_, const SegBlock& blk, char* lds) {
  float* S = reinterpret_cast<float*>(lds);                      // the rows of a1 of one pass
  float* Wl = S + kSmallRows * kSmallPitch;                      // W[k][j]
  const int rows = a_.rows, r = a_.r, splits = a_.splits;
  const int z = blk.z, split = blk.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (a_.w.base != nullptr) {
    const int gi = tid >> 3, gj = 4 * (tid & 7);
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (gi < r && gj < r) v = *reinterpret_cast<const f32x4*>(a_.w.base + (int64_t)z * a_.w.stride + gi * r + gj);
    *reinterpret_cast<f32x4*>(Wl + gi * kSmallPitch + gj) = v;
  } else {
    // (Wl holds the sum until the factorisation replaces it by W)
    small_sum_partials(a_.gram.base + (int64_t)z * a_.gram.stride, splits, r, Wl, tid);
    __syncthreads();
    if (wave == 0) small_factor(a_, Wl, z, split, lane);
  }
  int kend;
  const int kbeg = split_begin(rows, splits, 8, split, &kend);
  const float* A = a_.a0.base + (int64_t)z * a_.a0.stride;
  float* O = a_.a1.base + (int64_t)z * a_.a1.stride;
  // Gram of the produced rows, 64 per wave and pass; the four tiles are summed at the end
  f32x16 gacc;
#pragma unroll
  for (int v = 0; v < 16; ++v) gacc[v] = 0.f;
  bool first = true;
  for (int base = kbeg; base < kend; base += kSmallRows) {
    const int row = base + tid;
    const bool valid = row < kend;
    // this thread's row of A waits in its own row of S (which takes the row of a1 further down)
    float* xs = S + tid * kSmallPitch;
#pragma unroll
    for (int j4 = 0; j4 < 8; ++j4) {
      f32x4 v4 = {0.f, 0.f, 0.f, 0.f};
      if (valid && 4 * j4 < r) v4 = *reinterpret_cast<const f32x4*>(A + (int64_t)row * r + 4 * j4);
      *reinterpret_cast<f32x4*>(xs + 4 * j4) = v4;
    }
    // the first rows are requested before the wait for the factorisation
    if (first) { __syncthreads(); first = false; }
    f32x4 o[8];
    small_row_product(xs, Wl, r, o);
#pragma unroll
    for (int jb = 0; jb < 8; ++jb) {
      if (valid && 4 * jb < r) *reinterpret_cast<f32x4*>(O + (int64_t)row * r + 4 * jb) = o[jb];
      *reinterpret_cast<f32x4*>(S + tid * kSmallPitch + 4 * jb) = valid ? o[jb] : f32x4{0.f, 0.f, 0.f, 0.f};
    }
    __syncthreads();
    gacc = small_gram_rows(S, wave, lane, gacc);
    __syncthreads();
  }
  if (first) __syncthreads();          // a workgroup without rows still meets the others' barrier count
  small_gram_store(S, gacc, r, a_.part.base + (int64_t)z * a_.part.stride + (int64_t)split * r * r, tid);
}

// r <= 32, second pass (see k_corr and k_apply for the general form): every workgroup adds the Gram
// partials of a1 (I + E), takes T2 = I + Phi(E) and W2 = I - Phi(E), or the Cholesky factor and its inverse where
// the deviation is too large for the first-order form, and applies W2 to its rows in plain fp32.  Workgroup 0 of
// a matrix also writes T2 and the flags.  One launch in place of four (sum, guard, two triangular products; 22 us of
// launches and latency at 8192 rows, r = 16, against 10).
OD_DEV void small_result(const SmallArgs& a_, const SegBlock& blk, char* lds) {
  float* S = reinterpret_cast<float*>(lds);                      // the rows of a1
  float* Wl = S + kSmallRows * kSmallPitch;                      // I + E, then W2[k][j]
  const int rows = a_.rows, r = a_.r, side = a_.side;
  const int z = blk.z, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row = blk.x * kSmallRows + tid;
  const bool valid = row < rows;
  float* xs = S + tid * kSmallPitch;
  {
    const float* A = a_.a1.base + (int64_t)z * a_.a1.stride + (int64_t)row * r;
#pragma unroll
    for (int j4 = 0; j4 < 8; ++j4) {
      f32x4 v4 = {0.f, 0.f, 0.f, 0.f};
      if (valid && 4 * j4 < r) v4 = *reinterpret_cast<const f32x4*>(A + 4 * j4);
      *reinterpret_cast<f32x4*>(xs + 4 * j4) = v4;
    }
  }
  small_sum_partials(a_.part.base + (int64_t)z * a_.part.stride, a_.splits, r, Wl, tid);
  __syncthreads();
  if (wave == 0) {
    const int c = lane & 31;
    f32x16 d = small_acc_tile(Wl, lane), zt;
    // largest deviation, a NaN counting as a huge one
    float dev = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const float e = fabsf(acc_row(v, lane) == c ? d[v] - 1.f : d[v]);
      dev = e <= dev ? dev : e == e ? e : 3.0e38f;
    }
#pragma unroll
    for (int w = 32; w > 0; w >>= 1) dev = fmaxf(dev, __shfl_xor(dev, w));
    int* flag = &a_.info[z * kInfoPerMat + side];
    if (dev > kFirstOrderDeviation) {
      const int bad = diag_tile_factor(d, zt, lane, r);
      if (blk.x == 0 && lane == 0) {
        if (dev > kMaxGramDeviation) atomicCAS(flag, 0, r);
        if (bad != 0) atomicCAS(flag, 0, bad);
      }
    } else {
      // d = column c, rows i of the symmetric E; zt[v] = W2[c][i]
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int i = acc_row(v, lane);
        const float e = i == c ? d[v] - 1.f : d[v], phi = i == c ? 0.5f * e : e, id = i == c ? 1.f : 0.f;
        d[v] = i <= c ? id + phi : 0.f;
        zt[v] = i >= c ? id - phi : 0.f;
      }
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) Wl[c * kSmallPitch + acc_row(v, lane)] = zt[v];
    if (blk.x == 0) {
      if (c < r) {
        float* tp = a_.t2.base + (int64_t)z * a_.t2.stride;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int i = acc_row(v, lane);
          if (i < r) tp[(int64_t)i * r + c] = d[v];
        }
      }
      // numerical rank from the diagonal of the first pass's factor (see k_corr)
      const float* t = a_.t1.base + (int64_t)z * a_.t1.stride;
      const float dg = t[(int64_t)(c < r ? c : 0) * (r + 1)];
      float lo = dg == dg ? dg : 0.f, hi = dg > 0.f ? dg : 0.f;
#pragma unroll
      for (int w = 16; w > 0; w >>= 1) {
        lo = fminf(lo, __shfl_xor(lo, w));
        hi = fmaxf(hi, __shfl_xor(hi, w));
      }
      if (lane == 0) {
        a_.scal[z * kScalPerMat + 2 + side] = dev;
        if (!(lo > kMinPivotRatio * hi)) atomicCAS(flag, 0, r);
      }
    }
  }
  __syncthreads();
  f32x4 o[8];
  small_row_product(xs, Wl, r, o);
  float* dst = a_.only_q != nullptr ? a_.only_q : a_.q_mats != nullptr ? a_.q_mats[z].Q : a_.a0.base + (int64_t)z * a_.a0.stride;
  if (valid) {
#pragma unroll
    for (int jb = 0; jb < 8; ++jb)
      if (4 * jb < r) *reinterpret_cast<f32x4*>(dst + (int64_t)row * r + 4 * jb) = o[jb];
    if (a_.hn.base != nullptr) {
      uint16_t* hn = a_.hn.base + (int64_t)z * a_.hn.stride + (int64_t)row * r;
#pragma unroll
      for (int jb = 0; jb < 8; ++jb)
        if (4 * jb < r)
          *reinterpret_cast<u32x2*>(hn + 4 * jb) = u32x2{pack_f16_sat(o[jb][0] * kUnitScale, o[jb][1] * kUnitScale),
                                                         pack_f16_sat(o[jb][2] * kUnitScale, o[jb][3] * kUnitScale)};
    }
    if (a_.ht.base != nullptr) {       // adjacent lanes hold adjacent rows: whole segments of every column
      uint16_t* ht = a_.ht.base + (int64_t)z * a_.ht.stride + row;
#pragma unroll
      for (int jb = 0; jb < 8; ++jb)
        if (4 * jb < r) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            ht[(int64_t)(4 * jb + e) * rows] = __builtin_bit_cast(uint16_t, (_Float16)__builtin_amdgcn_fmed3f(o[jb][e] * kUnitScale, -65504.f, 65504.f));
        }
    }
  }
}

// The three stages as kernels of their own, and beside the 64 x 64 tiles that larger ranks of the same launch take
// in their place (Gram matrix, A W, result): workgroups from `first` on belong to the small ranks.  The small
// ranks' arithmetic is the same either way, so a matrix does not depend on the ranks beside it.  Five matrices of
// ranks 24 to 72 take 208 us a step with these and 243 with separate launches; 197 with the larger ranks' kernels
// for all of them, which have 16 bits in A W where the small ranks have 24.
enum SmallStage : int { SMALL_GRAM, SMALL_FIRST, SMALL_RESULT };
template <int STAGE>
OD_DEV void small_stage(const SmallArgs& a_, const SegBlock& blk, char* lds) {
  if constexpr (STAGE == SMALL_GRAM) small_gram(a_, blk, lds);
  else if constexpr (STAGE == SMALL_FIRST) small_first_pass(a_, blk, lds);
  else small_result(a_, blk, lds);
}
template <int STAGE, class SegsT>
__global__ __launch_bounds__(kSmallRows, 2) void k_small(SegsT segs) {
  extern __shared__ __align__(16) char lds[];
  OD_SEGMENT(SmallArgs);
  small_stage<STAGE>(a_, blk, lds);
}
#define OD_SMALL_SEGMENTS(STAGE)                                          \
  if ((int)blockIdx.x >= first) {                                         \
    SegBlock blk;                                                         \
    const int seg_ = seg_locate(small, blk, (int)blockIdx.x - first);     \
    if (seg_ >= 0) small_stage<STAGE>(small.seg[seg_], blk, lds);         \
    return;                                                               \
  }
template <class Num>
__global__ __launch_bounds__(kSmallRows, 2) void k_gram_and_small(Segs<GramArgs> segs, Segs<SmallArgs> small, int first) {
  static_assert(TileSmall::THREADS == kSmallRows, "both kinds of workgroup have the same threads");
  extern __shared__ __align__(16) char lds[];
  OD_SMALL_SEGMENTS(SMALL_GRAM);
  OD_SEGMENT(GramArgs);
  gram_tile<TileSmall, Num>(a_, blk, lds);
}
template <class Num, int STAGE>
__global__ __launch_bounds__(kSmallRows, 2) void k_apply_and_small(Segs<ApplyArgs> segs, Segs<SmallArgs> small, int first) {
  extern __shared__ __align__(16) char lds[];
  OD_SMALL_SEGMENTS(STAGE);
  OD_SEGMENT(ApplyArgs);
  apply_tile<TileSmall, Num, true, false>(a_, blk, lds);
}
__global__ __launch_bounds__(kSmallRows, 2) void k_apply_result_and_small(Segs<ApplyArgs> segs, Segs<SmallArgs> small, int first) {
  extern __shared__ __align__(16) char lds[];
  OD_SMALL_SEGMENTS(SMALL_RESULT);
  OD_SEGMENT(ApplyArgs);
  apply_result_tile(a_, blk, lds);
}

// ------------------------------------------------------------------------------------
// small general product on r x r workspace matrices, used by the blocked Cholesky and
// triangular inverse:  C[cr.., cc..] = alpha * A * B + beta * C over Mc x Nc x Kc with
// block origins that advance affinely with the inner batch index q.
// ------------------------------------------------------------------------------------
struct SgemmArgs {
  WsArr a, b, c;
  int r;                 // all three are r x r, ld r
  int a_r0, a_k0, b_k0, b_c0, c_r0, c_c0;
  int q_step;            // every origin advances by q * q_step
  int nq;
  int Mc, Nc, Kc;
  float alpha, beta;
  Pred pred;
};

template <class D> OD_DEV constexpr bool DirA_is_kc() { return false; }
template <> OD_DEV constexpr bool DirA_is_kc<KC>() { return true; }

OD_DEV SrcF32 sub_view(const float* base, int r, int row0, int col0, int rows, int cols) {
  int R = r - row0, C = r - col0;
  if (R > rows) R = rows;
  if (C > cols) C = cols;
  if (R < 0) R = 0;
  if (C < 0) C = 0;
  return SrcF32{base + (int64_t)row0 * r + col0, R, C, r};
}

// DEEP: three register stages of loads in flight
template <class T, class Num, class DirA, bool DEEP = true>
OD_DEV void sgemm_tile(const SgemmArgs& g, int bx, int bz, char* lds) {
  const int tiles_n = (g.Nc + T::NT - 1) / T::NT;
  const int tn = bx % tiles_n, tm = bx / tiles_n;
  const int q = bz % g.nq, z = bz / g.nq;
  if (!pred_on(g.pred, z)) return;      // uniform over the workgroup: nobody reaches a barrier
  const int o = q * g.q_step;
  const float* ap = g.a.base + (int64_t)z * g.a.stride;
  const float* bp = g.b.base + (int64_t)z * g.b.stride;
  float* cp = g.c.base + (int64_t)z * g.c.stride;
  SrcF32 sa = DirA_is_kc<DirA>() ? sub_view(ap, g.r, g.a_r0 + o, g.a_k0 + o, g.Mc, g.Kc)
                                 : sub_view(ap, g.r, g.a_k0 + o, g.a_r0 + o, g.Kc, g.Mc);
  SrcF32 sb = sub_view(bp, g.r, g.b_k0 + o, g.b_c0 + o, g.Kc, g.Nc);
  f32x16 acc[T::FM][T::FN];
  zero_acc<T>(acc);
  if constexpr (DEEP) gemm_mainloop_deep<T, Num, DirA, SrcF32, KSF, SrcF32, 3>(sa, sb, tm * T::MT, tn * T::NT, 0, g.Kc, 1.f, 1.f, lds, acc);
  else gemm_mainloop<T, Num, DirA, SrcF32, KSF, SrcF32>(sa, sb, tm * T::MT, tn * T::NT, 0, g.Kc, 1.f, 1.f, lds, acc);
  const int cr = g.c_r0 + o, cc = g.c_c0 + o;
  for_each_acc<T>(acc, tm * T::MT, tn * T::NT, [&](int row, int col, float v) {
    if (row < g.Mc && col < g.Nc && cr + row < g.r && cc + col < g.r) {
      float* dst = cp + (int64_t)(cr + row) * g.r + (cc + col);
      float old = g.beta != 0.f ? *dst : 0.f;
      *dst = g.alpha * v + g.beta * old;
    }
  });
}

// diagonal block `blk` of every matrix of a segment's batch; ranks up to 256: the whole factorisation
template <class SegsT>
__global__ __launch_bounds__(kCholThreads) void k_chol256(SegsT segs) {
  extern __shared__ __align__(16) char lds[];
  OD_SEGMENT(CholArgs);
  chol256_block(a_, blk.x, lds);
}

template <class T, class Num, class DirA>
__global__ __launch_bounds__(T::THREADS) void k_sgemm(SgemmArgs g) {
  extern __shared__ __align__(16) char lds[];
  sgemm_tile<T, Num, DirA>(g, blockIdx.x, blockIdx.z, lds);
}

// Two independent products in one launch (the first `tiles1` workgroups of a matrix work on
// g1, the rest on g2): the blocked factorisation is a chain of short launches, and pairing
// the products that do not depend on each other shortens it.
template <class T, class Num, class DirA1, class DirA2>
__global__ __launch_bounds__(T::THREADS) void k_sgemm_pair(SgemmArgs g1, SgemmArgs g2, int tiles1) {
  extern __shared__ __align__(16) char lds[];
  if ((int)blockIdx.x < tiles1) sgemm_tile<T, Num, DirA1>(g1, blockIdx.x, blockIdx.z, lds);
  else sgemm_tile<T, Num, DirA2>(g2, blockIdx.x - tiles1, blockIdx.z, lds);
}

// Look-ahead of the blocked factorisation: workgroup 0 of a matrix factors the next diagonal
// block (whose own update has already been applied) while the others apply the rest of the
// current block's trailing update (g1, g2) and finish block column p of the inverse (g3).
// The products run on the first T::THREADS threads of their workgroups; the surplus waves end
// at once (a barrier counts only the waves that are still alive).  They have the time of a factorisation, so
// one register stage is enough (the registers are those of three waves per SIMD).
template <class T>
__global__ __launch_bounds__(kCholThreads) void k_chol_ahead(CholArgs ca, SgemmArgs g1, SgemmArgs g2, SgemmArgs g3, int tiles1, int tiles2) {
  extern __shared__ __align__(16) char lds[];
  typedef NumBF<3> Num;
  if (blockIdx.x == 0) {
    chol256_block(ca, blockIdx.z, lds);
    return;
  }
  if ((int)threadIdx.x >= T::THREADS) return;
  const int bx = (int)blockIdx.x - 1;
  if (bx < tiles1) sgemm_tile<T, Num, KSF, false>(g1, bx, blockIdx.z, lds);
  else if (bx < tiles1 + tiles2) sgemm_tile<T, Num, KSF, false>(g2, bx - tiles1, blockIdx.z, lds);
  else sgemm_tile<T, Num, KC, false>(g3, bx - tiles1 - tiles2, blockIdx.z, lds);
}

constexpr int kLeaf = kCholMax;   // diagonal block of the blocked factorisation

// ------------------------------------------------------------------------------------
// Second CholeskyQR pass as a first-order correction.  After the first pass the Gram matrix
// is I + E with small E; its Cholesky factor is I + Phi(E) + O(E^2), Phi = strict upper
// triangle + half the diagonal, and the inverse factor I - Phi(E) + O(E^2).  Writes
// T2 = I + Phi(E), W2 = I - Phi(E) and the largest |E| entry (scal[mat][scal_slot]).
// ------------------------------------------------------------------------------------
// Fast precision (phit.base non-null) writes Phi(E)^T as fp16 scaled by 2^13 ([r][r]) instead of W2.  A
// deviation above kMaxGramDeviation (or NaN) is a breakdown: info[mat][info_slot] = r unless already
// set; so is a ratio of the smallest to the largest diagonal entry of t1 below kMinPivotRatio.
struct CorrArgs {
  int r, splits;
  WsArr part, t1, t2, w2;
  HalfArr phit;
  float* scal;
  int scal_slot;
  int* info;
  int info_slot;
};
template <class SegsT>
__global__ __launch_bounds__(256) void k_corr(SegsT segs) {
  OD_SEGMENT(CorrArgs);
  const int r = a_.r, splits = a_.splits, scal_slot = a_.scal_slot, info_slot = a_.info_slot;
  const HalfArr& phit = a_.phit;
  float* scal = a_.scal;
  int* info = a_.info;
  const int z = blk.z;
  const float* src = a_.part.base + (int64_t)z * a_.part.stride;
  float* tp = a_.t2.base + (int64_t)z * a_.t2.stride;
  float* wp = a_.w2.base + (int64_t)z * a_.w2.stride;
  const int64_t count = (int64_t)r * r;
  float emax = 0.f;
  // four consecutive entries of one row per thread (r is a multiple of 8)
  for (int64_t i4 = (int64_t)blk.x * 256 + threadIdx.x; i4 < count / 4; i4 += (int64_t)blk.grid.x * 256) {
    const int i = r <= 32768 ? (int)i4 * 4 / r : (int)(i4 * 4 / r);       // the 32-bit division where it is enough
    const int j0 = (int)(i4 * 4 - (int64_t)i * r);
    f32x4 g = reinterpret_cast<const f32x4*>(src)[i4];
#pragma unroll 8
    for (int sp = 1; sp < splits; ++sp) g += reinterpret_cast<const f32x4*>(src + (int64_t)sp * count)[i4];
    f32x4 to, wo, pt;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int j = j0 + c;
      const float e = (i == j) ? g[c] - 1.f : g[c];
      emax = fmaxf(emax, fabsf(e));
      float phi = 0.f;
      if (j > i) phi = e;
      else if (j == i) phi = 0.5f * e;
      const float id = (i == j) ? 1.f : 0.f;
      to[c] = id + phi;
      wo[c] = id - phi;
      // E is symmetric, so row i of Phi^T (the operand layout [column][k]) is made of the same
      // entries of row i of E, taken below the diagonal instead of above
      float lower = 0.f;
      if (j < i) lower = e;
      else if (j == i) lower = 0.5f * e;
      pt[c] = lower * kPhiScale;
    }
    reinterpret_cast<f32x4*>(tp)[i4] = to;
    if (phit.base == nullptr) {
      reinterpret_cast<f32x4*>(wp)[i4] = wo;
    } else {
      const u32x2 h = {pack_f16_sat(pt[0], pt[1]), pack_f16_sat(pt[2], pt[3])};
      reinterpret_cast<u32x2*>(phit.base + (int64_t)z * phit.stride)[i4] = h;
    }
  }
  __shared__ float red[256];
  red[threadIdx.x] = emax;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + w]);
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    float v = red[0];
    if (!(v == v)) v = 3.0e38f;       // NaN -> huge
    atomicMax(reinterpret_cast<int*>(scal + z * kScalPerMat + scal_slot), __float_as_int(v));
    // The first pass left the factor far from orthonormal: the input had (numerically) less
    // than full column rank, which the Cholesky pivots alone do not always show.
    if (v > kMaxGramDeviation) atomicCAS(&info[z * kInfoPerMat + info_slot], 0, r);
  }
  // Numerical rank: the diagonal of the first pass's triangular factor spans the factor's
  // condition number from below.  Beyond about 1 / sqrt(rounding of the Gram matrix) the small
  // pivots are rounding noise - CholeskyQR would return an orthonormal basis of that noise -
  // so such a matrix is reported as rank deficient whatever deviation the noise happened to leave.
  if (blk.x == 0) {
    const float* t = a_.t1.base + (int64_t)z * a_.t1.stride;
    float lo = 3.0e38f, hi = 0.f;
    for (int i = threadIdx.x; i < r; i += 256) {
      const float d = t[(int64_t)i * r + i];
      lo = fminf(lo, d == d ? d : 0.f);
      hi = fmaxf(hi, d);
    }
    __shared__ float rlo[256], rhi[256];
    rlo[threadIdx.x] = lo;
    rhi[threadIdx.x] = hi;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
      if ((int)threadIdx.x < w) {
        rlo[threadIdx.x] = fminf(rlo[threadIdx.x], rlo[threadIdx.x + w]);
        rhi[threadIdx.x] = fmaxf(rhi[threadIdx.x], rhi[threadIdx.x + w]);
      }
      __syncthreads();
    }
    if (threadIdx.x == 0 && !(rlo[0] > kMinPivotRatio * rhi[0])) atomicCAS(&info[z * kInfoPerMat + info_slot], 0, r);
  }
}

// ------------------------------------------------------------------------------------
// small helpers
// ------------------------------------------------------------------------------------
// zero the r x r matrices of two per-matrix workspace arrays, all matrices in one launch
__global__ __launch_bounds__(256) void k_zero_pair(WsArr a, WsArr b, int64_t count, Pred pred) {
  const int z = blockIdx.y;
  if (!pred_on(pred, z)) return;
  f32x4* pa = reinterpret_cast<f32x4*>(a.base + (int64_t)z * a.stride);
  f32x4* pb = reinterpret_cast<f32x4*>(b.base + (int64_t)z * b.stride);
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < count / 4; i += (int64_t)gridDim.x * 256) {
    pa[i] = zero;
    pb[i] = zero;
  }
}
// ColNorm stage 1: partial column sums of squares over a slab of rows (deterministic).  Four columns per thread and as
// many rows side by side as a workgroup has threads for; stage 2 adds the slabs with 16 threads per column.  (One
// column and one row per thread, one thread per column: 8192 x 64 10.7 + 7.4 us, now 4.8 + 4.6.)
struct ColnormArgs {
  int n, r, slabs;
  WsArr rr, part, colsq;
  int* info;
  const MatEntry* mats;
  HalfArr qh;
};
template <class SegsT>
__global__ __launch_bounds__(256) void k_colsq_partial(SegsT segs) {
  OD_SEGMENT(ColnormArgs);
  const int n = a_.n, r = a_.r, slabs = a_.slabs;
  const WsArr &rr = a_.rr, &part = a_.part;
  const int z = blk.z, slab = blk.y, tid = threadIdx.x;
  const int cols4 = min(64, (r - blk.x * 256) / 4), groups = 256 / cols4;
  const int g = tid / cols4, c = blk.x * 256 + 4 * (tid - g * cols4);
  const int per = (n + slabs - 1) / slabs;
  const int r0 = slab * per, r1 = (r0 + per) < n ? (r0 + per) : n;
  const float* src = rr.base + (int64_t)z * rr.stride + c;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  if (g < groups) {
#pragma unroll 4
    for (int i = r0 + g; i < r1; i += groups) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(src + (int64_t)i * r);
      acc += v * v;
    }
  }
  __shared__ f32x4 red[256];
  red[tid] = acc;
  __syncthreads();
  if (g != 0) return;
  for (int k = 1; k < groups; ++k) acc += red[tid + k * cols4];
  *reinterpret_cast<f32x4*>(part.base + (int64_t)z * part.stride + (int64_t)slab * r + c) = acc;
}
// stage 2: reciprocal column lengths and the zero-column flag
template <class SegsT>
__global__ __launch_bounds__(1024) void k_colsq_final(SegsT segs) {
  OD_SEGMENT(ColnormArgs);
  const int z = blk.z, r = a_.r, g = threadIdx.x >> 6, c = blk.x * 64 + (threadIdx.x & 63);
  const float* p = a_.part.base + (int64_t)z * a_.part.stride + c;
  float s = 0.f;
  if (c < r) {
#pragma unroll 16
    for (int k = g; k < a_.slabs; k += 16) s += p[(int64_t)k * r];
  }
  __shared__ float red[1024];
  red[threadIdx.x] = s;
  __syncthreads();
  if (g != 0 || c >= r) return;
  for (int k = 1; k < 16; ++k) s += red[threadIdx.x + 64 * k];
  const float len = sqrtf(s);
  float inv = 0.f;
  if (len > 1e-30f && len < 3.0e38f) inv = 1.f / len;
  else atomicCAS(&a_.info[z * kInfoPerMat + 2], 0, c + 1);
  a_.colsq.base[(int64_t)z * a_.colsq.stride + c] = inv;
}
// stage 3: Q = R * diag(1/len)
template <class SegsT>
__global__ __launch_bounds__(256) void k_colnorm_apply(SegsT segs) {
  OD_SEGMENT(ColnormArgs);
  const int n = a_.n, r = a_.r, z = blk.z;
  const HalfArr& qh = a_.qh;
  const float* src = a_.rr.base + (int64_t)z * a_.rr.stride;
  const float* inv = a_.colsq.base + (int64_t)z * a_.colsq.stride;
  float* q = a_.mats[z].Q;
  const int64_t n4 = (int64_t)n * r / 4;
  for (int64_t i = (int64_t)blk.x * 256 + threadIdx.x; i < n4; i += (int64_t)blk.grid.x * 256) {
    int c = (int)((i * 4) % r);
    f32x4 v = reinterpret_cast<const f32x4*>(src)[i];
    f32x4 s = *reinterpret_cast<const f32x4*>(inv + c);
    f32x4 o = v * s;
    reinterpret_cast<f32x4*>(q)[i] = o;
    if (qh.base != nullptr) {
      u32x2 h = {pack_f16_sat(o[0] * kUnitScale, o[1] * kUnitScale), pack_f16_sat(o[2] * kUnitScale, o[3] * kUnitScale)};
      reinterpret_cast<u32x2*>(qh.base + (int64_t)z * qh.stride)[i] = h;
    }
  }
}

// ------------------------------------------------------------------------------------
// Error feedback and parameter update in one pass over M, G and X:
//   M_new = a (M + G) - b P R^T     (Alg. 1 line 7 / default form)
//   X_new = X - lr P Q^T            (Alg. 1 lines 5-6)
// The products are computed transposed (tile rows = columns j of the matrix) so that each
// lane owns 4 consecutive j of one row i and moves M, G, X with vector accesses.
// ------------------------------------------------------------------------------------
OD_DEV bool matrix_flagged(const int* info, int z) {
  const int* w = info + z * kInfoPerMat;
  return (w[0] | w[1] | w[2]) != 0;
}

// The fast-precision contractions read B = M + G as fp16 under a scale sampled from 32 rows.
// The pass that sees every entry of B anyway (error feedback) checks the sample: `bmax` is the
// largest |B| this lane has met.
OD_DEV void report_b_range(const ClassDims& d, const float* scal, int* info, int z, float bmax) {
  const float sb = b_scale(d, scal, z);
  int warn = 0;
  if (!(bmax * sb <= 65504.f)) warn |= kWarnBClipped;
  if (bmax > 0.f) {
    const f32x4* p = reinterpret_cast<const f32x4*>(scal + z * kScalPerMat + kScalSample);
    f32x4 acc4 = p[0];
#pragma unroll
    for (int i = 1; i < kStatRows / 4; ++i) acc4 += p[i];
    if ((acc4[0] + acc4[1]) + (acc4[2] + acc4[3]) == 0.f) warn |= kWarnBScaleBlind;
  }
  if (warn != 0) atomicOr(&info[z * kInfoPerMat + kWarnSlot], warn);
}

// Arguments of the error-feedback pass (one segment): fp32 factors (exact) or their fp16 copies.
struct EfxArgs {
  ClassDims d;
  const MatEntry* mats;
  MatEntry only;
  const float* scal;
  int* info;
  WsArr p, rr;
  HalfArr ph, rh, qh;
};
struct EfxCoef { float a, b, lr; };

template <class T, class Num, bool XBF, bool GBF, class SegsT>
__global__ __launch_bounds__(T::THREADS) void k_efx(SegsT segs, EfxCoef coef) {
  extern __shared__ __align__(16) char lds[];
  OD_SEGMENT(EfxArgs);
  const ClassDims& d = a_.d;
  const int* info = a_.info;
  const float a_coef = coef.a;
  const int tiles_i = (d.m + T::NT - 1) / T::NT;
  const int ti = blk.x % tiles_i, tj = blk.x / tiles_i;
  const int z = blk.z;
  const MatEntry mat = OD_MATRIX(z);
  SrcF32 sp{a_.p.base + (int64_t)z * a_.p.stride, d.m, d.r, d.r};
  SrcF32 sr{a_.rr.base + (int64_t)z * a_.rr.stride, d.n, d.r, d.r};
  SrcF32 sq{mat.Q, d.n, d.r, d.r};
  f32x16 acc_r[T::FM][T::FN], acc_q[T::FM][T::FN];
  zero_acc<T>(acc_r);
  zero_acc<T>(acc_q);
  gemm_mainloop<T, Num, KC, SrcF32, KC, SrcF32>(sr, sp, tj * T::MT, ti * T::NT, 0, d.r, 1.f, 1.f, lds, acc_r);
  gemm_mainloop<T, Num, KC, SrcF32, KC, SrcF32>(sq, sp, tj * T::MT, ti * T::NT, 0, d.r, 1.f, 1.f, lds, acc_q);
  const float cr = coef.b, cq = coef.lr;
  if (matrix_flagged(info, z)) {        // unspecified factors (possibly NaN) never reach X and M
    zero_acc<T>(acc_r);
    zero_acc<T>(acc_q);
  }

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / T::WN, wn = wave % T::WN;
  float* Mz = mat.M;
#pragma unroll
  for (int fn = 0; fn < T::FN; ++fn) {
    const int i = ti * T::NT + wn * T::WTN + fn * 32 + (lane & 31);
#pragma unroll
    for (int fm = 0; fm < T::FM; ++fm) {
#pragma unroll
      for (int vq = 0; vq < 4; ++vq) {
        const int j = tj * T::MT + wm * T::WTM + fm * 32 + 8 * vq + 4 * (lane >> 5);
        if (i < d.m && j < d.n) {
          float g[4], x[4];
          if constexpr (GBF) {
            u32x2 gv = *reinterpret_cast<const u32x2*>(reinterpret_cast<const uint16_t*>(mat.G) + (int64_t)i * d.ldg + j);
            g[0] = bf16_lo(gv[0]); g[1] = bf16_hi(gv[0]); g[2] = bf16_lo(gv[1]); g[3] = bf16_hi(gv[1]);
          } else {
            f32x4 gv = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(mat.G) + (int64_t)i * d.ldg + j);
            g[0] = gv[0]; g[1] = gv[1]; g[2] = gv[2]; g[3] = gv[3];
          }
          f32x4* mp = reinterpret_cast<f32x4*>(Mz + (int64_t)i * d.ldm + j);
          f32x4 mv = *mp, mo;
#pragma unroll
          for (int e = 0; e < 4; ++e) mo[e] = a_coef * (mv[e] + g[e]) - cr * acc_r[fm][fn][4 * vq + e];
          *mp = mo;
          if constexpr (XBF) {
            u32x2* xp = reinterpret_cast<u32x2*>(reinterpret_cast<uint16_t*>(mat.X) + (int64_t)i * d.ldx + j);
            u32x2 xv = *xp;
            x[0] = bf16_lo(xv[0]); x[1] = bf16_hi(xv[0]); x[2] = bf16_lo(xv[1]); x[3] = bf16_hi(xv[1]);
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] -= cq * acc_q[fm][fn][4 * vq + e];
            u32x2 xo;
            xo[0] = pack_bf16_rne(x[0], x[1]);
            xo[1] = pack_bf16_rne(x[2], x[3]);
            *xp = xo;
          } else {
            f32x4* xp = reinterpret_cast<f32x4*>(reinterpret_cast<float*>(mat.X) + (int64_t)i * d.ldx + j);
            f32x4 xv = *xp;
#pragma unroll
            for (int e = 0; e < 4; ++e) xv[e] -= cq * acc_q[fm][fn][4 * vq + e];
            *xp = xv;
          }
        }
      }
    }
  }
}

// ------------------------------------------------------------------------------------
// The same pass with every factor already in matrix-core format (fp16, pre-scaled by its
// producer): P [m][r], R [n][r], Q [n][r].  Tile: 128 rows i x 128 columns j, 8 waves.
//   * one K loop feeds both products from one P tile;
//   * wave w owns rows 32 (w % 4) .. +31 and the column half 64 (w / 4) .. +63; the R and Q
//     tiles are laid out in LDS so that lane c of the wave's two accumulator blocks holds
//     columns 2c and 2c + 1: every lane moves pairs, every wave instruction moves whole
//     256-byte (M) or 128-byte (G, X) row segments;
//   * all M, G, X values of the lane are requested together after the K loop; two workgroups
//     per CU (16 waves) overlap one's HBM traffic with the other's products.  (Requests
//     issued before the K loop would not overlap it: the loop's waits for its own operand
//     loads complete in issue order, behind the older requests.)
// ------------------------------------------------------------------------------------
// (second bound: four waves per SIMD, i.e. at most 128 registers, so that two of these 8-wave
// workgroups share a CU as the last point above needs)
// streamed once and not needed again before they are evicted anyway: keep them from pushing the
// factor panels out of L2 (used for long K loops, where the panels are re-read by many tiles)
template <bool STREAM, class V>
OD_DEV V ld_stream(const V* p) {
  if constexpr (STREAM) return __builtin_nontemporal_load(p);
  else return *p;
}
template <bool STREAM, class V>
OD_DEV void st_stream(V* p, V v) {
  if constexpr (STREAM) __builtin_nontemporal_store(v, p);
  else *p = v;
}

template <bool XBF, bool GBF, class SegsT>
__global__ __launch_bounds__(512, 4) void k_efx_h(SegsT segs, EfxCoef coef) {
  constexpr int TJ = 128, TI = 128, KT = 32, PITCH = KT * 2 + 16, PLANE = 128 * PITCH, BUF = 3 * PLANE;
  extern __shared__ __align__(16) char lds[];
  OD_SEGMENT(EfxArgs);
  const ClassDims& d = a_.d;
  const float* scal = a_.scal;
  int* info = a_.info;
  const HalfArr &ph = a_.ph, &rh = a_.rh, &qh = a_.qh;
  const float a_coef = coef.a, b_coef = coef.b, lr = coef.lr;
  const int z = blk.z;
  const MatEntry mat = OD_MATRIX(z);
  const int tiles_i = (d.m + TI - 1) / TI;
  int ti = blk.x % tiles_i, tj = blk.x / tiles_i;
  if (d.col_fast) {
    const int tiles_jj = (d.n + TJ - 1) / TJ;
    tj = blk.x % tiles_jj;
    ti = blk.x / tiles_jj;
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wi = wave & 3, wj = wave >> 2, c = lane & 31;
  SrcH16 sp{ph.base + (int64_t)z * ph.stride, d.m, d.r, d.r};
  SrcH16 sr{rh.base + (int64_t)z * rh.stride, d.n, d.r, d.r};
  SrcH16 sq{qh.base + (int64_t)z * qh.stride, d.n, d.r, d.r};
  // loader: thread t brings 16 bytes (8 k) of row t / 4 of each tile
  const int lrow = tid >> 2, lkg = tid & 3;
  const int jj = lrow & 63;
  const int prow = (lrow & 64) + (jj & 1) * 32 + (jj >> 1);     // LDS position of column lrow of the R / Q tiles
  const int off_p = lrow * PITCH + lkg * 16, off_rq = prow * PITCH + lkg * 16;

  f32x16 acc_r[2], acc_q[2];
#pragma unroll
  for (int f = 0; f < 2; ++f)
#pragma unroll
    for (int v = 0; v < 16; ++v) { acc_r[f][v] = 0.f; acc_q[f][v] = 0.f; }

  u32x4 nr = sr.load8(tj * TJ + lrow, lkg * 8), nq = sq.load8(tj * TJ + lrow, lkg * 8), np = sp.load8(ti * TI + lrow, lkg * 8);
  *reinterpret_cast<u32x4*>(lds + off_rq) = nr;
  *reinterpret_cast<u32x4*>(lds + PLANE + off_rq) = nq;
  *reinterpret_cast<u32x4*>(lds + 2 * PLANE + off_p) = np;
  __syncthreads();
  int buf = 0;
  for (int k = 0; k < d.r; k += KT) {
    const bool more = (k + KT) < d.r;
    if (more) {
      nr = sr.load8(tj * TJ + lrow, k + KT + lkg * 8);
      nq = sq.load8(tj * TJ + lrow, k + KT + lkg * 8);
      np = sp.load8(ti * TI + lrow, k + KT + lkg * 8);
    }
    const char* base = lds + buf * BUF;
#pragma unroll
    for (int kk = 0; kk < KT / 16; ++kk) {
      const int off = c * PITCH + (2 * kk + (lane >> 5)) * 16;
      const u32x4 fp = *reinterpret_cast<const u32x4*>(base + 2 * PLANE + (wi * 32) * PITCH + off);
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        const u32x4 fr = *reinterpret_cast<const u32x4*>(base + (wj * 64 + f * 32) * PITCH + off);
        const u32x4 fq = *reinterpret_cast<const u32x4*>(base + PLANE + (wj * 64 + f * 32) * PITCH + off);
        acc_r[f] = mfma_32x32x16<true>(fp, fr, acc_r[f]);
        acc_q[f] = mfma_32x32x16<true>(fp, fq, acc_q[f]);
      }
    }
    if (more) {
      char* nb = lds + (buf ^ 1) * BUF;
      *reinterpret_cast<u32x4*>(nb + off_rq) = nr;
      *reinterpret_cast<u32x4*>(nb + PLANE + off_rq) = nq;
      *reinterpret_cast<u32x4*>(nb + 2 * PLANE + off_p) = np;
    }
    __syncthreads();
    buf ^= 1;
  }

  // ---- epilogue: this lane's 16 rows x 2 adjacent columns, in two halves of 8 rows; within a
  // half every load is issued before the first store
  const int j0 = tj * TJ + 64 * wj + 2 * c;
  float* __restrict__ Mz = mat.M;
  const char* __restrict__ Gz = reinterpret_cast<const char*>(mat.G);
  char* __restrict__ Xz = reinterpret_cast<char*>(mat.X);
  constexpr int GE = GBF ? 2 : 4, XE = XBF ? 2 : 4;
  const float s_r = r_scale(d, scal, z);
  const float cr = b_coef / (s_r * kUnitScale), cq = lr / (kUnitScale * kUnitScale);
  if (matrix_flagged(info, z)) {        // unspecified factors (possibly NaN) never reach X and M
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
      for (int v = 0; v < 16; ++v) { acc_r[f][v] = 0.f; acc_q[f][v] = 0.f; }
  }
  float bmax = 0.f;
#pragma unroll
  for (int hv = 0; hv < 2; ++hv) {
    f32x2 mv[8], gv[8], xv[8];
    uint32_t gp[8], xp[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int v = 8 * hv + u;
      const int i = ti * TI + 32 * wi + acc_row(v, lane);
      mv[u] = f32x2{0.f, 0.f};
      gp[u] = 0u; xp[u] = 0u; gv[u] = f32x2{0.f, 0.f}; xv[u] = f32x2{0.f, 0.f};
      if (i < d.m && j0 < d.n) {
        mv[u] = *reinterpret_cast<const f32x2*>(Mz + (int64_t)i * d.ldm + j0);
        if constexpr (GBF) gp[u] = *reinterpret_cast<const uint32_t*>(Gz + ((int64_t)i * d.ldg + j0) * GE);
        else gv[u] = *reinterpret_cast<const f32x2*>(Gz + ((int64_t)i * d.ldg + j0) * GE);
        if constexpr (XBF) xp[u] = *reinterpret_cast<const uint32_t*>(Xz + ((int64_t)i * d.ldx + j0) * XE);
        else xv[u] = *reinterpret_cast<const f32x2*>(Xz + ((int64_t)i * d.ldx + j0) * XE);
      }
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int v = 8 * hv + u;
      const int i = ti * TI + 32 * wi + acc_row(v, lane);
      if (i < d.m && j0 < d.n) {
        f32x2 g = gv[u], x = xv[u];
        if constexpr (GBF) g = f32x2{bf16_lo(gp[u]), bf16_hi(gp[u])};
        if constexpr (XBF) x = f32x2{bf16_lo(xp[u]), bf16_hi(xp[u])};
        f32x2 mo, xo;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const float bval = mv[u][e] + g[e];
          bmax = fmaxf(bmax, fabsf(bval));
          mo[e] = a_coef * bval - cr * acc_r[e][v];
          xo[e] = x[e] - cq * acc_q[e][v];
        }
        *reinterpret_cast<f32x2*>(Mz + (int64_t)i * d.ldm + j0) = mo;
        if constexpr (XBF) *reinterpret_cast<uint32_t*>(Xz + ((int64_t)i * d.ldx + j0) * XE) = pack_bf16_rne(xo[0], xo[1]);
        else *reinterpret_cast<f32x2*>(Xz + ((int64_t)i * d.ldx + j0) * XE) = xo;
      }
    }
  }
  report_b_range(d, scal, info, z, bmax);
}

// ------------------------------------------------------------------------------------
// The same pass with direct-to-LDS operand loads.  Tile: 128 rows i x
// 128 columns j, 4 waves; wave (wi, wj) owns rows 64 wi .. +63 and columns 64 wj .. +63 of BOTH
// products: eight 32 x 32 accumulators (two row blocks x even / odd columns x {P R^T, P Q^T}),
// six LDS operand reads for eight matrix-core products per 16-deep step (0.75 per product,
// against 1.25 with 32 x 64 wave tiles).  Three LDS stages of 32-deep P, R, Q tiles are kept
// in flight by `dma16` (od_dma.h), one barrier per step.  The R / Q rows arrive permuted so
// that operand row rho of parity f is column 2 rho + f: lane c then owns the adjacent columns
// 2c, 2c + 1 and every wave instruction of the epilogue moves whole 256-byte (M) or 128-byte
// (G, X) row segments, as in k_efx_h.  Two workgroups per CU (72 KB of LDS each): one streams
// M, G, X while the other multiplies.  WI = 4: 256 rows, one workgroup of eight waves per CU, five stages (four are within
// 0.4 %).
//
// The epilogue is bound by latency as much as by bandwidth: four parts of 8 rows, each a round trip to memory.  Their
// loads go out one part ahead, the first ones ahead of the last products: 8192 x 8192, r = 64, column
// normalised: 424 -> 405 us a step, 4096 x 4096, r = 256: 335 -> 330, 126 matrices of r = 192: 1655 -> 1609.
// ------------------------------------------------------------------------------------
// LDS stages: what fits beside a second workgroup, or all of LDS
constexpr int efx_stages(int wi) { return wi == 4 ? 5 : 3; }
template <bool XBF, bool GBF, bool STREAM, int WI, class SegsT>
__global__ __launch_bounds__(128 * WI, (WI == 2 ? 2 : 1)) void k_efx_d(SegsT segs, EfxCoef coef) {
  constexpr int TI = 64 * WI, TJ = 128, KT = 32, ROWB = KT * 2, ST = efx_stages(WI), NW = 2 * WI;
  constexpr int PLANE = 128 * ROWB, STAGE = 2 * PLANE + TI * ROWB;       // R | Q | P
  constexpr int CPW = (16 + TI / 16) / NW;                    // 1 KB chunks per wave and stage
  extern __shared__ __align__(16) char lds[];
  OD_SEGMENT(EfxArgs);
  const ClassDims& d = a_.d;
  const float* scal = a_.scal;
  int* info = a_.info;
  const HalfArr &ph = a_.ph, &rh = a_.rh, &qh = a_.qh;
  const float a_coef = coef.a, b_coef = coef.b, lr = coef.lr;
  const int z = blk.z;
  const MatEntry mat = OD_MATRIX(z);
  const int tiles_i = (d.m + TI - 1) / TI;
  int ti = blk.x % tiles_i, tj = blk.x / tiles_i;
  if (d.col_fast) {
    const int tiles_jj = (d.n + TJ - 1) / TJ;
    tj = blk.x % tiles_jj;
    ti = blk.x / tiles_jj;
  }
  if (d.r > 256) {
    // Long K loops re-read the panels of P, R and Q often enough to matter: bands of eight tile
    // columns, row-major inside a band, one contiguous range of that order per XCD, so that the
    // workgroups an XCD holds at a time form a block of tiles and every panel fetched
    // into its L2 serves eight of them (measured -4 to -5 %; at r = 256 the plain order is 2 us
    // faster).
    const int tiles_j = (d.n + TJ - 1) / TJ;
    const int logical = xcd_contiguous(blk.x, blk.grid.x);
    const int band = logical / (tiles_i * 8);
    const int in_band = logical - band * tiles_i * 8;
    const int bw = min(8, tiles_j - band * 8);
    ti = in_band / bw;
    tj = band * 8 + in_band % bw;
  }
  const int tid = threadIdx.x, lane = tid & 63, c = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wi = wave % WI, wj = wave / WI;

  // ---- this lane's share of every stage: chunk = 16 LDS rows of one of the three tiles
  const uint16_t* gp[CPW];
  uint32_t loff[CPW];
  int kgq[CPW];
  const uint32_t lds0 = lds_offset_of(lds);
#pragma unroll
  for (int q = 0; q < CPW; ++q) {
    const int chunk = wave + NW * q;                // 0..7 R, 8..15 Q, 16.. P
    const int which = chunk < 16 ? chunk >> 3 : 2, rel = chunk < 16 ? chunk & 7 : chunk - 16;
    const int row = rel * 16 + (lane >> 2), slot = lane & 3;
    const int kg = slot ^ swz32(row);
    kgq[q] = kg;
    int grow;
    const uint16_t* base;
    if (which == 2) {
      grow = min(ti * TI + row, d.m - 1);
      base = ph.base + (int64_t)z * ph.stride;
    } else {
      const int col = (row & 64) + 2 * (row & 31) + ((row >> 5) & 1);     // LDS row -> tile column
      grow = min(tj * TJ + col, d.n - 1);
      base = (which == 0 ? rh.base + (int64_t)z * rh.stride : qh.base + (int64_t)z * qh.stride);
    }
    gp[q] = base + (int64_t)grow * d.r + kg * 8;
    loff[q] = lds0 + which * PLANE + rel * 1024;
  }
  // The last step of a rank that is no multiple of 32 holds fewer k: its groups of eight beyond the rank read the
  // row's last group once more, and those of P are zeroed in LDS before the products.
  const int nsteps = (d.r + KT - 1) / KT, tail = d.r % KT;
  auto issue = [&](int step) {
    const uint32_t boff = (uint32_t)(step % ST) * STAGE;
    if (tail != 0 && step == nsteps - 1) {
#pragma unroll
      for (int q = 0; q < CPW; ++q) dma16(gp[q] + step * KT - max(kgq[q] * 8 + 8 - tail, 0), loff[q] + boff);
    } else {
#pragma unroll
      for (int q = 0; q < CPW; ++q) dma16(gp[q] + step * KT, loff[q] + boff);
    }
  };

  f32x16 acc_r[2][2], acc_q[2][2];
#pragma unroll
  for (int fm = 0; fm < 2; ++fm)
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
      for (int v = 0; v < 16; ++v) { acc_r[fm][f][v] = 0.f; acc_q[fm][f][v] = 0.f; }

#pragma unroll
  for (int s = 0; s < ST - 1; ++s)
    if (s < nsteps) issue(s);

  const int prow = wi * 64 + c, jrow = wj * 64 + c;
  auto products = [&](int i) {
    const char* base = lds + (i % ST) * STAGE;
#pragma unroll
    for (int kk = 0; kk < KT / 16; ++kk) {
      const int kg = 2 * kk + (lane >> 5);
      u32x4 fp[2], fr[2], fq[2];
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        const int rp = prow + 32 * f, rj = jrow + 32 * f;
        fp[f] = *reinterpret_cast<const u32x4*>(base + 2 * PLANE + rp * ROWB + ((kg ^ swz32(rp)) * 16));
        fr[f] = *reinterpret_cast<const u32x4*>(base + rj * ROWB + ((kg ^ swz32(rj)) * 16));
        fq[f] = *reinterpret_cast<const u32x4*>(base + PLANE + rj * ROWB + ((kg ^ swz32(rj)) * 16));
      }
#pragma unroll
      for (int fm = 0; fm < 2; ++fm)
#pragma unroll
        for (int f = 0; f < 2; ++f) {
          acc_r[fm][f] = mfma_32x32x16<true>(fp[fm], fr[f], acc_r[fm][f]);
          acc_q[fm][f] = mfma_32x32x16<true>(fp[fm], fq[f], acc_q[fm][f]);
        }
    }
  };
  // the last steps, whose stages are waited for together, so that the epilogue's first loads can go out ahead of them
  constexpr int LAST = ST - 2;
  const int main_steps = nsteps > LAST ? nsteps - LAST : 0;
  for (int i = 0; i < main_steps; ++i) {
    // stage i has landed when at most the loads of the younger stages are outstanding
    if (i + ST - 2 < nsteps) __builtin_amdgcn_s_waitcnt(vmcnt_only((ST - 2) * CPW));
    else __builtin_amdgcn_s_waitcnt(vmcnt_only(0));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (i + ST - 1 < nsteps) issue(i + ST - 1);       // into the buffer every wave has finished reading
    products(i);
  }
  __builtin_amdgcn_s_waitcnt(vmcnt_only(0));
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  if (tail != 0) {
    char* p = lds + ((nsteps - 1) % ST) * STAGE + 2 * PLANE;
    for (int row = tid; row < TI; row += 128 * WI)
      for (int kg = tail / 8; kg < 4; ++kg) *reinterpret_cast<u32x4*>(p + row * ROWB + ((kg ^ swz32(row)) * 16)) = u32x4{0u, 0u, 0u, 0u};
    __syncthreads();
  }

  // ---- epilogue: 2 row blocks x 16 rows x 2 adjacent columns per lane, in four parts of 8 rows.  The loads of a part
  // go out before the arithmetic and stores of the part before it, those of the first one before the last
  // products.  Addresses are clamped into the matrix, stores are not made outside.
  const int j0 = tj * TJ + 64 * wj + 2 * c, jc = min(j0, d.n - 2);
  float* __restrict__ Mz = mat.M;
  const char* __restrict__ Gz = reinterpret_cast<const char*>(mat.G);
  char* __restrict__ Xz = reinterpret_cast<char*>(mat.X);
  constexpr int GE = GBF ? 2 : 4, XE = XBF ? 2 : 4;
  struct Part {
    f32x2 m[8];
    typename std::conditional<GBF, uint32_t, f32x2>::type g[8];
    typename std::conditional<XBF, uint32_t, f32x2>::type x[8];
  };
  auto row_of = [&](int part, int u) { return ti * TI + 64 * wi + 32 * (part >> 1) + acc_row(8 * (part & 1) + u, lane); };
  auto fetch = [&](int part, Part& v) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int64_t i = min(row_of(part, u), d.m - 1);
      v.m[u] = ld_stream<STREAM>(reinterpret_cast<const f32x2*>(Mz + i * d.ldm + jc));
      v.g[u] = ld_stream<STREAM>(reinterpret_cast<const decltype(v.g[u] + 0)*>(Gz + (i * d.ldg + jc) * GE));
      v.x[u] = ld_stream<STREAM>(reinterpret_cast<const decltype(v.x[u] + 0)*>(Xz + (i * d.ldx + jc) * XE));
    }
  };
  Part even;
  fetch(0, even);
  __builtin_amdgcn_sched_barrier(0);
  for (int i = main_steps; i < nsteps; ++i) products(i);

  const float s_r = r_scale(d, scal, z);
  const float cr = b_coef / (s_r * kUnitScale), cq = lr / (kUnitScale * kUnitScale);
  if (matrix_flagged(info, z)) {        // unspecified factors (possibly NaN) never reach X and M
#pragma unroll
    for (int fm = 0; fm < 2; ++fm)
#pragma unroll
      for (int f = 0; f < 2; ++f)
#pragma unroll
        for (int v = 0; v < 16; ++v) { acc_r[fm][f][v] = 0.f; acc_q[fm][f][v] = 0.f; }
  }
  float bmax = 0.f;
  auto update = [&](int part, const Part& in) {
    const int fm = part >> 1;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int v = 8 * (part & 1) + u, i = row_of(part, u);
      f32x2 g, x;
      if constexpr (GBF) g = f32x2{bf16_lo(in.g[u]), bf16_hi(in.g[u])};
      else g = in.g[u];
      if constexpr (XBF) x = f32x2{bf16_lo(in.x[u]), bf16_hi(in.x[u])};
      else x = in.x[u];
      f32x2 bval, mo, xo;
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        bval[e] = in.m[u][e] + g[e];
        mo[e] = a_coef * bval[e] - cr * acc_r[fm][e][v];
        xo[e] = x[e] - cq * acc_q[fm][e][v];
      }
      // At a clamped address the owner may have stored its new M already, which is no entry of B.  Groups of eight rows lie
      // inside or outside together; columns follow at the end.
      const float bm = fmaxf(fmaxf(bmax, fabsf(bval[0])), fabsf(bval[1]));
      bmax = ti * TI + 64 * wi + 32 * fm + 8 * (v >> 2) < d.m ? bm : bmax;
      if (i < d.m && j0 < d.n) {
        st_stream<STREAM>(reinterpret_cast<f32x2*>(Mz + (int64_t)i * d.ldm + j0), mo);
        if constexpr (XBF) st_stream<STREAM>(reinterpret_cast<uint32_t*>(Xz + ((int64_t)i * d.ldx + j0) * XE), pack_bf16_rne(xo[0], xo[1]));
        else st_stream<STREAM>(reinterpret_cast<f32x2*>(Xz + ((int64_t)i * d.ldx + j0) * XE), xo);
      }
    }
  };
  if constexpr (XBF && GBF) {
    Part odd;
    fetch(1, odd);
    __builtin_amdgcn_sched_barrier(0);
    update(0, even);
    __builtin_amdgcn_sched_barrier(0);
    fetch(2, even);
    __builtin_amdgcn_sched_barrier(0);
    update(1, odd);
    __builtin_amdgcn_sched_barrier(0);
    fetch(3, odd);
    __builtin_amdgcn_sched_barrier(0);
    update(2, even);
    update(3, odd);
  } else {                  // wider elements leave no registers for a second part
    update(0, even);
#pragma unroll
    for (int part = 1; part < 4; ++part) {
      __builtin_amdgcn_sched_barrier(0);
      fetch(part, even);
      __builtin_amdgcn_sched_barrier(0);
      update(part, even);
    }
  }
  report_b_range(d, scal, info, z, j0 < d.n ? bmax : 0.f);
}

// ------------------------------------------------------------------------------------
// Projection and back-projection with every global load direct to LDS (fast precision, bf16
// gradients, r > 64):
//   TRANS = false   out[i][c] = sum_j (M + G)[i][j] Qt[c][j]     P_raw = B Q      (Alg. 1 line 2)
//   TRANS = true    out[j][c] = sum_i (M + G)[i][j] Pt[c][i]     R = B^T P        (Alg. 1 line 3)
// One workgroup (8 waves, 2 x 4) computes 128 output rows x NT = 128, 256 or 512 columns over a K range; wave
// tile 64 x NT / 4.  Per 32-deep step:
//   * the factor operand (Qt / Pt: fp16 words, k contiguous) arrives by `dma16` in the swizzled
//     layout of od_dma.h, SB stages: two at NT = 512, three below;
//   * the streamed operand arrives raw - the fp32 tile of M and the bf16 tile of G, exactly as
//     they lie in memory - by `dma16` into three staging stages, so two steps of HBM traffic
//     (48 KB per CU) are in flight with no staging registers and no compiler-scheduled waits;
//     all threads then turn one raw stage into fp16 operand words of (M + G) * scale in a
//     double-buffered operand tile while the matrix cores work on the previous one;
//   * TRANS: the operand tile keeps memory's [k = i][j] order and the wave reads its
//     [row = j][8 consecutive k] fragments with the LDS transpose read (`ds_read_b64_tr_b16`:
//     within 16 lanes, lane c receives element c % 4 of the 8 bytes addressed by lanes
//     4 e + c / 4, e = 0..3; so lanes 4 e + q address row k0 + e, columns j0 + 4 q .. + 3, and
//     lane c receives k0 .. k0 + 3 of column j0 + c); rows are 320 bytes apart so that the four
//     rows a half-wave touches fall into different banks.
// One barrier per step.  Waits count loads: per step and wave kCB factor loads, then kNR raw loads.
// ------------------------------------------------------------------------------------
template <bool TRANS, int NT, int SB, class SegsT>
__global__ __launch_bounds__(512, 1) void k_stream_d(SegsT segs) {
  constexpr int MT = 128, KT = 32, ROWB = 64, SR = 3;
  constexpr int FN = NT / 128;                                // 32-column accumulator blocks per wave
  constexpr int B_STAGE = NT * ROWB, RAW_M = MT * KT * 4, RAW_G = MT * KT * 2, RAW_STAGE = RAW_M + RAW_G;
  constexpr int A_PITCH = TRANS ? 320 : ROWB, A_ROWS = TRANS ? KT : MT, A_BYTES = A_ROWS * A_PITCH;
  constexpr int OFF_RAW = SB * B_STAGE, OFF_A = OFF_RAW + SR * RAW_STAGE;
  constexpr int kCB = NT / 16 / 8, kNR = 3;                   // 1 KB chunks per wave: factor stage, raw stage (2 of M, 1 of G)
  extern __shared__ __align__(16) char lds[];
  OD_SEGMENT(StreamArgs);
  const ClassDims& d = a_.d;
  const float* scal = a_.scal;
  int* info = a_.info;
  const HalfArr &fh = a_.fh, &rh = a_.rh;
  const int splits = a_.splits, rotate = a_.rotate;
  const int Mdim = TRANS ? d.n : d.m, Kdim = TRANS ? d.m : d.n;
  const int tiles_n = (d.r + NT - 1) / NT;
  // Workgroups go to the 8 XCDs round robin by their flattened index.  Each XCD gets one
  // contiguous range of the order (matrix, split, row panel, column tile): the workgroups that
  // run side by side under one L2 then read the same k range of the same factor operand (and
  // the column tiles of a row panel the same raw tile), instead of 16 different ones.
  const int per_z = blk.grid.x * blk.grid.y;
  const int logical = xcd_contiguous(blk.flat, per_z * blk.grid.z);
  const int z = logical / per_z, in_z = logical - z * per_z;
  const int split = in_z / blk.grid.x, bid = in_z - split * blk.grid.x;
  const int tn = bid % tiles_n, tm = bid / tiles_n;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  int kend;
  const int kbeg = split_begin(Kdim, splits, KT, split, &kend);
  const int nsteps = kend > kbeg ? (kend - kbeg + KT - 1) / KT : 0;
  // rotated k order (the projection of one matrix whose rows lie a multiple of 32 KB apart):
  // every row panel starts its k range `rotate` steps after the panel before it, otherwise all
  // panels would read the same columns - the same memory channels - in lockstep
  const int rot = (rotate > 0 && nsteps > 0) ? (int)(((int64_t)tm * rotate) % nsteps) : 0;
  auto k_of = [&](int step) {
    int s2 = step + rot;
    if (s2 >= nsteps) s2 -= nsteps;
    return kbeg + s2 * KT;
  };
  const float sa = b_scale(d, scal, z);
  const uint32_t lds0 = lds_offset_of(lds);
  const MatEntry mat = OD_MATRIX(z);
  const float* Mz = mat.M;
  const uint16_t* Gz = reinterpret_cast<const uint16_t*>(mat.G);
  const uint16_t* Fz = fh.base + (int64_t)z * fh.stride;      // [r][Kdim]

  // ---- factor operand: chunk = 16 rows (output columns) x 64 bytes
  const uint16_t* fp[kCB];
  uint32_t foff[kCB];
#pragma unroll
  for (int q = 0; q < kCB; ++q) {
    const int chunk = wave + 8 * q;
    const int row = chunk * 16 + (lane >> 2), kg = (lane & 3) ^ swz32(row);
    fp[q] = Fz + (int64_t)min(tn * NT + row, d.r - 1) * Kdim + kg * 8;
    foff[q] = lds0 + chunk * 1024;
  }
  // ---- raw operand: M chunks of 1 KB (not TRANS: 8 rows x 128 B; TRANS: 2 rows x 512 B), G
  // chunks of 1 KB (16 rows x 64 B; 4 rows x 256 B).  Wave w moves M chunks w and w + 8 and G chunk w.
  // Addresses are clamped into the matrix; what lies outside is zeroed at conversion.
  int64_t raw_off[kNR];          // element offset of this lane's 16 bytes at k step 0
  uint32_t roff[kNR];
#pragma unroll
  for (int q = 0; q < kNR; ++q) {
    const bool isg = q == 2;
    const int chunk = isg ? wave : wave + 8 * q;
    int row, col;                // within the tile: row along the matrix's rows, col along its columns
    if (!TRANS) {
      row = isg ? chunk * 16 + (lane >> 2) : chunk * 8 + (lane >> 3);
      col = isg ? (lane & 3) * 8 : (lane & 7) * 4;
    } else {
      row = isg ? chunk * 4 + (lane >> 4) : chunk * 2 + (lane >> 5);
      col = isg ? (lane & 15) * 8 : (lane & 31) * 4;
    }
    // not TRANS: rows are output rows (fixed), columns advance with k; TRANS: the other way round
    const int grow = TRANS ? row : min(tm * MT + row, d.m - 1);
    const int gcol = TRANS ? min(tm * MT + col, d.n - (isg ? 8 : 4)) : col;
    raw_off[q] = (int64_t)grow * (isg ? d.ldg : d.ldm) + gcol;
    roff[q] = lds0 + OFF_RAW + (isg ? RAW_M : 0) + chunk * 1024;
  }
  auto issue_f = [&](int step) {
    const uint32_t boff = (uint32_t)(step % SB) * B_STAGE;
    const int k0 = min(k_of(step), Kdim - KT);                // a clamped step only meets zeros of the other operand
#pragma unroll
    for (int q = 0; q < kCB; ++q) dma16(fp[q] + k0, foff[q] + boff);
  };
  auto issue_raw = [&](int step) {
    const uint32_t boff = (uint32_t)(step % SR) * RAW_STAGE;
    const int k0 = k_of(step);
#pragma unroll
    for (int q = 0; q < kNR; ++q) {
      const bool isg = q == 2;
      int64_t off;
      if (!TRANS) off = raw_off[q] + min(k0, d.n - KT);        // clamped like the factor operand
      else off = raw_off[q] + (int64_t)min(k0, d.m - KT) * (isg ? d.ldg : d.ldm);
      if (isg) dma16(Gz + off, roff[q] + boff);
      else dma16(Mz + off, roff[q] + boff);
    }
  };
  // A step whose k range was clamped re-reads earlier k positions: conversion zeroes every k
  // outside [k0, kend) of the step, and every row / column outside the matrix.
  auto convert = [&](int step) {
    const char* raw = lds + OFF_RAW + (step % SR) * RAW_STAGE;
    char* abuf = lds + OFF_A + (step & 1) * A_BYTES;
    const int k0 = k_of(step);
    const int kld = TRANS ? min(k0, d.m - KT) : min(k0, d.n - KT);       // where the loaded tile really starts
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int e = tid + 512 * h;                             // 16 bytes of M = 4 elements each
      const f32x4 mv = *reinterpret_cast<const f32x4*>(raw + e * 16);
      const u32x2 gv = *reinterpret_cast<const u32x2*>(raw + RAW_M + e * 8);
      int row, col;                                            // tile row along the matrix's rows, column along its columns
      if (!TRANS) { row = e >> 3; col = (e & 7) * 4; }
      else { row = e >> 5; col = (e & 31) * 4; }
      const int kk = (TRANS ? row : col) + kld;                // global k of the first element
      float x[4] = {mv[0] + bf16_lo(gv[0]), mv[1] + bf16_hi(gv[0]), mv[2] + bf16_lo(gv[1]), mv[3] + bf16_hi(gv[1])};
      bool ok;
      if (!TRANS) ok = tm * MT + row < d.m && kk >= k0 && kk < kend;       // k advances in groups of 4 inside multiples of 8
      else ok = kk >= k0 && kk < kend && tm * MT + col < d.n;
      if (!TRANS && tm * MT + row >= d.m) ok = false;
      u32x2 w = {0u, 0u};
      if (ok) { w[0] = pack_f16_sat(x[0] * sa, x[1] * sa); w[1] = pack_f16_sat(x[2] * sa, x[3] * sa); }
      if (!TRANS) {
        const int kg = col >> 3;
        *reinterpret_cast<u32x2*>(abuf + row * ROWB + ((kg ^ swz32(row)) * 16) + (col & 4) * 2) = w;
      } else {
        *reinterpret_cast<u32x2*>(abuf + row * A_PITCH + col * 2) = w;
      }
    }
  };

  f32x16 acc[2][FN];
#pragma unroll
  for (int fm = 0; fm < 2; ++fm)
#pragma unroll
    for (int fn = 0; fn < FN; ++fn)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[fm][fn][v] = 0.f;

  if (nsteps > 0) {
    issue_raw(0);
    issue_f(0);
    if (nsteps > 1) issue_raw(1);
    if (SB == 3 && nsteps > 1) issue_f(1);
    if (nsteps > 2) issue_raw(2);
    if (nsteps > 2) __builtin_amdgcn_s_waitcnt(vmcnt_only(2 * kNR + (SB == 3 ? kCB : 0)));
    else __builtin_amdgcn_s_waitcnt(vmcnt_only(0));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    convert(0);
  }
  const int arow = wm * 64 + (lane & 31), brow = wn * (NT / 4) + (lane & 31);
  for (int i = 0; i < nsteps; ++i) {
    // factor stage i and raw stage i + 1 have landed when only raw stage i + 2 (and, with three
    // factor stages, factor stage i + 1 issued before it) is outstanding
    if (i + 2 < nsteps) __builtin_amdgcn_s_waitcnt(vmcnt_only(kNR + (SB == 3 ? kCB : 0)));
    else __builtin_amdgcn_s_waitcnt(vmcnt_only(0));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (i + SB - 1 < nsteps) issue_f(i + SB - 1);
    if (i + 3 < nsteps) issue_raw(i + 3);
    if (i + 1 < nsteps) convert(i + 1);
    const char* ab = lds + OFF_A + (i & 1) * A_BYTES;
    const char* bb = lds + (i % SB) * B_STAGE;
#pragma unroll
    for (int kk = 0; kk < KT / 16; ++kk) {
      const int kg = 2 * kk + (lane >> 5);
      u32x4 af[2], bf[FN];
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        if constexpr (!TRANS) {
          const int r0 = arow + 32 * f;
          af[f] = *reinterpret_cast<const u32x4*>(ab + r0 * ROWB + ((kg ^ swz32(r0)) * 16));
        } else {
          // lane l = 16 b + i: addresses row k = 16 kk + 8 (b >> 1) + i / 4 (+ 4), columns j0 + 16 (b & 1) + 4 (i % 4)
          const int b = lane >> 4, ii = lane & 15;
          const int k = 16 * kk + 8 * (b >> 1) + (ii >> 2);
          const int j = wm * 64 + 32 * f + 16 * (b & 1) + 4 * (ii & 3);
          const char* p0 = ab + k * A_PITCH + j * 2;
          const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p0));
          const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p0 + 4 * A_PITCH));
          const u32x2 l2 = __builtin_bit_cast(u32x2, lo), h2 = __builtin_bit_cast(u32x2, hi);
          af[f] = u32x4{l2[0], l2[1], h2[0], h2[1]};
        }
      }
#pragma unroll
      for (int f = 0; f < FN; ++f) {
        const int r0 = brow + 32 * f;
        bf[f] = *reinterpret_cast<const u32x4*>(bb + r0 * ROWB + ((kg ^ swz32(r0)) * 16));
      }
#pragma unroll
      for (int fm = 0; fm < 2; ++fm)
#pragma unroll
        for (int fn = 0; fn < FN; ++fn) acc[fm][fn] = mfma_32x32x16<true>(af[fm], bf[fn], acc[fm][fn]);
    }
  }
  const float inv = 1.f / (sa * kUnitScale);
  float* out = a_.part.base + (int64_t)z * a_.part.stride + (int64_t)split * Mdim * d.r;
#pragma unroll
  for (int fm = 0; fm < 2; ++fm)
#pragma unroll
    for (int fn = 0; fn < FN; ++fn)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = tm * MT + wm * 64 + fm * 32 + acc_row(v, lane);
        const int col = tn * NT + wn * (NT / 4) + fn * 32 + acc_col(lane);
        if (row < Mdim && col < d.r) out[(int64_t)row * d.r + col] = acc[fm][fn][v] * inv;
      }
  // A single split of the back-projection is R itself: its pre-scaled fp16 copy (what
  // k_reduce_r would make in a pass of its own) is written here, with the same range check.
  if (TRANS && rh.base != nullptr) {
    const float sr = r_scale(d, scal, z) * inv;
    uint16_t* dh = rh.base + (int64_t)z * rh.stride;
    float rmax = 0.f;
#pragma unroll
    for (int fm = 0; fm < 2; ++fm)
#pragma unroll
      for (int fn = 0; fn < FN; ++fn)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int row = tm * MT + wm * 64 + fm * 32 + acc_row(v, lane);
          const int col = tn * NT + wn * (NT / 4) + fn * 32 + acc_col(lane);
          if (row < Mdim && col < d.r) {
            const float x = acc[fm][fn][v] * sr;
            rmax = fmaxf(rmax, fabsf(x));
            dh[(int64_t)row * d.r + col] = __builtin_bit_cast(uint16_t, (_Float16)__builtin_amdgcn_fmed3f(x, -65504.f, 65504.f));
          }
        }
    if (!(rmax <= 65504.f)) atomicOr(&info[z * kInfoPerMat + kWarnSlot], kWarnRClipped);
  }
}

// ====================================================================================
// launchers
// ====================================================================================
#define OD_CHECK_LAUNCH()                       \
  do {                                          \
    hipError_t e_ = hipGetLastError();          \
    if (e_ != hipSuccess) return e_;            \
  } while (0)
#define OD_RETURN_IF(expr)                      \
  do {                                          \
    const hipError_t e_ = (expr);               \
    if (e_ != hipSuccess) return e_;            \
  } while (0)

// One-shot timing of the next streaming phase (projection, back-projection, error feedback): the
// events receive the start time stamp of its first dispatch and the stop time stamp of its last
// one, without the gaps around separately recorded events.
static thread_local hipEvent_t g_time_start = nullptr, g_time_stop = nullptr;
void time_next_launch(hipEvent_t start, hipEvent_t stop) { g_time_start = start; g_time_stop = stop; }

template <class K>
static hipError_t allow_lds(K kernel, int bytes) {
  if (bytes > 64 * 1024) return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  return hipSuccess;
}

// The segments of one launch.
template <class A>
struct SegList {
  Segs<A> g;
  int total;
  SegList() : g{}, total(0) {}
  bool full() const { return g.n == kMaxSeg; }
  void add(const A& a, int x, int y, int z) {
    g.first[g.n] = total;
    g.grid[g.n] = SegGrid{x, y, z};
    g.seg[g.n] = a;
    total += (x * y * z + 7) / 8 * 8;         // segments start at multiples of 8 workgroups (see above)
    ++g.n;
  }
  // enqueues what was added, with `single` for one segment and `multi` for several; `timed` bit 0 / 1:
  // the first / last launch of a timed phase
  template <class K1, class K2, class... Extra>
  hipError_t launch(K1 single, K2 multi, int threads, int lds, hipStream_t st, int timed, Extra... extra) {
    if (g.n == 0) return hipSuccess;
    hipEvent_t e0 = (timed & 1) ? g_time_start : nullptr, e1 = (timed & 2) ? g_time_stop : nullptr;
    if (timed & 2) g_time_start = g_time_stop = nullptr;
    if (g.n == 1) {
      OD_RETURN_IF(allow_lds(single, lds));
      const One<A> one = {{g.seg[0]}};
      const dim3 grid(g.grid[0].x, g.grid[0].y, g.grid[0].z);
      if (e0 != nullptr || e1 != nullptr) hipExtLaunchKernelGGL(single, grid, dim3(threads), (uint32_t)lds, st, e0, e1, 0u, one, extra...);
      else hipLaunchKernelGGL(single, grid, dim3(threads), lds, st, one, extra...);
    } else {
      OD_RETURN_IF(allow_lds(multi, lds));
      if (e0 != nullptr || e1 != nullptr) hipExtLaunchKernelGGL(multi, dim3(total), dim3(threads), (uint32_t)lds, st, e0, e1, 0u, g, extra...);
      else hipLaunchKernelGGL(multi, dim3(total), dim3(threads), lds, st, g, extra...);
    }
    g.n = 0;
    total = 0;
    OD_CHECK_LAUNCH();
    return hipSuccess;
  }
};

// One launch of the segments of `a` and, behind them, of `b`, with kernel(a, b, first workgroup of b).
template <class A, class B, class K>
static hipError_t launch_both(SegList<A>& a, SegList<B>& b, K kernel, int threads, int lds, hipStream_t st) {
  OD_RETURN_IF(allow_lds(kernel, lds));
  hipLaunchKernelGGL(kernel, dim3(a.total + b.total), dim3(threads), lds, st, a.g, b.g, a.total);
  OD_CHECK_LAUNCH();
  return hipSuccess;
}

// Calls one(variant, members, count, timed) for groups of at most kMaxSeg batches that take the same
// kernel; variant(batch) < 0 leaves a batch out.
template <class V, class F>
static hipError_t by_variant(BatchList b, int n, V variant, F one) {
  constexpr int kMany = 256;                  // batches looked at together
  for (int base = 0; base < n; base += kMany) {
    const int cnt = n - base < kMany ? n - base : kMany;
    int var[kMany], left = 0;
    for (int i = 0; i < cnt; ++i) {
      var[i] = variant(*b[base + i]);
      left += var[i] >= 0;
    }
    bool first = base == 0;
    for (int i = 0; i < cnt && left > 0; ++i) {
      if (var[i] < 0) continue;
      const int v = var[i];
      const BatchRef* group[kMaxSeg];
      int k = 0;
      for (int j = i; j < cnt && k < kMaxSeg; ++j)
        if (var[j] == v) { group[k++] = b[base + j]; var[j] = -1; }
      left -= k;
      const bool last = left == 0 && base + cnt == n;
      OD_RETURN_IF(one(v, group, k, (first ? 1 : 0) | (last ? 2 : 0)));
      first = false;
      if (left > 0) --i;                      // more of the same variant may remain behind this position
    }
  }
  return hipSuccess;
}

static int ceil_div(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }
static int copy_blocks(int64_t count4, int most) {
  const int64_t blocks = (count4 + 255) / 256;
  return blocks < 1 ? 1 : blocks > most ? most : (int)blocks;
}

hipError_t launch_begin(BatchList b, int n, Prec prec, hipStream_t st) {
  const bool fast = prec == PREC_F16;
  SegList<BeginArgs> segs;
  MatChunk chunk = {};
  int used = 0;
  auto flush = [&]() -> hipError_t {
    used = 0;
    if (!fast) return segs.launch(k_begin<SrcF32, false, One<BeginArgs>>, k_begin<SrcF32, false, Segs<BeginArgs>>, 256, 0, st, 0, chunk);
    return b[0]->d.g_bf16 ? segs.launch(k_begin<SrcBF16, true, One<BeginArgs>>, k_begin<SrcBF16, true, Segs<BeginArgs>>, 256, 0, st, 0, chunk) : segs.launch(k_begin<SrcF32, true, One<BeginArgs>>, k_begin<SrcF32, true, Segs<BeginArgs>>, 256, 0, st, 0, chunk);
  };
  for (int i = 0; i < n; ++i) {
    const BatchRef& r = *b[i];
    const int per_mat = fast ? kStatRows + ceil_div(r.d.n, 64) * ceil_div(r.d.r, 64) : 1;
    for (int z = 0; z < r.d.nb;) {
      if (used == kMatChunk || segs.full()) OD_RETURN_IF(flush());
      const int take = r.d.nb - z < kMatChunk - used ? r.d.nb - z : kMatChunk - used;
      for (int k = 0; k < take; ++k) chunk.e[used + k] = r.host_mats[z + k];
      BeginArgs a = {};
      a.d = r.d;
      a.table = const_cast<MatEntry*>(r.mats) + z;
      a.chunk0 = used;
      a.scal = r.scal + (int64_t)z * kScalPerMat;
      a.info = r.info + (int64_t)z * kInfoPerMat;
      a.qht = HalfArr{r.qht.base + (int64_t)z * r.qht.stride, r.qht.stride};
      segs.add(a, per_mat, 1, take);
      used += take;
      z += take;
    }
  }
  return flush();
}

// ---- projection and back-projection -------------------------------------------------
// What the direct-to-LDS contraction takes (fast precision only): bf16 gradients and at least one whole 32-deep
// step.  Ranks above 64: up to 128 columns per tile the register kernels are 1 to 7 % slower per step (4096 x 4096,
// r = 72 | 104 | 128: 239 | 253 | 246 us with them, 234 | 247 | 240; nine 1840 x 7384, r = 104: 1302 -> 1214;
// 8192 x 8192, r = 96: 481 -> 457 with rotated k order), with half-filled 256-column tiles 2 to 9 % (six ragged matrices of
// r = 136: 476 -> 437, 8192 x 8192, r = 160: 567 -> 520, 4096 x 4096, r = 184: 293 -> 286).  Below r = 192 only from
// 2^21 elements on, of all that step together, or 2^20 in matrices of 2^19 each: less is a few short k loops, where the
// pipeline costs what it hides (register | direct, r = 72 and 128: 384 x 384 137 | 142 and 150 | 154, eight of them 149 | 152
// and 164 | 165, 640 x 640 142 | 146 and 154 | 157, four of them 152 | 155 and 167 | 168, 1024 x 1024 153 | 152 and
// 167 | 165; ten 448 x 512 158 | 158 and 175 | 173, forty 221 | 209 and 260 | 237).  By the whole work and not the size of one
// matrix, so that one set does not take two kernels where it could share a launch (four of 256 x 384 to 512 x 640, ranks 72 to
// 128: 191 | 196, 216 with both).
static bool stream_kernel_eligible(const ClassDims& d, const Work& work) {
  if (!d.g_bf16 || d.r <= 64 || d.m < 32 || d.n < 32) return false;
  return d.r >= 192 || work.elements >= 1 << 21 || (work.elements >= 1 << 20 && work.elements >= work.matrices << 19);
}
static int stream_tile_cols(int r) { return r <= 128 ? 128 : r <= 256 ? 256 : 512; }
// Few wide tiles need many splits to fill the chip; 64-row tiles get there with half of them,
// i.e. half the partial sums to write and to add up.  With enough tiles the wide one wins.
// `peers`: matrices of this shape that would fill the launch the batch is part of.
static bool proj_uses_flat_tiles(int m, int r, int64_t peers) { return r > 128 && (int64_t)ceil_div(m, 128) * ceil_div(r, 256) * peers < 256; }

void proj_tiling(const ClassDims& d, Prec prec, int64_t peers, const Work& work, bool staged, int* rows, int* cols, int* slots) {
  *rows = 128;
  *cols = d.r <= 64 ? 64 : (d.r <= 128 ? 128 : 256);
  *slots = 512;                                // two workgroups per CU
  if (prec != PREC_F16) return;
  if (stream_kernel_eligible(d, work) && !(staged && d.r < 192)) {       // one 8-wave workgroup per CU
    *cols = stream_tile_cols(d.r);
    *slots = 256;
  } else if (proj_uses_flat_tiles(d.m, d.r, peers)) {
    *rows = 64;
  }
}
void back_tiling(const ClassDims& d, Prec prec, const Work& work, bool staged, int* rows, int* cols, int* slots) {
  *rows = 128;
  *cols = d.r <= 64 ? 64 : (d.r <= 128 ? 128 : 256);
  *slots = 512;
  if (prec == PREC_F16 && stream_kernel_eligible(d, work) && !(staged && d.r < 192)) {
    *cols = stream_tile_cols(d.r);
    *slots = 256;
  }
}

enum ProjVariant : int { PV_STREAM128, PV_STREAM256, PV_STREAM512, PV_NARROW, PV_SQUARE, PV_FLAT, PV_FLAT2, PV_WIDE, PV_HUGE, PV_EXACT_SMALL, PV_EXACT };

static StreamArgs stream_args(const BatchRef& r, bool back) {
  StreamArgs a = {};
  a.d = r.d;
  a.mats = r.mats;
  a.only = r.host_mats[0];
  a.scal = r.scal;
  a.info = r.info;
  a.factor = r.pa;
  a.fh = back ? r.pht : r.qht;
  a.splits = back ? r.splits_back : r.splits_proj;
  a.part = a.splits == 1 ? (back ? r.ra : r.pa) : r.part;
  return a;
}
// one matrix whose rows are a multiple of 32 KB apart (in M): measured 10-20 % faster with
// rotated k order at 8192 columns; with several matrices in flight the order does not matter
static bool rows_share_channels(const BatchRef& r) { return r.peers == 1 && (r.d.ldm * (int64_t)sizeof(float)) % 32768 == 0; }

template <class T, class Num, class GSrc, int PF = 1>
static hipError_t proj_t(BatchList b, int n, hipStream_t st, int timed) {
  SegList<StreamArgs> segs;
  for (int i = 0; i < n; ++i) {
    StreamArgs a = stream_args(*b[i], false);
    a.rotate = rows_share_channels(*b[i]) ? 1 : 0;
    segs.add(a, ceil_div(a.d.m, T::MT) * ceil_div(a.d.r, T::NT), a.splits, a.d.nb);
  }
  return segs.launch(k_proj<T, Num, GSrc, PF, One<StreamArgs>>, k_proj<T, Num, GSrc, PF, Segs<StreamArgs>>, T::THREADS, T::template lds_bytes<Num>(), st, timed);
}
template <bool TRANS, int NT>
static hipError_t stream_d_t(BatchList b, int n, hipStream_t st, int timed) {
  constexpr int SB = NT == 512 ? 2 : 3;
  constexpr int lds = SB * NT * 64 + 3 * (128 * 32 * 6) + 2 * (TRANS ? 32 * 320 : 128 * 64);
  SegList<StreamArgs> segs;
  for (int i = 0; i < n; ++i) {
    StreamArgs a = stream_args(*b[i], TRANS);
    if (TRANS && a.splits == 1) a.rh = b[i]->rh;
    // rotated k order for the projection of a single matrix at 8192 columns (see the kernel): 120 ->
    // 102 us at r = 256.  With several matrices in flight the order does not matter, and the
    // 512-column tiles of the larger ranks are not waiting for memory (no gain measured there).
    a.rotate = !TRANS && NT <= 256 && rows_share_channels(*b[i]) ? 1 : 0;
    segs.add(a, ceil_div(TRANS ? a.d.n : a.d.m, 128) * ceil_div(a.d.r, NT), a.splits, a.d.nb);
  }
  return segs.launch(k_stream_d<TRANS, NT, SB, One<StreamArgs>>, k_stream_d<TRANS, NT, SB, Segs<StreamArgs>>, 512, lds, st, timed);
}
template <class GSrc>
static hipError_t proj_v(int v, BatchList b, int n, hipStream_t st, int timed) {
  switch (v) {
    case PV_NARROW: return proj_t<TileNarrow, NumF16, GSrc>(b, n, st, timed);
    case PV_SQUARE: return proj_t<TileSquare, NumF16, GSrc>(b, n, st, timed);
    case PV_FLAT: return proj_t<TileFlat, NumF16, GSrc>(b, n, st, timed);
    case PV_FLAT2: return proj_t<TileFlat, NumF16, GSrc, 2>(b, n, st, timed);
    case PV_WIDE: return proj_t<TileWide, NumF16, GSrc>(b, n, st, timed);
    case PV_EXACT_SMALL: return proj_t<TileSmall, NumBF<3>, GSrc>(b, n, st, timed);
    default: return proj_t<TileSquare8, NumBF<3>, GSrc>(b, n, st, timed);
  }
}
hipError_t launch_proj(BatchList b, int n, Prec prec, hipStream_t st) {
  const auto variant = [&](const BatchRef& r) -> int {
    const ClassDims& d = r.d;
    if (prec == PREC_BF3)
      // small problems: 64-deep steps halve the number of round trips of a loop that is all latency
      return (int64_t)ceil_div(d.m, 128) * ceil_div(d.r, 128) * r.splits_proj * r.peers < 256 ? PV_EXACT_SMALL : PV_EXACT;
    if (stream_kernel_eligible(d, r.work)) return stream_tile_cols(d.r) == 128 ? PV_STREAM128 : stream_tile_cols(d.r) == 256 ? PV_STREAM256 : PV_STREAM512;
    if (d.r <= 64) return PV_NARROW;
    if (d.r <= 128) return PV_SQUARE;
    // long enough K loops per column tile pay for a second register stage
    if (proj_uses_flat_tiles(d.m, d.r, r.peers)) return d.r > 256 ? PV_FLAT2 : PV_FLAT;
    return PV_WIDE;
  };
  return by_variant(b, n, variant, [&](int v, BatchList g, int k, int timed) -> hipError_t {
    if (v == PV_STREAM128) return stream_d_t<false, 128>(g, k, st, timed);
    if (v == PV_STREAM256) return stream_d_t<false, 256>(g, k, st, timed);
    if (v == PV_STREAM512) return stream_d_t<false, 512>(g, k, st, timed);
    return g[0]->d.g_bf16 ? proj_v<SrcBF16>(v, g, k, st, timed) : proj_v<SrcF32>(v, g, k, st, timed);
  });
}

template <class T, class Num, class GSrc, int PF = 1>
static hipError_t back_t(BatchList b, int n, hipStream_t st, int timed) {
  SegList<StreamArgs> segs;
  for (int i = 0; i < n; ++i) {
    const StreamArgs a = stream_args(*b[i], true);
    segs.add(a, ceil_div(a.d.n, T::MT) * ceil_div(a.d.r, T::NT), a.splits, a.d.nb);
  }
  return segs.launch(k_back<T, Num, GSrc, PF, One<StreamArgs>>, k_back<T, Num, GSrc, PF, Segs<StreamArgs>>, T::THREADS, T::template lds_bytes<Num>(), st, timed);
}
template <class GSrc>
static hipError_t back_v(int v, BatchList b, int n, hipStream_t st, int timed) {
  switch (v) {
    case PV_NARROW: return back_t<TileNarrow, NumF16, GSrc>(b, n, st, timed);
    case PV_SQUARE: return back_t<TileSquare, NumF16, GSrc>(b, n, st, timed);
    case PV_HUGE: return back_t<TileHuge, NumF16, GSrc, 2>(b, n, st, timed);
    case PV_WIDE: return back_t<TileWide, NumF16, GSrc>(b, n, st, timed);
    case PV_EXACT_SMALL: return back_t<TileSmall, NumBF<3>, GSrc>(b, n, st, timed);
    default: return back_t<TileSquare8, NumBF<3>, GSrc>(b, n, st, timed);
  }
}
hipError_t launch_back(BatchList b, int n, Prec prec, hipStream_t st) {
  const auto variant = [&](const BatchRef& r) -> int {
    const ClassDims& d = r.d;
    if (prec == PREC_BF3)
      return (int64_t)ceil_div(d.n, 128) * ceil_div(d.r, 128) * r.splits_back * r.peers < 256 ? PV_EXACT_SMALL : PV_EXACT;
    if (stream_kernel_eligible(d, r.work)) return stream_tile_cols(d.r) == 128 ? PV_STREAM128 : stream_tile_cols(d.r) == 256 ? PV_STREAM256 : PV_STREAM512;
    if (d.r <= 64) return PV_NARROW;
    if (d.r <= 128) return PV_SQUARE;
    // several column tiles per row panel: 256 x 256 tiles halve the operand traffic per product
    // and run one workgroup per CU with two register stages of loads in flight
    return d.r > 256 ? PV_HUGE : PV_WIDE;
  };
  return by_variant(b, n, variant, [&](int v, BatchList g, int k, int timed) -> hipError_t {
    if (v == PV_STREAM128) return stream_d_t<true, 128>(g, k, st, timed);
    if (v == PV_STREAM256) return stream_d_t<true, 256>(g, k, st, timed);
    if (v == PV_STREAM512) return stream_d_t<true, 512>(g, k, st, timed);
    return g[0]->d.g_bf16 ? back_v<SrcBF16>(v, g, k, st, timed) : back_v<SrcF32>(v, g, k, st, timed);
  });
}

// ---- ordered sums of partials ----------------------------------------------------------
static void add_reduce(SegList<ReduceArgs>& segs, int nb, WsArr part, int splits, int64_t count, WsArr out, Pred pred) {
  ReduceArgs a = {};
  a.part = part;
  a.out = out;
  a.count = count;
  a.splits = splits;
  a.pred = pred;
  segs.add(a, copy_blocks(count / 4, 2048), 1, nb);
}
static const Pred kAlways = {nullptr, 0, 0.f, 0};

hipError_t launch_reduce(int nb, WsArr part, int splits, int64_t count, WsArr out, hipStream_t st, Pred pred) {
  SegList<ReduceArgs> segs;
  add_reduce(segs, nb, part, splits, count, out, pred);
  return segs.launch(k_reduce<One<ReduceArgs>>, k_reduce<Segs<ReduceArgs>>, 256, 0, st, 0);
}
hipError_t launch_proj_reduce(BatchList b, int n, hipStream_t st) {
  return by_variant(b, n, [](const BatchRef& r) { return r.splits_proj > 1 ? 0 : -1; }, [&](int, BatchList g, int k, int) {
    SegList<ReduceArgs> segs;
    for (int i = 0; i < k; ++i) add_reduce(segs, g[i]->d.nb, g[i]->part, g[i]->splits_proj, (int64_t)g[i]->d.m * g[i]->d.r, g[i]->pa, kAlways);
    return segs.launch(k_reduce<One<ReduceArgs>>, k_reduce<Segs<ReduceArgs>>, 256, 0, st, 0);
  });
}
hipError_t launch_back_reduce(BatchList b, int n, Prec prec, hipStream_t st) {
  const auto variant = [&](const BatchRef& r) -> int {
    if (prec != PREC_F16) return r.splits_back > 1 ? 0 : -1;
    return r.splits_back == 1 && stream_kernel_eligible(r.d, r.work) ? -1 : 1;      // that kernel has written the fp16 copy itself
  };
  return by_variant(b, n, variant, [&](int v, BatchList g, int k, int) -> hipError_t {
    if (v == 0) {
      SegList<ReduceArgs> segs;
      for (int i = 0; i < k; ++i) add_reduce(segs, g[i]->d.nb, g[i]->part, g[i]->splits_back, (int64_t)g[i]->d.n * g[i]->d.r, g[i]->ra, kAlways);
      return segs.launch(k_reduce<One<ReduceArgs>>, k_reduce<Segs<ReduceArgs>>, 256, 0, st, 0);
    }
    SegList<ReduceRArgs> segs;
    for (int i = 0; i < k; ++i) {
      const BatchRef& r = *g[i];
      ReduceRArgs a = {};
      a.d = r.d;
      a.part = r.splits_back == 1 ? r.ra : r.part;
      a.out = r.ra;
      a.splits = r.splits_back;
      a.rh = r.rh;
      a.scal = r.scal;
      a.info = r.info;
      segs.add(a, copy_blocks((int64_t)r.d.n * r.d.r / 4, 2048), 1, r.d.nb);
    }
    return segs.launch(k_reduce_r<One<ReduceRArgs>>, k_reduce_r<Segs<ReduceRArgs>>, 256, 0, st, 0);
  });
}

// ---- orthogonalisation ------------------------------------------------------------------
// Ranks of one 32 x 32 tile take the first CholeskyQR pass in a single launch, factorisation included.

// Gram partials of a0 (pass 0) and of a1 (pass 1) for small ranks.  The first pass reads the former while it
// writes the latter, so they lie in the array of the result's fp16 copy, which holds them from two row ranges
// (of 256 rows and more) on.
WsArr small_partials(const BatchRef& r, int side, int pass) {
  if (pass == 1) return r.part;
  if (r.splits_gram[side] == 1) return r.gram;
  const HalfArr& h = side == 0 ? r.ph : r.qh;
  return WsArr{reinterpret_cast<float*>(h.base), h.stride / 2};
}

// The small batches of a list that wait for a stage of theirs: with launches of larger ranks while there
// are some, then by themselves.
struct SmallQueue {
  BatchList b;
  int n, next, side;
  Prec prec;
  SmallQueue(BatchList b_, int n_, int side_, Prec prec_) : b(b_), n(n_), next(0), side(side_), prec(prec_) {}
  // fills `segs` with the next of them
  void take(SegList<SmallArgs>& segs, int stage) {
    for (; next < n && !segs.full(); ++next) {
      const BatchRef& r = *b[next];
      if (!r.small) continue;
      SmallArgs a = {};
      a.rows = r.rows(side);
      a.r = r.d.r;
      a.splits = r.splits_gram[side];
      a.side = side;
      a.a0 = r.a0(side);
      a.a1 = r.a1(side);
      a.gram = small_partials(r, side, 0);
      a.part = small_partials(r, side, 1);
      a.t1 = r.t1[side];
      a.t2 = r.t2[side];
      if (r.beside) a.w = r.w;
      a.scal = r.scal;
      a.info = r.info;
      if (side == 1) a.q_mats = r.mats;
      if (side == 1 && r.d.nb == 1) a.only_q = r.host_mats[0].Q;
      if (prec == PREC_F16) {
        a.hn = side == 0 ? r.ph : r.qh;
        if (side == 0) a.ht = r.pht;
      }
      segs.add(a, stage == SMALL_RESULT ? ceil_div(a.rows, kSmallRows) : a.splits, 1, r.d.nb);
    }
  }
  template <int STAGE>
  hipError_t rest(hipStream_t st) {
    while (next < n) {
      SegList<SmallArgs> segs;
      take(segs, STAGE);
      OD_RETURN_IF(segs.launch(k_small<STAGE, One<SmallArgs>>, k_small<STAGE, Segs<SmallArgs>>, kSmallRows, kSmallLds, st, 0));
    }
    return hipSuccess;
  }
};

// Gram partials of a0 (`first`, into gram_out or with several splits `part`) or a1 (into `part`); `queue`: small
// batches that may join, or null
template <class T, class Num>
static hipError_t gram_tt(BatchList b, int n, int side, bool first, SmallQueue* queue, hipStream_t st) {
  SegList<GramArgs> segs;
  for (int i = 0; i < n; ++i) {
    const BatchRef& r = *b[i];
    GramArgs a = {};
    a.d = r.d;
    a.scal = r.scal;
    a.rows = r.rows(side);
    a.r = r.d.r;
    a.splits = r.splits_gram[side];
    a.side = first ? side : 2;
    a.a = first ? r.a0(side) : r.a1(side);
    a.part = first && a.splits == 1 ? r.gram : r.part;       // a single split is the Gram matrix itself
    const int tiles = ceil_div(a.r, T::NT);
    segs.add(a, tiles * (tiles + 1) / 2, a.splits, r.d.nb);
  }
  constexpr int lds = T::template lds_bytes<Num>();
  if constexpr (std::is_same<T, TileSmall>::value) {
    SegList<SmallArgs> small;
    if (queue != nullptr) queue->take(small, SMALL_GRAM);
    if (small.g.n > 0) return launch_both(segs, small, k_gram_and_small<Num>, T::THREADS, lds > kSmallLds ? lds : kSmallLds, st);
  }
  return segs.launch(k_gram<T, Num, One<GramArgs>>, k_gram<T, Num, Segs<GramArgs>>, T::THREADS, lds, st, 0);
}
static hipError_t gram_pass(BatchList b, int n, int side, bool first, Prec prec, SmallQueue* queue, hipStream_t st) {
  const auto variant = [&](const BatchRef& r) -> int {
    if (r.small) return -1;
    // few large tiles leave most of the chip idle: use small ones until the grid fills it
    const int64_t t = ceil_div(r.d.r, 128);
    return t * t * r.splits_gram[side] * r.peers < kSmallGramTiles ? 0 : 1;
  };
  return by_variant(b, n, variant, [&](int v, BatchList g, int k, int) -> hipError_t {
    // fast precision has the sampled scale of B at hand: two-term fp16 operands (half the
    // matrix-core work of the three-way bf16 split at 22 instead of 24 bits)
    if (prec == PREC_F16) return v == 0 ? gram_tt<TileSmall, NumH2>(g, k, side, first, queue, st) : gram_tt<TileSquare8, NumH2>(g, k, side, first, queue, st);
    return v == 0 ? gram_tt<TileSmall, NumBF<3>>(g, k, side, first, queue, st) : gram_tt<TileSquare, NumBF<3>>(g, k, side, first, queue, st);
  });
}
hipError_t launch_gram_plain(int nb, int rows, int r, WsArr a, WsArr part, int splits, hipStream_t st) {
  GramArgs ga = {};
  ga.rows = rows;
  ga.r = r;
  ga.splits = splits;
  ga.side = -1;
  ga.a = a;
  ga.part = part;
  SegList<GramArgs> segs;
  // (a launch of its own, so that the matrices of the batch are all there are)
  const int t = ceil_div(r, 128);
  const int tiles = (int64_t)t * t * splits * nb < kSmallGramTiles ? ceil_div(r, 64) : t;
  segs.add(ga, tiles * (tiles + 1) / 2, splits, nb);
  return tiles == t && r > 64 ? segs.launch(k_gram<TileSquare, NumBF<3>, One<GramArgs>>, k_gram<TileSquare, NumBF<3>, Segs<GramArgs>>, TileSquare::THREADS, TileSquare::lds_bytes<NumBF<3>>(), st, 0)
                              : segs.launch(k_gram<TileSmall, NumBF<3>, One<GramArgs>>, k_gram<TileSmall, NumBF<3>, Segs<GramArgs>>, TileSmall::THREADS, TileSmall::lds_bytes<NumBF<3>>(), st, 0);
}

hipError_t launch_orth_gram(BatchList b, int n, int side, Prec prec, hipStream_t st) {
  SmallQueue queue(b, n, side, prec);
  OD_RETURN_IF(gram_pass(b, n, side, true, prec, &queue, st));
  OD_RETURN_IF(queue.rest<SMALL_GRAM>(st));
  // ordered reduction of the split partial sums on many workgroups: the factorisation runs on
  // one workgroup per matrix and should not spend its time summing
  return by_variant(b, n, [&](const BatchRef& r) { return !r.small && r.splits_gram[side] > 1 ? 0 : -1; }, [&](int, BatchList g, int k, int) {
    SegList<ReduceArgs> segs;
    for (int i = 0; i < k; ++i) add_reduce(segs, g[i]->d.nb, g[i]->part, g[i]->splits_gram[side], (int64_t)g[i]->d.r * g[i]->d.r, g[i]->gram, kAlways);
    return segs.launch(k_reduce<One<ReduceArgs>>, k_reduce<Segs<ReduceArgs>>, 256, 0, st, 0);
  });
}

// ---- triangular products
enum ApplyKind : int { APPLY_W, APPLY_FULL, APPLY_CORRECTION };     // a0 W1 -> a1; a1 W2 -> result; a1 - a1 Phi -> result
static Pred deviation(const BatchRef& r, int side, int want) { return Pred{r.scal, 2 + side, kFirstOrderDeviation, want}; }

template <class T, class Num, bool DEEP, bool CORR, bool EITHER = false>
static hipError_t apply_tt(BatchList b, int n, int side, ApplyKind kind, Prec prec, SmallQueue* queue, hipStream_t st) {
  SegList<ApplyArgs> segs;
  for (int i = 0; i < n; ++i) {
    const BatchRef& r = *b[i];
    ApplyArgs a = {};
    a.rows = r.rows(side);
    a.r = r.d.r;
    a.w = r.w;
    a.pred = kAlways;
    if (kind == APPLY_W) {
      a.a = r.a0(side);
      a.out = r.a1(side);
    } else {
      a.a = r.a1(side);
      a.out = r.a0(side);
      a.q_mats = side == 1 ? r.mats : nullptr;
      if (side == 1 && r.d.nb == 1) a.only_q = r.host_mats[0].Q;
      if (prec == PREC_F16) {
        a.wh = HalfArr{reinterpret_cast<uint16_t*>(r.tmp.base), 2 * r.tmp.stride};      // Phi^T (see k_corr)
        a.pred = deviation(r, side, kind == APPLY_FULL ? 1 : 0);
        a.hn = side == 0 ? r.ph : r.qh;
        if (side == 0) a.ht = r.pht;
      }
    }
    segs.add(a, ceil_div(a.rows, T::MT) * ceil_div(a.r, T::NT), 1, r.d.nb);
  }
  SegList<SmallArgs> small;
  if constexpr (EITHER) {
    constexpr int corr = TileSmall::template lds_bytes<NumF16>(), full = TileSmallFlat::template lds_bytes<NumBF<2>>(), lds = corr > full ? corr : full;
    if (queue != nullptr) queue->take(small, SMALL_RESULT);
    if (small.g.n > 0) return launch_both(segs, small, k_apply_result_and_small, TileSmall::THREADS, lds > kSmallLds ? lds : kSmallLds, st);
    return segs.launch(k_apply_result<One<ApplyArgs>>, k_apply_result<Segs<ApplyArgs>>, TileSmall::THREADS, lds, st, 0);
  }
  constexpr int lds = T::template lds_bytes<Num>();
  if constexpr (std::is_same<T, TileSmall>::value && !CORR) {
    constexpr int both = lds > kSmallLds ? lds : kSmallLds;
    if (queue != nullptr) queue->take(small, kind == APPLY_W ? SMALL_FIRST : SMALL_RESULT);
    if (small.g.n > 0 && kind == APPLY_W) return launch_both(segs, small, k_apply_and_small<Num, SMALL_FIRST>, T::THREADS, both, st);
    if (small.g.n > 0) return launch_both(segs, small, k_apply_and_small<Num, SMALL_RESULT>, T::THREADS, both, st);
  }
  return segs.launch(k_apply<T, Num, DEEP, CORR, One<ApplyArgs>>, k_apply<T, Num, DEEP, CORR, Segs<ApplyArgs>>, T::THREADS, lds, st, 0);
}
// `merged`: small grids take the correction and the full product of a result in one launch, that of the former;
// `queue`: small batches whose stage may join the launches of 64 x 64 tiles, or null
template <class Num, bool CORR>
static hipError_t apply_t(BatchList b, int n, int side, ApplyKind kind, Prec prec, bool merged, SmallQueue* queue, hipStream_t st) {
  const auto variant = [&](const BatchRef& r) -> int {
    if (r.small) return -1;
    if ((int64_t)ceil_div(r.rows(side), 128) * ceil_div(r.d.r, 128) * r.peers >= 512) return 1;
    return merged && kind == APPLY_FULL ? -1 : 0;
  };
  return by_variant(b, n, variant, [&](int v, BatchList g, int k, int) -> hipError_t {
    if constexpr (CORR)
      if (v == 0 && merged) return apply_tt<TileSmall, Num, true, CORR, true>(g, k, side, kind, prec, queue, st);
    if (v == 0) return apply_tt<TileSmall, Num, true, CORR>(g, k, side, kind, prec, queue, st);
    // 128 columns per tile: the loop of a column tile ends at its last row of W (upper triangular),
    // so narrower tiles skip more of the zero half than 256-column ones would (measured -10 %)
    // one operand part leaves LDS room for 64-deep steps at two workgroups per CU (measured -13 to
    // -23 %); with two parts the deeper tile halves the occupancy and loses
    if constexpr (Num::PARTS == 1) return apply_tt<TileSquareDeepK, Num, false, CORR>(g, k, side, kind, prec, queue, st);
    else return apply_tt<TileSquare8, Num, false, CORR>(g, k, side, kind, prec, queue, st);
  });
}
static hipError_t apply_product(BatchList b, int n, int side, ApplyKind kind, Prec prec, bool merged, SmallQueue* queue, hipStream_t st) {
  return prec == PREC_BF3 ? apply_t<NumBF<3>, false>(b, n, side, kind, prec, merged, queue, st) : apply_t<NumBF<2>, false>(b, n, side, kind, prec, merged, queue, st);
}

hipError_t launch_orth_second(BatchList b, int n, int side, Prec prec, hipStream_t st) {
  SmallQueue queue(b, n, side, prec);
  OD_RETURN_IF(apply_product(b, n, side, APPLY_W, prec, false, &queue, st));
  OD_RETURN_IF(queue.rest<SMALL_FIRST>(st));
  OD_RETURN_IF(gram_pass(b, n, side, false, prec, nullptr, st));
  OD_RETURN_IF(by_variant(b, n, [](const BatchRef& r) { return r.small ? -1 : 0; }, [&](int, BatchList g, int k, int) {
    SegList<CorrArgs> segs;
    for (int i = 0; i < k; ++i) {
      const BatchRef& r = *g[i];
      CorrArgs a = {};
      a.r = r.d.r;
      a.splits = r.splits_gram[side];
      a.part = r.part;
      a.t1 = r.t1[side];
      a.t2 = r.t2[side];
      a.w2 = r.w;
      // fast precision: Phi^T as fp16 operand words lives in the r x r scratch the factorisation no
      // longer needs; exact precision: W2 = I - Phi(E)
      if (prec == PREC_F16) a.phit = HalfArr{reinterpret_cast<uint16_t*>(r.tmp.base), 2 * r.tmp.stride};
      a.scal = r.scal;
      a.scal_slot = 2 + side;
      a.info = r.info;
      a.info_slot = side;
      segs.add(a, copy_blocks((int64_t)a.r * a.r / 4, 1024), 1, r.d.nb);
    }
    return segs.launch(k_corr<One<CorrArgs>>, k_corr<Segs<CorrArgs>>, 256, 0, st, 0);
  }));
  // ranks above 256: the summed Gram matrix of a flagged matrix goes to the class array for the
  // class-wide guard
  return by_variant(b, n, [](const BatchRef& r) { return r.d.r > kCholMax ? 0 : -1; }, [&](int, BatchList g, int k, int) {
    SegList<ReduceArgs> segs;
    for (int i = 0; i < k; ++i)
      add_reduce(segs, g[i]->d.nb, g[i]->part, g[i]->splits_gram[side], (int64_t)g[i]->d.r * g[i]->d.r, g[i]->gram, deviation(*g[i], side, 1));
    return segs.launch(k_reduce<One<ReduceArgs>>, k_reduce<Segs<ReduceArgs>>, 256, 0, st, 0);
  });
}

static hipError_t launch_leaf(const CholArgs* args, const int* counts, int n, hipStream_t st) {
  SegList<CholArgs> segs;
  for (int i = 0; i < n; ++i) {
    segs.add(args[i], counts[i], 1, 1);
    if (segs.full() || i + 1 == n) OD_RETURN_IF(segs.launch(k_chol256<One<CholArgs>>, k_chol256<Segs<CholArgs>>, kCholThreads, kCholLds, st, 0));
  }
  return hipSuccess;
}

hipError_t launch_orth_guard(BatchList b, int n, int side, hipStream_t st) {
  return by_variant(b, n, [](const BatchRef& r) { return r.d.r <= kCholMax && !r.small ? 0 : -1; }, [&](int, BatchList g, int k, int) {
    CholArgs args[kMaxSeg];
    int counts[kMaxSeg];
    for (int i = 0; i < k; ++i) {
      const BatchRef& r = *g[i];
      CholArgs ca = {};
      ca.t = r.t2[side];
      ca.w = r.w;
      ca.r = r.d.r;
      ca.info = r.info;
      ca.info_slot = side;
      ca.src = r.part;
      ca.splits = r.splits_gram[side];
      ca.split_stride = (int64_t)r.d.r * r.d.r;
      ca.pred = deviation(r, side, 1);
      args[i] = ca;
      counts[i] = r.d.nb;
    }
    return launch_leaf(args, counts, k, st);
  });
}

hipError_t launch_orth_result(BatchList b, int n, int side, Prec prec, int which, hipStream_t st) {
  SmallQueue queue(b, n, side, prec);
  if (prec == PREC_BF3) OD_RETURN_IF(apply_product(b, n, side, APPLY_FULL, prec, false, &queue, st));
  else if (which != 2) OD_RETURN_IF((apply_t<NumF16, true>(b, n, side, APPLY_CORRECTION, prec, which == 0, &queue, st)));
  if (which != 2) OD_RETURN_IF(queue.rest<SMALL_RESULT>(st));
  if (prec != PREC_BF3 && which != 1) OD_RETURN_IF(apply_product(b, n, side, APPLY_FULL, prec, which == 0, nullptr, st));
  return hipSuccess;
}

// ---- Cholesky --------------------------------------------------------------------------
template <class T, class Num, class DirA>
static hipError_t sgemm_tt(int nb, const SgemmArgs& g, hipStream_t st) {
  constexpr int lds = T::template lds_bytes<Num>();
  hipError_t e = allow_lds(k_sgemm<T, Num, DirA>, lds);
  if (e != hipSuccess) return e;
  dim3 grid(((g.Mc + T::MT - 1) / T::MT) * ((g.Nc + T::NT - 1) / T::NT), 1, nb * g.nq);
  hipLaunchKernelGGL((k_sgemm<T, Num, DirA>), grid, dim3(T::THREADS), lds, st, g);
  OD_CHECK_LAUNCH();
  return hipSuccess;
}
template <class DirA>
static hipError_t sgemm_t(int nb, const SgemmArgs& g, hipStream_t st) {
  const int big = ((g.Mc + 127) / 128) * ((g.Nc + 127) / 128) * nb * g.nq;
  if (big < 256) return sgemm_tt<TileSmall, NumBF<3>, DirA>(nb, g, st);      // one 128 x 128 tile per CU fills the chip
  return sgemm_tt<TileSquare, NumBF<3>, DirA>(nb, g, st);
}
// six-product operands
static hipError_t sgemm(int nb, const SgemmArgs& g, bool a_kc, hipStream_t st) {
  if (g.Mc <= 0 || g.Nc <= 0 || g.Kc <= 0 || g.nq <= 0) return hipSuccess;
  return a_kc ? sgemm_t<KC>(nb, g, st) : sgemm_t<KSF>(nb, g, st);
}

// g1 with A read as [k][row] (KSF) and g2 with A read as [row][k] (KC), six-product operands,
// in one launch; either may be empty.  Both have nq = 1.
template <class T>
static hipError_t sgemm_pair_tt(int nb, const SgemmArgs& g1, const SgemmArgs& g2, hipStream_t st) {
  typedef NumBF<3> Num;
  constexpr int lds = T::template lds_bytes<Num>();
  hipError_t e = allow_lds(k_sgemm_pair<T, Num, KSF, KC>, lds);
  if (e != hipSuccess) return e;
  const int tiles1 = ((g1.Mc + T::MT - 1) / T::MT) * ((g1.Nc + T::NT - 1) / T::NT);
  const int tiles2 = ((g2.Mc + T::MT - 1) / T::MT) * ((g2.Nc + T::NT - 1) / T::NT);
  hipLaunchKernelGGL((k_sgemm_pair<T, Num, KSF, KC>), dim3(tiles1 + tiles2, 1, nb), dim3(T::THREADS), lds, st, g1, g2, tiles1);
  OD_CHECK_LAUNCH();
  return hipSuccess;
}
static hipError_t sgemm_pair(int nb, const SgemmArgs& g1, const SgemmArgs& g2, hipStream_t st) {
  const bool has1 = g1.Mc > 0 && g1.Nc > 0 && g1.Kc > 0, has2 = g2.Mc > 0 && g2.Nc > 0 && g2.Kc > 0;
  if (!has1 && !has2) return hipSuccess;
  if (!has2) return sgemm(nb, g1, false, st);
  if (!has1) return sgemm(nb, g2, true, st);
  const int big = (((g1.Mc + 127) / 128) * ((g1.Nc + 127) / 128) + ((g2.Mc + 127) / 128) * ((g2.Nc + 127) / 128)) * nb;
  if (big < 256) return sgemm_pair_tt<TileSmall>(nb, g1, g2, st);
  return sgemm_pair_tt<TileSquare>(nb, g1, g2, st);
}

// ranks above 256: blocked factorisation of one class
static hipError_t blocked_cholinv(const CholJob& job, hipStream_t st) {
  const int nb = job.nb, r = job.r;
  const WsArr gram = job.gram, t = job.t, w = job.w, tmp = job.tmp;
  const Pred pred = job.pred;
  hipError_t e;
  const int nblk = (r + kLeaf - 1) / kLeaf;
  CholArgs ca = {};
  ca.t = t; ca.w = w; ca.r = r; ca.info = job.info; ca.info_slot = job.info_slot;
  ca.src = gram; ca.splits = 1; ca.split_stride = 0;
  ca.pred = pred;
  // lower block triangles of T and W are never written below; clear them once
  {
    const int64_t count = (int64_t)r * r;          // a multiple of 64
    int blocks = (int)((count / 4 + 255) / 256);
    if (blocks > 256) blocks = 256;
    hipLaunchKernelGGL(k_zero_pair, dim3(blocks, nb), dim3(256), 0, st, t, w, count, pred);
    OD_CHECK_LAUNCH();
  }
  // Step p: the diagonal block (T_pp, W_pp) is factored; then
  //   (1) the panel of the factor      T(p, rest) = W_pp^T G(p, rest)
  //       and, for the inverse,        tmp(0:p, p) = T(0:p, p) W_pp              (one launch)
  //   (2) the update of the next diagonal block alone
  //                                    G(p+1, p+1) -= T(p, p+1)^T T(p, p+1)      (one short launch)
  //   (3) one launch: the factorisation of block p + 1, beside the rest of the trailing update
  //       G(rest, rest) -= T(p, rest)^T T(p, rest) and block column p of the inverse,
  //       W(0:p, p) = -W(0:p, 0:p) tmp(0:p, p)
  // (the inverse of [[A, b], [0, c]] is [[A^-1, -A^-1 b c^-1], [0, c^-1]]).  The serial chain is
  // the factorisations and launches (1), (2); the bulk of the update hides behind a factorisation.
  auto tiles_of = [](const SgemmArgs& g, int mt) { return g.Mc > 0 && g.Nc > 0 && g.Kc > 0 ? ((g.Mc + mt - 1) / mt) * ((g.Nc + mt - 1) / mt) : 0; };
  for (int p = 0; p < nblk; ++p) {
    if (p == 0) {
      ca.blk = 0;
      OD_RETURN_IF(launch_leaf(&ca, &nb, 1, st));
    }
    const int o = p * kLeaf, o1 = (p + 1) * kLeaf, rest = r > o1 ? r - o1 : 0;
    const int bw = r - o < kLeaf ? r - o : kLeaf;       // width of block column p
    SgemmArgs panel = {}, prod = {}, trail = {}, wcol = {};
    panel.pred = prod.pred = trail.pred = wcol.pred = pred;
    panel.r = prod.r = trail.r = wcol.r = r;
    panel.nq = prod.nq = trail.nq = wcol.nq = 1;
    if (rest > 0) {
      panel.a = w; panel.b = gram; panel.c = t;
      panel.a_r0 = o; panel.a_k0 = o; panel.b_k0 = o; panel.b_c0 = o1; panel.c_r0 = o; panel.c_c0 = o1;
      panel.Mc = kLeaf; panel.Nc = rest; panel.Kc = kLeaf; panel.alpha = 1.f; panel.beta = 0.f;
      trail.a = t; trail.b = t; trail.c = gram;
      trail.a_r0 = o1; trail.a_k0 = o; trail.b_k0 = o; trail.b_c0 = o1; trail.c_r0 = o1; trail.c_c0 = o1;
      trail.Mc = rest; trail.Nc = rest; trail.Kc = kLeaf; trail.alpha = -1.f; trail.beta = 1.f;
    }
    if (p > 0) {
      prod.a = t; prod.b = w; prod.c = tmp;
      prod.a_r0 = 0; prod.a_k0 = o; prod.b_k0 = o; prod.b_c0 = o; prod.c_r0 = 0; prod.c_c0 = o;
      prod.Mc = o; prod.Nc = bw; prod.Kc = bw; prod.alpha = 1.f; prod.beta = 0.f;
      wcol.a = w; wcol.b = tmp; wcol.c = w;
      wcol.a_r0 = 0; wcol.a_k0 = 0; wcol.b_k0 = 0; wcol.b_c0 = o; wcol.c_r0 = 0; wcol.c_c0 = o;
      wcol.Mc = o; wcol.Nc = bw; wcol.Kc = o; wcol.alpha = -1.f; wcol.beta = 0.f;
    }
    if ((e = sgemm_pair(nb, panel, prod, st)) != hipSuccess) return e;
    if (rest == 0) {
      if ((e = sgemm_pair(nb, trail, wcol, st)) != hipSuccess) return e;
      continue;
    }
    // the trailing update in three pieces: the next diagonal block, the columns right of it
    // (all rows), and the rows below it (its own columns)
    const int nb1 = rest < kLeaf ? rest : kLeaf, o2 = o1 + nb1;
    SgemmArgs diag = trail, right = trail, below = trail;
    diag.Mc = nb1; diag.Nc = nb1;
    right.b_c0 = o2; right.c_c0 = o2; right.Nc = rest - nb1;
    below.a_r0 = o2; below.c_r0 = o2; below.Mc = rest - nb1; below.Nc = nb1;
    if ((e = sgemm(nb, diag, false, st)) != hipSuccess) return e;
    ca.blk = p + 1;
    const int big = (tiles_of(right, 128) + tiles_of(below, 128) + tiles_of(wcol, 128)) * nb;
    if (big < 256) {
      typedef TileSmall T;
      constexpr int lds = T::lds_bytes<NumBF<3>>() > kCholLds ? T::lds_bytes<NumBF<3>>() : kCholLds;
      if ((e = allow_lds(k_chol_ahead<T>, lds)) != hipSuccess) return e;
      const int t1 = tiles_of(right, T::MT), t2 = tiles_of(below, T::MT), t3 = tiles_of(wcol, T::MT);
      hipLaunchKernelGGL(k_chol_ahead<T>, dim3(1 + t1 + t2 + t3, 1, nb), dim3(kCholThreads), lds, st, ca, right, below, wcol, t1, t2);
    } else {
      typedef TileSquare8 T;
      constexpr int lds = T::lds_bytes<NumBF<3>>() > kCholLds ? T::lds_bytes<NumBF<3>>() : kCholLds;
      if ((e = allow_lds(k_chol_ahead<T>, lds)) != hipSuccess) return e;
      const int t1 = tiles_of(right, T::MT), t2 = tiles_of(below, T::MT), t3 = tiles_of(wcol, T::MT);
      hipLaunchKernelGGL(k_chol_ahead<T>, dim3(1 + t1 + t2 + t3, 1, nb), dim3(kCholThreads), lds, st, ca, right, below, wcol, t1, t2);
    }
    OD_CHECK_LAUNCH();
  }
  return hipSuccess;
}

hipError_t launch_cholinv(const CholJob* jobs, int njobs, hipStream_t st) {
  CholArgs args[kMaxSeg];
  int counts[kMaxSeg], k = 0;
  for (int i = 0; i < njobs; ++i) {
    const CholJob& j = jobs[i];
    if (j.r > kLeaf) {
      OD_RETURN_IF(blocked_cholinv(j, st));
      continue;
    }
    CholArgs ca = {};
    ca.t = j.t; ca.w = j.w; ca.r = j.r; ca.info = j.info; ca.info_slot = j.info_slot;
    ca.src = j.gram; ca.splits = j.splits; ca.split_stride = j.split_stride;
    ca.pred = j.pred;
    args[k] = ca;
    counts[k++] = j.nb;
    if (k == kMaxSeg) {
      OD_RETURN_IF(launch_leaf(args, counts, k, st));
      k = 0;
    }
  }
  return k > 0 ? launch_leaf(args, counts, k, st) : hipSuccess;
}

hipError_t launch_colnorm(BatchList b, int n, Prec prec, hipStream_t st) {
  const auto all = [](const BatchRef&) { return 0; };
  return by_variant(b, n, all, [&](int, BatchList g, int k, int) -> hipError_t {
    SegList<ColnormArgs> sum, fin, app;
    for (int i = 0; i < k; ++i) {
      const BatchRef& r = *g[i];
      ColnormArgs a = {};
      a.n = r.d.n;
      a.r = r.d.r;
      a.slabs = r.slabs;
      a.rr = r.ra;
      a.part = r.part;
      a.colsq = r.colsq;
      a.info = r.info;
      a.mats = r.mats;
      if (prec == PREC_F16) a.qh = r.qh;
      sum.add(a, ceil_div(a.r, 256), a.slabs, r.d.nb);
      fin.add(a, ceil_div(a.r, 64), 1, r.d.nb);
      app.add(a, copy_blocks((int64_t)a.n * a.r / 4, 2048), 1, r.d.nb);
    }
    OD_RETURN_IF(sum.launch(k_colsq_partial<One<ColnormArgs>>, k_colsq_partial<Segs<ColnormArgs>>, 256, 0, st, 0));
    OD_RETURN_IF(fin.launch(k_colsq_final<One<ColnormArgs>>, k_colsq_final<Segs<ColnormArgs>>, 1024, 0, st, 0));
    return app.launch(k_colnorm_apply<One<ColnormArgs>>, k_colnorm_apply<Segs<ColnormArgs>>, 256, 0, st, 0);
  });
}

// ---- error feedback and update -----------------------------------------------------------
static EfxArgs efx_args(const BatchRef& r) {
  EfxArgs a = {};
  a.d = r.d;
  a.mats = r.mats;
  a.only = r.host_mats[0];
  a.scal = r.scal;
  a.info = r.info;
  a.p = r.pa;
  a.rr = r.ra;
  a.ph = r.ph;
  a.rh = r.rh;
  a.qh = r.qh;
  // up to r = 256 (above, the XCD-aware band order takes over) consecutive workgroups walk along a
  // row of tiles, i.e. through consecutive addresses of M, G, X, instead of down a column of tiles
  // whose rows lie a whole leading dimension apart: 8192 x 8192: 172 -> 156 us at r = 16, 233 ->
  // 224 us at r = 256; no difference at 4096 x 4096
  a.d.col_fast = r.d.r <= 256 ? 1 : 0;
  return a;
}
enum EfxVariant : int { EV_EXACT_SMALL, EV_EXACT, EV_H, EV_D, EV_D_STREAM, EV_TALL, EV_TALL_STREAM };

template <class K1, class K2>
static hipError_t efx_launch(K1 single, K2 multi, BatchList b, int n, int tile_i, int tile_j, int threads, int lds, EfxCoef coef, hipStream_t st, int timed) {
  SegList<EfxArgs> segs;
  for (int i = 0; i < n; ++i) segs.add(efx_args(*b[i]), ceil_div(b[i]->d.m, tile_i) * ceil_div(b[i]->d.n, tile_j), 1, b[i]->d.nb);
  return segs.launch(single, multi, threads, lds, st, timed, coef);
}
template <bool XBF, bool GBF>
static hipError_t efx_v(int v, BatchList b, int n, EfxCoef c, hipStream_t st, int timed) {
  typedef NumBF<3> Num;
  constexpr int lds_h = 2 * 3 * 128 * 80, lds_d = 3 * 3 * 128 * 64, lds_tall = efx_stages(4) * (2 * 128 + 256) * 64;
  switch (v) {
    case EV_EXACT_SMALL: return efx_launch(k_efx<TileSmall, Num, XBF, GBF, One<EfxArgs>>, k_efx<TileSmall, Num, XBF, GBF, Segs<EfxArgs>>, b, n, 64, 64, TileSmall::THREADS, TileSmall::lds_bytes<Num>(), c, st, timed);
    case EV_EXACT: return efx_launch(k_efx<TileSquare8, Num, XBF, GBF, One<EfxArgs>>, k_efx<TileSquare8, Num, XBF, GBF, Segs<EfxArgs>>, b, n, 128, 128, TileSquare8::THREADS, TileSquare8::lds_bytes<Num>(), c, st, timed);
    case EV_H: return efx_launch(k_efx_h<XBF, GBF, One<EfxArgs>>, k_efx_h<XBF, GBF, Segs<EfxArgs>>, b, n, 128, 128, 512, lds_h, c, st, timed);
    case EV_D: return efx_launch(k_efx_d<XBF, GBF, false, 2, One<EfxArgs>>, k_efx_d<XBF, GBF, false, 2, Segs<EfxArgs>>, b, n, 128, 128, 256, lds_d, c, st, timed);
    case EV_D_STREAM: return efx_launch(k_efx_d<XBF, GBF, true, 2, One<EfxArgs>>, k_efx_d<XBF, GBF, true, 2, Segs<EfxArgs>>, b, n, 128, 128, 256, lds_d, c, st, timed);
    case EV_TALL: return efx_launch(k_efx_d<XBF, GBF, false, 4, One<EfxArgs>>, k_efx_d<XBF, GBF, false, 4, Segs<EfxArgs>>, b, n, 256, 128, 512, lds_tall, c, st, timed);
    default: return efx_launch(k_efx_d<XBF, GBF, true, 4, One<EfxArgs>>, k_efx_d<XBF, GBF, true, 4, Segs<EfxArgs>>, b, n, 256, 128, 512, lds_tall, c, st, timed);
  }
}
hipError_t launch_efx(BatchList b, int n, Prec prec, float a_coef, float b_coef, float lr, hipStream_t st) {
  const EfxCoef coef = {a_coef, b_coef, lr};
  const auto variant = [&](const BatchRef& r) -> int {
    const ClassDims& d = r.d;
    // small problems: more, smaller tiles (the kernel is a few microseconds of latency per tile)
    if (prec == PREC_BF3) return (int64_t)ceil_div(d.m, 128) * ceil_div(d.n, 128) * r.peers < 256 ? EV_EXACT_SMALL : EV_EXACT;
    // nontemporal stores also for sets far beyond the Infinity Cache at any rank: they leave no dirty
    // lines behind for the next kernel to wait on (measured on 8192 x 8192: the step is 2-7 % faster)
    const int stream = d.r > 256 || r.work.elements >= ((int64_t)48 << 20) ? 1 : 0;
    // Small sets: the kernel with eight waves per tile, which has the shorter start, unless the rank is whole 32-deep
    // steps from 64 on (392 x 264, r = 40: 136 against 139 us a step, four 512 x 512 of r = 56 135 | 136; five matrices of
    // ranks 24 to 72 211 in one launch, 220 with r = 72 in one of its own); above, the direct-to-LDS kernel (twenty
    // 1024 x 1024 of r = 40 233 | 230, 4096 x 4096, r = 40 213 | 206, r = 104 246 | 238, 8192 x 8192, r = 16 349 | 343,
    // r = 1000 2089 | 2047).  The elements of all that step together, which are the same for every batch: by m n peers, rounded
    // down, the shapes of one set fell on both sides and took two launches (three 2768 x 496 of r = 16 beside three 232 x 192 of
    // r = 8: 134 us, 125 in one)
    if ((d.r < 64 || d.r % 32 != 0) && r.work.elements < (int64_t)4 << 20) return EV_H;
    // r > 256: 256-row tiles (one 8-wave workgroup per CU) while they still fill the chip twice:
    // a third less operand traffic into LDS per product than 128-row tiles
    const int64_t tall = (int64_t)ceil_div(d.m, 256) * ceil_div(d.n, 128) * r.peers;
    return (d.r > 256 && tall >= 512 ? EV_TALL : EV_D) + stream;
  };
  return by_variant(b, n, variant, [&](int v, BatchList g, int k, int timed) -> hipError_t {
    if (g[0]->d.x_bf16) return g[0]->d.g_bf16 ? efx_v<true, true>(v, g, k, coef, st, timed) : efx_v<true, false>(v, g, k, coef, st, timed);
    return g[0]->d.g_bf16 ? efx_v<false, true>(v, g, k, coef, st, timed) : efx_v<false, false>(v, g, k, coef, st, timed);
  });
}

}  // namespace od

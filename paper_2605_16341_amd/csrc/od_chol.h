// Cholesky factorisation and triangular inverse of one SPD block of up to 256 x 256 in a
// single workgroup (12 waves):  G = T^T T with T upper triangular, W = T^-1.
//
// Used by the CholeskyQR orthogonalisation (orth() of Alg. 1 lines 2 and 4): T is the
// triangular factor of the thin QR, W turns the triangular solve into a product.
//
// Layout of the computation.  The block is cut into 32 x 32 tiles, nt per side.
//   * Two chain waves (1 and 5) run the serial chain of diagonal tiles.  One of them factors tile (J, J)
//     four pivots at a time (chain_group) and leaves every group of four rows in LDS the moment it is done.  The
//     other one takes tile (J, J+1) through the same elimination in fp32 (follow_group), subtracts
//     T(J, J+1)^T T(J, J+1) from the next diagonal tile, which it holds in registers, and factors that one next.
//   * The inverse wave (9) takes an identity tile through the elimination, one group behind the chain: V(J, J),
//     V = W^T.  It leaves it in LDS as product operand, split into three bf16 terms.
//   * The output wave (11) writes T(J, J) and the zero triangles.
//   * The other eight waves are workers (the first three roles have a SIMD to themselves).  They keep the tiles (I, K),
//     I < K, as matrix-core accumulators (16 registers per lane: register v of lane l is row
//     8 (v / 4) + 4 (l / 32) + v % 4, column l % 32), three or four each and never two that share a row or column of
//     tiles.  In step J a worker forms T(J, K) = V(J, J) S(J, K) or V(J, I) = -V(J, J) S'(J, I) (the accumulator
//     serves directly as the k-side operand) and publishes it to LDS already split; then every remaining tile
//     gets its update of the step from those operands, the one that the chain waits for first.
//   * The inverse is built alongside, right-looking: once T(I, K) has left its accumulator the same registers
//     collect S'(K, I) = sum_{I <= L < K} T(L, K)^T V(L, I).
//   * Signs: the accumulators hold -S and -S', and the panel -T, so that no operand is ever negated.
//   * Waves hand tiles over through counters in LDS (bounded waits); there is no barrier in the loop.
//     Products of the workers use three-way split bf16 operands (six products, 24 significant bits).
//
// What bounds it: per step, in turn, the chain (3900 cycles), the inverse wave's lag and its hand-over (3000), a panel
// tile and its publication (3000), the chain's next tile (1300) and its elimination (3700), of which two steps overlap;
// in the first steps the workers' products (9 tiles per SIMD of 384 matrix-core cycles each).  Before, one wave ran the
// chain, its factor by readlane and 32 x 32 x 2 products (7400 cycles a tile), with a barrier per step, and the loads went
// through the mirrored element, four times over every line.  One r = 256 matrix 48 -> 38 us, r = 128 24 -> 19,
// r = 72 14.5 -> 13; 4096 x 4096, r = 256: 356 -> 335 us a step, 8192 x 8192, r = 2048: 4350 -> 4200,
// four 1024-wide fp32 matrices, r = 128: 333 -> 321, six ragged ones, r = 136: 514 -> 499.  Sixteen waves
// (twelve workers) are no faster and leave no registers for another stream's kernels beside it.
#pragma once

#include <type_traits>

#include "od_common.h"
#include "od_kernels.h"

namespace od {

constexpr int kCholMax = kLeafRank;    // largest block one workgroup factors
constexpr int kCT = 32;                // tile size
constexpr int kCNT = kCholMax / kCT;   // 8 tiles per side
constexpr int kCholThreads = 768;      // three waves per SIMD
constexpr int kCWorkers = 8;
constexpr int kCSlots = 4;             // off-diagonal tiles per worker: 28 over 8 workers
constexpr int kCholInverseWave = 9, kCholOutWave = 11;
constexpr int kPPitch = 80;            // bytes per row of a pre-split operand tile (32 bf16 + pad)
constexpr int kPPlane = kCT * kPPitch; // bytes per part of a pre-split tile
constexpr int kPTile = 3 * kPPlane;    // bytes per pre-split tile
// A finished group of four rows of a diagonal tile in LDS: -t as [4][kGroupPitch] floats (columns left of the
// group are not defined), then its 4 x 4 block: reciprocals of the diagonal, (01 02 03 12), (13 23).
constexpr int kGroupPitch = 48, kGroupCoef = 4 * kGroupPitch, kGroupFloats = kGroupCoef + 12;
// LDS: V(J, J) pre-split as left operand | panel[8] pre-split -T(J, K)^T | vpanel[8] pre-split V(J, I); before step I: the waiting tile (I, I) | groups of
// even / odd steps | two tile images: S(J, J+1) for the chain | counters
constexpr int kCholOffPanel = kPTile;
constexpr int kCholOffVPanel = kCholOffPanel + kCNT * kPTile;
constexpr int kCholOffGroups = kCholOffVPanel + kCNT * kPTile;
constexpr int kCholOffStash = kCholOffGroups + 2 * 8 * kGroupFloats * 4;
constexpr int kCholOffSync = kCholOffStash + 2 * 4096;
struct CholSync {
  int groups;              // groups finished by the chain, 8 per step
  int updated;             // workers past the updates of a step, summed over the steps
  int v_ready;             // steps whose V(J, J) is in place
  int t_done;              // steps whose T(J, J) has been read
  int rows[kCNT];          // panel tiles of step J published
  int cols[kCNT];          // V tiles of step J published
  int s_ready[kCNT];       // S(J, J+1) has its last update and is in the stash
  int diag[kCNT];          // waiting tile (K, K): loaded, and updates so far
};
constexpr int kCholLds = kCholOffSync + (int)sizeof(CholSync);
constexpr int kCholSpinLimit = 1 << 20;  // bound of every wait below (never reached)

struct CholArgs {
  WsArr src;           // Gram block source: `splits` partial sums, `split_stride` elements apart
  int splits;
  int64_t split_stride;
  WsArr t, w;          // outputs, r x r each (ld r)
  int r;               // matrix order (ld of everything)
  int blk;             // which diagonal block of kCholMax
  int* info;
  int info_slot;
  Pred pred;           // the matrix is skipped unless its predicate holds
};

// tile (I, K), I < K, of slot s of worker u, four bits per slot, 15 = no tile (kept in scalar registers: a table in
// memory would cost a dependent load per use).  An edge colouring of the complete graph on the eight rows of tiles:
// two tiles of a worker never share a row or column, so a step finds each worker with one tile of its panel at most.
OD_DEV uint32_t own_rows(int u) {
  return u == 0 ? 0xf530u : u == 1 ? 0xf610u : u == 2 ? 0x4210u : u == 3 ? 0xf210u : u == 4 ? 0x5320u : u == 5 ? 0xf431u
       : u == 6 ? 0x4210u : u == 7 ? 0x3210u : 0xffffu;
}
OD_DEV uint32_t own_cols(int u) {
  return u == 0 ? 0xf642u : u == 1 ? 0xf753u : u == 2 ? 0x6537u : u == 3 ? 0xf764u : u == 4 ? 0x7641u : u == 5 ? 0xf752u
       : u == 6 ? 0x5376u : u == 7 ? 0x7645u : 0xffffu;
}
// worker of a wave (15: none)
OD_DEV int worker_of(int wave) { return (int)(0xfffff5f274f163f0ull >> (4 * wave)) & 15; }

// A tile in LDS in accumulator layout: plane q holds registers 4q .. 4q+3
// of every lane (16 bytes per lane, conflict free).
OD_DEV f32x16 load_dtile(const char* p, int lane) {
  f32x16 t;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const f32x4 v = *reinterpret_cast<const f32x4*>(p + q * 1024 + lane * 16);
#pragma unroll
    for (int e = 0; e < 4; ++e) t[4 * q + e] = v[e];
  }
  return t;
}
OD_DEV void store_dtile(char* p, const f32x16& t, int lane) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const f32x4 v = {t[4 * q], t[4 * q + 1], t[4 * q + 2], t[4 * q + 3]};
    *reinterpret_cast<f32x4*>(p + q * 1024 + lane * 16) = v;
  }
}

// workgroup barrier that orders LDS traffic only (outstanding global stores keep flying)
OD_DEV void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

OD_DEV float lane_bcast(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

// Three-way split bf16 operand words of 8 floats.
OD_DEV void split3(const float* x, u32x4* parts) { NumBF<3>::pack(x, 1.f, parts); }

OD_DEV f32x16 mma6(const u32x4* a, const u32x4* b, f32x16 c) {
#pragma unroll
  for (int i = 2; i >= 0; --i)
#pragma unroll
    for (int j = 2 - i; j >= 0; --j) c = mfma_32x32x16<false>(a[i], b[j], c);
  return c;
}

// k-side operand of k-step kk straight from an accumulator tile.
OD_DEV void acc_operand(const f32x16& acc, int kk, u32x4* parts) {
  float x[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) x[e] = acc[8 * kk + e];
  split3(x, parts);
}

// Pre-split operand tile in LDS: the transpose of an accumulator tile (element (row, col) is
// operand row col, k = row), three bf16 planes, each row holding its 32 k in register order
// so that the operand words of k-step kk are one 16-byte read per plane.
OD_DEV void store_presplit(char* tile, const f32x16& acc, int lane) {
  char* p = tile + (lane & 31) * kPPitch + (lane >> 5) * 16;
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) {
    u32x4 parts[3];
    acc_operand(acc, kk, parts);
#pragma unroll
    for (int s = 0; s < 3; ++s) *reinterpret_cast<u32x4*>(p + s * kPPlane + kk * 32) = parts[s];
  }
}
OD_DEV void load_presplit(const char* tile, int lane, int kk, u32x4* parts) {
  const char* p = tile + (lane & 31) * kPPitch + (lane >> 5) * 16 + kk * 32;
#pragma unroll
  for (int s = 0; s < 3; ++s) parts[s] = *reinterpret_cast<const u32x4*>(p + s * kPPlane);
}

// Hand-off between the waves of the workgroup through LDS words.  LDS operations of a wave are carried out in
// order, so what it wrote before the word changes is there for whoever has seen the new value, and what it read has
// been read; only the compiler has to be kept from moving them.  Every wait is bounded, so that a wave can
// always run to the end of the kernel.
OD_DEV void lds_signal_add(int* word, int lane) {
  asm volatile("" ::: "memory");
  if (lane == 0) __hip_atomic_fetch_add(word, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  asm volatile("" ::: "memory");
}
// Returns whether the bound ran out (the caller reports it; the kernel still ends); `expired`: one has already.
// SLEEP: for waits that nothing urgent hangs on, so that they leave LDS and issue slots to the others.
template <bool SLEEP>
OD_DEV bool lds_wait(const int* word, int target, bool expired) {
  for (int spins = 0; !expired; ++spins) {
    const int seen = __builtin_amdgcn_readfirstlane(__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
    if (seen >= target) break;
    if (spins >= kCholSpinLimit) expired = true;
    if constexpr (SLEEP) __builtin_amdgcn_s_sleep(1);
  }
  asm volatile("" ::: "memory");
  return expired;
}

// ---------------------------------------------------------------------------------------
// Diagonal tile: in-place upper Cholesky factor of the symmetric tile `d` and, in `zt`, the
// inverse of its transpose (M = L^-1, lower triangular), both in accumulator layout.
// Returns the 1-based index of the first bad pivot within the tile, or 0.
// ---------------------------------------------------------------------------------------
// The rows a and b, valid in the lanes of half `hh`: a in the lower lane half, b in the upper one.
OD_DEV float half_pair(float a, float b, int hh) {
  // swaps lanes 32..63 of the first operand with lanes 0..31 of the second
  auto pr = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(hh ? pr[1] : pr[0]);
}

OD_DEV f32x16 mfma_f32_k2(float a, float b, f32x16 c) {
  // D(32x32) += A(32x2) B(2x32) in fp32: lane l holds A[l % 32][l / 32] and B[l / 32][l % 32]
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// `nv`: valid rows (a multiple of 8); the tile is the identity beyond them.
//
// For ranks up to 32, where one wave does the whole factorisation.  One serial chain, eight groups of four pivots
// long: per group the two products that update `d`, ten readlanes, four reciprocal square roots with two operations
// each between them.  What counts besides is the number of instructions: rows come by forward substitution (no
// inverse of the 4 x 4 block), are computed in the lane half that holds them only (one lane swap makes the operand of two
// rows), columns left of the diagonal are not masked before the end (they only ever meet each other), and bad
// pivots are found at the end.
OD_DEV int diag_tile_factor(f32x16& d_io, f32x16& zt_out, int lane, int nv) {
  const int c = lane & 31, h = lane >> 5;
  // `d` and `zt` are only ever changed by the matrix-core updates; the finished rows are
  // collected on the side (a finished row of `d` / `zt` itself is never read again)
  f32x16 d = d_io, zt;
  float tfin[16], zfin[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) tfin[v] = zfin[v] = zt[v] = (acc_row(v, lane) == c) ? 1.f : 0.f;
#pragma unroll
  for (int g = 0; g < 8; ++g) {
    const int q = g >> 1, hh = g & 1, src_lane = 32 * hh + 4 * g;
    if (hh == 0 && 8 * q >= nv) break;
    // 4 x 4 diagonal block (upper part), wave-uniform
    const float d00 = lane_bcast(d[4 * q + 0], src_lane + 0), d01 = lane_bcast(d[4 * q + 0], src_lane + 1);
    const float d02 = lane_bcast(d[4 * q + 0], src_lane + 2), d03 = lane_bcast(d[4 * q + 0], src_lane + 3);
    const float d11 = lane_bcast(d[4 * q + 1], src_lane + 1), d12 = lane_bcast(d[4 * q + 1], src_lane + 2);
    const float d13 = lane_bcast(d[4 * q + 1], src_lane + 3), d22 = lane_bcast(d[4 * q + 2], src_lane + 2);
    const float d23 = lane_bcast(d[4 * q + 2], src_lane + 3), d33 = lane_bcast(d[4 * q + 3], src_lane + 3);
    // pivots: the hardware reciprocal square root (1 ulp) is accurate enough here, since the
    // inverse is built from the same rounded values.  A non-positive or non-finite pivot leaves a NaN.
    // New rows of the factor: t_e = (s_e - sum_{b < e} t4[b][e] t_b) / t4[e][e]
    float tn[4], zn[4];
    const float i00 = __builtin_amdgcn_rsqf(d00);
    const float t01 = d01 * i00, t02 = d02 * i00, t03 = d03 * i00;
    const float i11 = __builtin_amdgcn_rsqf(d11 - t01 * t01);
    tn[0] = d[4 * q] * i00;
    const float t12 = (d12 - t01 * t02) * i11, t13 = (d13 - t01 * t03) * i11;
    const float i22 = __builtin_amdgcn_rsqf(d22 - t02 * t02 - t12 * t12);
    tn[1] = (d[4 * q + 1] - t01 * tn[0]) * i11;
    const float t23 = (d23 - t02 * t03 - t12 * t13) * i22;
    const float i33 = __builtin_amdgcn_rsqf(d33 - t03 * t03 - t13 * t13 - t23 * t23);
    tn[2] = (d[4 * q + 2] - t02 * tn[0] - t12 * tn[1]) * i22;
    tn[3] = (d[4 * q + 3] - t03 * tn[0] - t13 * tn[1] - t23 * tn[2]) * i33;
    // rank-4 update of the tile, -T_g^T T_g, as two k = 2 products: the lower lane half
    // carries rows 4g, 4g+2 and the upper half rows 4g+1, 4g+3
    float t01v, t23v;
    if (g < 7) {
      t01v = half_pair(tn[0], tn[1], hh);
      t23v = half_pair(tn[2], tn[3], hh);
      d = mfma_f32_k2(-t01v, t01v, d);
      d = mfma_f32_k2(-t23v, t23v, d);
    }
    __builtin_amdgcn_sched_barrier(0);
    // the same for the inverse, -T_g^T Z_g, while those products run
    zn[0] = zt[4 * q] * i00;
    zn[1] = (zt[4 * q + 1] - t01 * zn[0]) * i11;
    zn[2] = (zt[4 * q + 2] - t02 * zn[0] - t12 * zn[1]) * i22;
    zn[3] = (zt[4 * q + 3] - t03 * zn[0] - t13 * zn[1] - t23 * zn[2]) * i33;
    if (g < 7) {
      zt = mfma_f32_k2(-t01v, half_pair(zn[0], zn[1], hh), zt);
      zt = mfma_f32_k2(-t23v, half_pair(zn[2], zn[3], hh), zt);
    }
    // the rows of this group are final (register 4q + e of lane half hh; the other half's
    // turn for these registers comes with the next group)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (hh == 0 || h == 1) { tfin[4 * q + e] = tn[e]; zfin[4 * q + e] = zn[e]; }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  // column c starts at its diagonal, whose entry tells whether the pivot was a positive number
  // below 3e38 (the root of that here); the first column where it was not is the breakdown
  bool ok = true;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int row = acc_row(v, lane);
    if (row == c) ok = tfin[v] > 0.f && tfin[v] < 1.7320508e19f;
    d_io[v] = c < row ? 0.f : tfin[v];
    zt_out[v] = zfin[v];
  }
  const uint64_t failed = __ballot(!ok);
  const uint32_t columns = (uint32_t)failed | (uint32_t)(failed >> 32);
  return columns != 0u ? __ffs((int)columns) : 0;
}

// ---------------------------------------------------------------------------------------
// The chain waves hold 32 x 32 tiles as 16 x 16 blocks in the layout of the 16 x 16 x 4 product: register v of lane l
// is row 4 (l / 16) + v, column l % 16.  Rows 4 g .. 4 g + 3 are then the four registers of one 16-lane row of the
// wave (g % 4): an element of a row reaches the lanes of that row as a DPP operand of the next instruction (no
// readlane, no trip through scalar registers), and the rank-4 update of a block is a single product.
// ---------------------------------------------------------------------------------------
template <int N>
OD_DEV float row_bcast(float x) {       // lane N of each 16-lane row
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x150 + N, 0xf, 0xf, true));
}
OD_DEV f32x4 mfma_16x16x4(float a, float b, f32x4 c) {
  // D(16x16) += A(16x4) B(4x16) in fp32: lane l holds A[l % 16][l / 16] and B[l / 16][l % 16]
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
// operand of a rank-4 update: lane row e of the result is row G of t_e
template <int G>
OD_DEV float gather_rows(float t0, float t1, float t2, float t3) {
  // swaps the odd lane rows of the first operand with the even ones of the second
  const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(t0), __float_as_uint(t1), false, false);
  const auto q = __builtin_amdgcn_permlane16_swap(__float_as_uint(t2), __float_as_uint(t3), false, false);
  const auto s = __builtin_amdgcn_permlane32_swap(p[G & 1], q[G & 1], false, false);
  return __uint_as_float(s[G >> 1]);
}

// Group g of the diagonal tile with blocks d00, d01, d11 (by symmetry the fourth is not kept): factors its 4 x 4
// diagonal block, eliminates, publishes the rows.  The hardware reciprocal square root (1 ulp) is accurate enough, since
// everything else follows from the same rounded values.  A non-positive or non-finite pivot leaves a NaN.
template <int g>
OD_DEV void chain_group(f32x4& d00, f32x4& d01, f32x4& d11, int lane, float* grp, int* groups, int count) {
  constexpr int G = g & 3, C = 4 * G;
  constexpr bool low = g < 4;
  const f32x4 x = low ? d00 : d11;
  const float i0 = __builtin_amdgcn_rsqf(row_bcast<C>(x[0]));
  const float t0 = x[0] * i0;
  const float m01 = row_bcast<C + 1>(t0), m02 = row_bcast<C + 2>(t0), m03 = row_bcast<C + 3>(t0);
  const float x1 = x[1] - m01 * t0;
  const float i1 = __builtin_amdgcn_rsqf(row_bcast<C + 1>(x1));
  const float t1 = x1 * i1;
  const float m12 = row_bcast<C + 2>(t1), m13 = row_bcast<C + 3>(t1);
  const float x2 = x[2] - m02 * t0 - m12 * t1;
  const float i2 = __builtin_amdgcn_rsqf(row_bcast<C + 2>(x2));
  const float t2 = x2 * i2;
  const float m23 = row_bcast<C + 3>(t2);
  const float x3 = x[3] - m03 * t0 - m13 * t1 - m23 * t2;
  const float i3 = __builtin_amdgcn_rsqf(row_bcast<C + 3>(x3));
  const float t3 = x3 * i3;
  const float a = gather_rows<G>(t0, t1, t2, t3);
  const float na = -a;
  float* row = grp + (lane >> 4) * kGroupPitch + (lane & 15);
  if constexpr (low) {
    if constexpr (G < 3) d00 = mfma_16x16x4(na, a, d00);
    __builtin_amdgcn_sched_barrier(0);          // the next group waits for that product; the rest runs beside it
    const float u0 = d01[0] * i0;
    const float u1 = (d01[1] - m01 * u0) * i1;
    const float u2 = (d01[2] - m02 * u0 - m12 * u1) * i2;
    const float u3 = (d01[3] - m03 * u0 - m13 * u1 - m23 * u2) * i3;
    const float b = gather_rows<G>(u0, u1, u2, u3);
    const float nb = -b;
    if constexpr (G < 3) d01 = mfma_16x16x4(na, b, d01);
    d11 = mfma_16x16x4(nb, b, d11);
    row[0] = na;
    row[16] = nb;
  } else {
    if constexpr (G < 3) d11 = mfma_16x16x4(na, a, d11);
    row[16] = na;
  }
  asm volatile("" ::: "memory");
  if (lane == 16 * G) {
    *reinterpret_cast<f32x4*>(grp + kGroupCoef) = f32x4{i0, i1, i2, i3};
    *reinterpret_cast<f32x4*>(grp + kGroupCoef + 4) = f32x4{m01, m02, m03, m12};
    *reinterpret_cast<f32x2*>(grp + kGroupCoef + 8) = f32x2{m13, m23};
    asm volatile("" ::: "memory");
    __hip_atomic_store(groups, count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  asm volatile("" ::: "memory");
}

// The 4 x 4 block of a group as the others read it.  (Read as whole vectors without a spare element: the register of
// one would be given to the next load, which then waits for this one.)
struct GroupCoef {
  f32x4 inv, m;                // m: 01 02 03 12
  f32x2 n;                     // 13 23
};
OD_DEV GroupCoef load_coef(const float* grp) {
  return GroupCoef{*reinterpret_cast<const f32x4*>(grp + kGroupCoef), *reinterpret_cast<const f32x4*>(grp + kGroupCoef + 4),
                   *reinterpret_cast<const f32x2*>(grp + kGroupCoef + 8)};
}
// rows of a group by forward substitution
OD_DEV void solve_rows(const GroupCoef& k, float x0, float x1, float x2, float x3, float (&t)[4]) {
  t[0] = x0 * k.inv[0];
  t[1] = (x1 - k.m[0] * t[0]) * k.inv[1];
  t[2] = (x2 - k.m[1] * t[0] - k.m[3] * t[1]) * k.inv[2];
  t[3] = (x3 - k.m[2] * t[0] - k.n[0] * t[1] - k.n[1] * t[2]) * k.inv[3];
}
// A group as a chain wave reads it: coefficients and the rows as product operands.
struct GroupRows {
  GroupCoef k;
  float a0, a1;
};
OD_DEV GroupRows load_group(const float* step, int g, int lane) {
  const float* grp = step + g * kGroupFloats;
  const float* row = grp + (lane >> 4) * kGroupPitch + (lane & 15);
  return GroupRows{load_coef(grp), row[0], row[16]};
}
// Group g for the tile right of the diagonal one (s, 16 x 16 blocks [row half][column half]) and the next
// diagonal tile (n00, n01, n11, negated).
template <int g>
OD_DEV void follow_group(f32x4 (&s)[2][2], f32x4& n00, f32x4& n01, f32x4& n11, const GroupRows& in) {
  constexpr int G = g & 3, H = g >> 2;
  float b[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    float t[4];
    solve_rows(in.k, s[H][c][0], s[H][c][1], s[H][c][2], s[H][c][3], t);
    b[c] = gather_rows<G>(t[0], t[1], t[2], t[3]);
    if constexpr (G < 3) s[H][c] = mfma_16x16x4(H == 0 ? in.a0 : in.a1, b[c], s[H][c]);
    else if constexpr (H == 0) s[1][c] = mfma_16x16x4(in.a1, b[c], s[1][c]);
  }
  if constexpr (g < 3) {
#pragma unroll
    for (int c = 0; c < 2; ++c) s[1][c] = mfma_16x16x4(in.a1, b[c], s[1][c]);
  }
  n00 = mfma_16x16x4(b[0], b[0], n00);
  n01 = mfma_16x16x4(b[0], b[1], n01);
  n11 = mfma_16x16x4(b[1], b[1], n11);
}
// Four groups, the next one's reads ahead of a group's arithmetic.
template <int H>
OD_DEV void follow_half(f32x4 (&s)[2][2], f32x4& n00, f32x4& n01, f32x4& n11, int lane, const float* step) {
  GroupRows in0 = load_group(step, 4 * H, lane);
  GroupRows in1 = load_group(step, 4 * H + 1, lane);
  __builtin_amdgcn_sched_barrier(0);
  follow_group<4 * H>(s, n00, n01, n11, in0);
  in0 = load_group(step, 4 * H + 2, lane);
  __builtin_amdgcn_sched_barrier(0);
  follow_group<4 * H + 1>(s, n00, n01, n11, in1);
  in1 = load_group(step, 4 * H + 3, lane);
  __builtin_amdgcn_sched_barrier(0);
  follow_group<4 * H + 2>(s, n00, n01, n11, in0);
  follow_group<4 * H + 3>(s, n00, n01, n11, in1);
}

// Group g for the identity tile: z00, z10, z11 are eliminated, f00, f10, f11 receive the finished rows.  Waits for the
// group; what is read along with the count is valid once the count is there.
template <int g>
OD_DEV bool inverse_group(f32x4& z00, f32x4& z10, f32x4& z11, f32x4& f00, f32x4& f10, f32x4& f11, int lane, const float* step, const int* groups, int count, bool expired) {
  constexpr int G = g & 3;
  const float* grp = step + g * kGroupFloats;
  const float* row = grp + (lane >> 4) * kGroupPitch + (lane & 15);
  expired = lds_wait<false>(groups, count, expired);
  const GroupCoef k = load_coef(grp);
  const float na = row[0], nb = row[16];
  const bool mine = (lane >> 4) == G;
  float t[4], u[4];
  if constexpr (g < 4) {
    solve_rows(k, z00[0], z00[1], z00[2], z00[3], t);
    const float b = gather_rows<G>(t[0], t[1], t[2], t[3]);
    if constexpr (G < 3) z00 = mfma_16x16x4(na, b, z00);
    z10 = mfma_16x16x4(nb, b, z10);
#pragma unroll
    for (int e = 0; e < 4; ++e) f00[e] = mine ? t[e] : f00[e];
  } else {
    solve_rows(k, z10[0], z10[1], z10[2], z10[3], t);
    solve_rows(k, z11[0], z11[1], z11[2], z11[3], u);
    if constexpr (G < 3) {
      z10 = mfma_16x16x4(nb, gather_rows<G>(t[0], t[1], t[2], t[3]), z10);
      z11 = mfma_16x16x4(nb, gather_rows<G>(u[0], u[1], u[2], u[3]), z11);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      f10[e] = mine ? t[e] : f10[e];
      f11[e] = mine ? u[e] : f11[e];
    }
  }
  return expired;
}

// The factorisation of block `a.blk` of matrix `z` by one workgroup of kCholThreads threads;
// `lds_raw`: kCholLds bytes.
OD_DEV void chol256_block(const CholArgs& a, int z, char* lds_raw) {
  char* voperand = lds_raw;
  char* panel = lds_raw + kCholOffPanel;
  char* vpanel = lds_raw + kCholOffVPanel;
  float* const group_data = reinterpret_cast<float*>(lds_raw + kCholOffGroups);
  char* stash = lds_raw + kCholOffStash;
  CholSync& sync = *reinterpret_cast<CholSync*>(lds_raw + kCholOffSync);

  const int tid = threadIdx.x, lane = tid & 63;
  // uniform over the workgroup, before any barrier or LDS hand-off
  if (a.pred.scal != nullptr && (a.pred.scal[z * kScalPerMat + a.pred.slot] > a.pred.thr) != (a.pred.want != 0)) return;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int worker = worker_of(wave);
  const int r = a.r;
  const int o = a.blk * kCholMax;
  const int nb = (r - o) < kCholMax ? (r - o) : kCholMax;     // order of this block
  const int nt = (nb + kCT - 1) / kCT;                        // active tiles per side
  const int64_t off = (int64_t)o * r + o;
  const float* src = a.src.base + (int64_t)z * a.src.stride + off;
  float* tg = a.t.base + (int64_t)z * a.t.stride + off;
  float* wg = a.w.base + (int64_t)z * a.w.stride + off;
  if (tid < (int)(sizeof(CholSync) / sizeof(int))) reinterpret_cast<int*>(&sync)[tid] = 0;
  lds_barrier();
  bool expired = false;
  auto wait = [&](const int* word, int target) { expired = lds_wait<false>(word, target, expired); };
  auto wait_idle = [&](const int* word, int target) { expired = lds_wait<true>(word, target, expired); };
  auto valid_rows = [&](int J) { return (nb - J * kCT) < kCT ? (nb - J * kCT) : kCT; };
  auto step_groups = [&](int J) { return group_data + (J & 1) * 8 * kGroupFloats; };
  // Offset of element (row, col), clamped into the block, so that the loads of a tile are unconditional; `inside` replaces
  // what lies beyond by the identity.  Lanes read along a row: every line of the source is fetched once.
  auto offset = [&](int row, int col) { return (uint32_t)((row < nb ? row : nb - 1) * r + (col < nb ? col : nb - 1)); };
  auto inside = [&](float v, int row, int col) { return row < nb && col < nb ? v : row == col ? 1.f : 0.f; };

  if (worker == 15 && wave < kCholInverseWave) {
    // ================================ the chain ================================
    const int self = wave >> 2, j = lane & 15, lr = lane >> 4;
    f32x4 d00, d01, d11;
    if (self == 0) {
      uint32_t at[3][4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        at[0][v] = offset(4 * lr + v, j);
        at[1][v] = offset(4 * lr + v, 16 + j);
        at[2][v] = offset(16 + 4 * lr + v, 16 + j);
      }
      d00 = d01 = d11 = f32x4{0.f, 0.f, 0.f, 0.f};
      const float* p = src;
      for (int sp = 0; sp < a.splits; ++sp) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          d00[v] += p[at[0][v]];
          d01[v] += p[at[1][v]];
          d11[v] += p[at[2][v]];
        }
        p += a.split_stride;
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        d00[v] = inside(d00[v], 4 * lr + v, j);
        d01[v] = inside(d01[v], 4 * lr + v, 16 + j);
        d11[v] = inside(d11[v], 16 + 4 * lr + v, 16 + j);
      }
    }
    // 16 x 16 block (rh, ch) of a tile image
    auto block_of = [&](const char* image, int rh, int ch) {
      return *reinterpret_cast<const f32x4*>(image + (2 * rh + (lr >> 1)) * 1024 + (16 * ch + j + 32 * (lr & 1)) * 16);
    };
    for (int J = 0; J < nt; ++J) {
      float* grp = step_groups(J);
      if ((J & 1) == self) {
        // the groups of step J - 2 have been read
        if (J >= 2) wait(&sync.t_done, J - 1);
        const int nv = valid_rows(J), base = 8 * J;
        auto at = [&](int g) { return grp + g * kGroupFloats; };
        chain_group<0>(d00, d01, d11, lane, at(0), &sync.groups, base + 1);
        chain_group<1>(d00, d01, d11, lane, at(1), &sync.groups, base + 2);
        if (nv > 8) {
          chain_group<2>(d00, d01, d11, lane, at(2), &sync.groups, base + 3);
          chain_group<3>(d00, d01, d11, lane, at(3), &sync.groups, base + 4);
        }
        if (nv > 16) {
          chain_group<4>(d00, d01, d11, lane, at(4), &sync.groups, base + 5);
          chain_group<5>(d00, d01, d11, lane, at(5), &sync.groups, base + 6);
        }
        if (nv > 24) {
          chain_group<6>(d00, d01, d11, lane, at(6), &sync.groups, base + 7);
          chain_group<7>(d00, d01, d11, lane, at(7), &sync.groups, base + 8);
        }
      } else if (J + 1 < nt) {
        wait(&sync.diag[J + 1], 1 + J);
        const char* image = vpanel + (J + 1) * kPTile;
        f32x4 n00 = block_of(image, 0, 0), n01 = block_of(image, 0, 1), n11 = block_of(image, 1, 1);
        wait(&sync.s_ready[J], 1);
        const char* si = stash + (J & 1) * 4096;
        f32x4 s[2][2] = {{block_of(si, 0, 0), block_of(si, 0, 1)}, {block_of(si, 1, 0), block_of(si, 1, 1)}};
        wait(&sync.groups, 8 * J + 4);
        follow_half<0>(s, n00, n01, n11, lane, grp);
        wait(&sync.groups, 8 * J + 8);
        follow_half<1>(s, n00, n01, n11, lane, grp);
        d00 = -n00;
        d01 = -n01;
        d11 = -n11;
      }
    }
  } else if (wave == kCholInverseWave) {
    // ================================ V(J, J) ================================
    const int j = lane & 15, lr = lane >> 4;
    // in the left operand k = column 16 ch + j of V sits where the k-side operand has it in register order
    // (lanes j and j + 1 swap halves: even lanes write the even rows of a pair, odd lanes the odd ones)
    char* const left = voperand + (4 * lr + (j & 1)) * kPPitch + ((j >> 2) & 1) * 16 + ((j >> 3) * 4 + (j & 2)) * 2;
    const uint32_t pick = (j & 1) ? 0x03020706u : 0x05040100u;
    auto pair = [&](uint32_t w) { return __builtin_amdgcn_perm((uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0xb1, 0xf, 0xf, true), w, pick); };
#pragma unroll
    for (int s = 0; s < 3; ++s)
#pragma unroll
      for (int v = 0; v < 2; ++v) *reinterpret_cast<uint32_t*>(left + s * kPPlane + 2 * v * kPPitch + 32) = 0u;      // block (0, 1)
    for (int J = 0; J < nt; ++J) {
      const float* step = step_groups(J);
      const int nv = valid_rows(J), base = 8 * J;
      f32x4 z00, z10, z11;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        z00[v] = z11[v] = 4 * lr + v == j ? 1.f : 0.f;
        z10[v] = 0.f;
      }
      f32x4 f00 = z00, f10 = z10, f11 = z11;
      expired = inverse_group<0>(z00, z10, z11, f00, f10, f11, lane, step, &sync.groups, base + 1, expired);
      expired = inverse_group<1>(z00, z10, z11, f00, f10, f11, lane, step, &sync.groups, base + 2, expired);
      if (nv > 8) {
        expired = inverse_group<2>(z00, z10, z11, f00, f10, f11, lane, step, &sync.groups, base + 3, expired);
        expired = inverse_group<3>(z00, z10, z11, f00, f10, f11, lane, step, &sync.groups, base + 4, expired);
      }
      if (nv > 16) {
        expired = inverse_group<4>(z00, z10, z11, f00, f10, f11, lane, step, &sync.groups, base + 5, expired);
        expired = inverse_group<5>(z00, z10, z11, f00, f10, f11, lane, step, &sync.groups, base + 6, expired);
      }
      if (nv > 24) {
        expired = inverse_group<6>(z00, z10, z11, f00, f10, f11, lane, step, &sync.groups, base + 7, expired);
        expired = inverse_group<7>(z00, z10, z11, f00, f10, f11, lane, step, &sync.groups, base + 8, expired);
      }
      // split; the left operand of the step before has been read
      u32x4 w0[3], w1[3];
      {
        const float x0[8] = {f00[0], f00[1], f00[2], f00[3], f10[0], f10[1], f10[2], f10[3]};
        const float x1[8] = {0.f, 0.f, 0.f, 0.f, f11[0], f11[1], f11[2], f11[3]};
        split3(x0, w0);
        split3(x1, w1);
      }
      if (J > 0) {
        wait(&sync.rows[J - 1], nt - J);
        wait(&sync.cols[J - 1], J);
      }
      char* const vp = vpanel + J * kPTile + j * kPPitch + (lr & 1) * 16 + (lr >> 1) * 8;
#pragma unroll
      for (int s = 0; s < 3; ++s) {
#pragma unroll
        for (int v = 0; v < 2; ++v) {
          *reinterpret_cast<uint32_t*>(left + s * kPPlane + 2 * v * kPPitch) = pair(w0[s][v]);
          *reinterpret_cast<uint32_t*>(left + s * kPPlane + (16 + 2 * v) * kPPitch) = pair(w0[s][2 + v]);
          *reinterpret_cast<uint32_t*>(left + s * kPPlane + (16 + 2 * v) * kPPitch + 32) = pair(w1[s][2 + v]);
        }
        *reinterpret_cast<u32x2*>(vp + s * kPPlane) = u32x2{w0[s][0], w0[s][1]};
        *reinterpret_cast<u32x2*>(vp + s * kPPlane + 32) = u32x2{w0[s][2], w0[s][3]};
        *reinterpret_cast<u32x2*>(vp + s * kPPlane + 16 * kPPitch) = u32x2{0u, 0u};
        *reinterpret_cast<u32x2*>(vp + s * kPPlane + 16 * kPPitch + 32) = u32x2{w1[s][2], w1[s][3]};
      }
      lds_signal_add(&sync.v_ready, lane);
      lds_signal_add(&sync.cols[J], lane);
      // W(c, i) = V(i, c): four consecutive columns per store
      auto put = [&](int rh, int ch, const f32x4& f) {
        if (16 * ch + j < nv && 16 * rh + 4 * lr < nv) *reinterpret_cast<f32x4*>(wg + (int64_t)(J * kCT + 16 * ch + j) * r + J * kCT + 16 * rh + 4 * lr) = f;
      };
      put(0, 0, f00);
      put(1, 0, f10);
      put(0, 1, f32x4{0.f, 0.f, 0.f, 0.f});
      put(1, 1, f11);
    }
  } else if (wave == kCholOutWave) {
    // ================================ T(J, J), zeros ================================
    const int col = lane & 31, half = lane >> 5;
    for (int J = 0; J < nt; ++J) {
      const float* step = step_groups(J);
      const int nv = valid_rows(J);
      wait_idle(&sync.groups, 8 * J + nv / 4);
      // T_JJ, and whether every pivot was a positive number below 3e38 (its root is on the diagonal)
      bool ok = true;
      float* tp = tg + (int64_t)(J * kCT + 4 * half) * r + J * kCT + col;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (8 * q < nv) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int row = 8 * q + 4 * half + e;
            const float t = -step[(2 * q + half) * kGroupFloats + e * kGroupPitch + col];
            if (row == col) ok = t > 0.f && t < 1.7320508e19f;
            if (col < nv) tp[(int64_t)(8 * q + e) * r] = col < row ? 0.f : t;
          }
        }
      }
      lds_signal_add(&sync.t_done, lane);
      const uint64_t failed = __ballot(!ok);
      const uint32_t columns = (uint32_t)failed | (uint32_t)(failed >> 32);
      if (lane == 0 && columns != 0u) atomicCAS(&a.info[z * kInfoPerMat + a.info_slot], 0, o + J * kCT + __ffs((int)columns));
      // tiles left of the diagonal of T and W
      for (int K = 0; K < J; ++K)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int gi = J * kCT + 8 * q + (lane >> 3), gj = K * kCT + (lane & 7) * 4;
          if (gi < nb) {
            const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
            *reinterpret_cast<f32x4*>(tg + (int64_t)gi * r + gj) = zero;
            *reinterpret_cast<f32x4*>(wg + (int64_t)gi * r + gj) = zero;
          }
        }
    }
  } else {
    // ================================ the workers ================================
    const int col = lane & 31, half = lane >> 5;
    const uint32_t ownI = own_rows(worker), ownK = own_cols(worker);
    // One address per lane and a uniform offset per row (64-bit addresses per element had kept the vector units busy for
    // 20000 cycles).  The order is a multiple of 8, so the rows of a register group are inside or outside together.
    auto load_tile = [&](int I, int K) {
      f32x16 t;
      const float* p = src;
      const uint32_t at = (uint32_t)(4 * half * r + (K * kCT + col < nb ? K * kCT + col : nb - 1));
#pragma unroll
      for (int v = 0; v < 16; ++v) t[v] = 0.f;
      for (int sp = 0; sp < a.splits; ++sp) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int row8 = I * kCT + 8 * (v >> 2);
          t[v] += (p + ((row8 < nb ? row8 : nb - 8) + (v & 3)) * r)[at];
        }
        p += a.split_stride;
      }
      if (K * kCT + kCT > nb) {
#pragma unroll
        for (int v = 0; v < 16; ++v) t[v] = inside(t[v], I * kCT + acc_row(v, lane), K * kCT + col);
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) t[v] = -t[v];
      return t;
    };
    // the diagonal tiles behind the first wait in LDS for their updates
    const int waiting = kCWorkers - worker;
    f32x16 acc[kCSlots], dt;
    if (waiting < nt) dt = load_tile(waiting, waiting);
#pragma unroll
    for (int s = 0; s < kCSlots; ++s) {
      const int I = (int)(ownI >> (4 * s)) & 15, K = (int)(ownK >> (4 * s)) & 15;
      if (K < nt) acc[s] = load_tile(I, K);
      else {
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[s][v] = 0.f;
      }
    }
    if (waiting < nt) {
      store_dtile(vpanel + waiting * kPTile, dt, lane);
      lds_signal_add(&sync.diag[waiting], lane);
    }
#pragma unroll
    for (int s = 0; s < kCSlots; ++s) {
      const int I = (int)(ownI >> (4 * s)) & 15, K = (int)(ownK >> (4 * s)) & 15;
      if (I == 0 && K == 1 && K < nt) {
        store_dtile(stash, acc[s], lane);
        lds_signal_add(&sync.s_ready[0], lane);
      }
    }
    // tile += A^T B with both operands pre-split in LDS
    auto lds_product = [&](f32x16& tile, const char* pa, const char* pb) {
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        u32x4 ap[3], bp[3];
        load_presplit(pa, lane, kk, ap);
        load_presplit(pb, lane, kk, bp);
        tile = mma6(ap, bp, tile);
      }
    };
    // the waiting diagonal tile (K, K), negated, += T(J, K)^T T(J, K); (J+1, J+1) is with the chain by now
    auto update_diag = [&](int J, int K) {
      wait(&sync.diag[K], 1 + J);
      char* dk = vpanel + K * kPTile;
      f32x16 d = load_dtile(dk, lane);
      lds_product(d, panel + K * kPTile, panel + K * kPTile);
      store_dtile(dk, d, lane);
      lds_signal_add(&sync.diag[K], lane);
    };
    for (int J = 0; J < nt; ++J) {
      // ---- row J of T and row J of V: at most one tile per worker
      const int nv = valid_rows(J);
      int sel = -1, I = J, K = J;
#pragma unroll
      for (int s = 0; s < kCSlots; ++s) {
        const int Is = (int)(ownI >> (4 * s)) & 15, Ks = (int)(ownK >> (4 * s)) & 15;
        if (Ks < nt && (Is == J || Ks == J)) { sel = s; I = Is; K = Ks; }
      }
      f32x16 x;
      if (sel >= 0) {
        u32x4 b0[3], b1[3];
        {
          const f32x16 s = sel == 0 ? acc[0] : sel == 1 ? acc[1] : sel == 2 ? acc[2] : acc[3];
          acc_operand(s, 0, b0);
          acc_operand(s, 1, b1);
        }
        wait(&sync.v_ready, J + 1);
#pragma unroll
        for (int v = 0; v < 16; ++v) x[v] = 0.f;
        {
          u32x4 a0[3], a1[3];
          load_presplit(voperand, lane, 0, a0);
          load_presplit(voperand, lane, 1, a1);
          x = mma6(a0, b0, x);
          x = mma6(a1, b1, x);
        }
        // the panel of the step before has been read
        wait(&sync.updated, kCWorkers * J);
        if (I == J) {
          // -T(J, K): published first, the others wait for it
          store_presplit(panel + K * kPTile, x, lane);
          lds_signal_add(&sync.rows[J], lane);
          // from now on the sum -S'(K, J)
#pragma unroll
          for (int s = 0; s < kCSlots; ++s)
            if (sel == s) {
#pragma unroll
              for (int v = 0; v < 16; ++v) acc[s][v] = 0.f;
            }
          if (K == J + 2) update_diag(J, K);       // the chain needs this one next
        } else {
          store_presplit(vpanel + I * kPTile, x, lane);       // V(J, I)
          lds_signal_add(&sync.cols[J], lane);
        }
      }
      // ---- updates of the step: -S(I, K) += T(J, I)^T T(J, K) for J < I < K, the one that the chain waits for
      // first;  -S'(K, I) -= T(J, K)^T V(J, I) for I <= J < K
      if (J + 1 < nt) {
        wait(&sync.rows[J], nt - 1 - J);
#pragma unroll
        for (int s = 0; s < kCSlots; ++s) {
          const int Is = (int)(ownI >> (4 * s)) & 15, Ks = (int)(ownK >> (4 * s)) & 15;
          if (Is == J + 1 && Ks == J + 2 && Ks < nt) {
            lds_product(acc[s], panel + Is * kPTile, panel + Ks * kPTile);
            store_dtile(stash + ((J + 1) & 1) * 4096, acc[s], lane);
            lds_signal_add(&sync.s_ready[J + 1], lane);
          }
        }
#pragma unroll
        for (int s = 0; s < kCSlots; ++s) {
          const int Is = (int)(ownI >> (4 * s)) & 15, Ks = (int)(ownK >> (4 * s)) & 15;
          if (Is > J && Ks < nt && !(Is == J + 1 && Ks == J + 2)) lds_product(acc[s], panel + Is * kPTile, panel + Ks * kPTile);
        }
        wait_idle(&sync.cols[J], J + 1);
#pragma unroll
        for (int s = 0; s < kCSlots; ++s) {
          const int Is = (int)(ownI >> (4 * s)) & 15, Ks = (int)(ownK >> (4 * s)) & 15;
          if (Is <= J && Ks > J && Ks < nt) lds_product(acc[s], panel + Ks * kPTile, vpanel + Is * kPTile);
        }
        if (sel >= 0 && I == J && K > J + 2) update_diag(J, K);
        lds_signal_add(&sync.updated, lane);
      }
      // ---- the panel tile to memory
      if (sel >= 0 && I == J) {
        if (K * kCT + col < nb) {
          float* tp = tg + (int64_t)(J * kCT + 4 * half) * r + K * kCT + col;
#pragma unroll
          for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) tp[(int64_t)(8 * q + e) * r] = -x[4 * q + e];
        }
      } else if (sel >= 0) {
        // W(I*32 + c, J*32 + i) = V(J, I)(i, c): four consecutive columns per store
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (8 * q < nv) {
            const f32x4 v4 = {x[4 * q], x[4 * q + 1], x[4 * q + 2], x[4 * q + 3]};
            *reinterpret_cast<f32x4*>(wg + (int64_t)(I * kCT + col) * r + J * kCT + 8 * q + 4 * half) = v4;
          }
        }
      }
    }
  }
  // a wait that ran out means a tile was used before its producer finished: the factors of this
  // matrix are wrong, which the breakdown word says (the warning bit says why)
  if (expired && lane == 0) {
    atomicOr(&a.info[z * kInfoPerMat + kWarnSlot], kWarnWaitExpired);
    atomicCAS(&a.info[z * kInfoPerMat + a.info_slot], 0, o + 1);
  }
}

}  // namespace od

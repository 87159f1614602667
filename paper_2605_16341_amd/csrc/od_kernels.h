// Host-callable launchers of the HIP kernels of the Orth-Dion step (defined in
// od_kernels.hip).  Every launcher only enqueues work on `stream`; none synchronises
// or allocates.  A launcher takes any number of launch batches (matrices of one shape class,
// i.e. equal m, n, r and leading dimensions); batches that need the same kernel share a launch.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace od {

// Caller-owned buffers of one matrix.  The table of all matrices of a step lives in the workspace
// (slot order); the first kernel of the step writes it from its arguments.
struct MatEntry {
  void* X;
  const void* G;
  float* M;
  float* Q;
};

// largest rank that one workgroup factors (launch_cholinv)
constexpr int kLeafRank = 256;
// Gram matrices: 64 x 64 tiles below this many 128 x 128 ones (of the full square, all splits and matrices together)
constexpr int kSmallGramTiles = 512;

enum Prec : int { PREC_F16 = 0, PREC_BF3 = 1 };   // operand format of the big contractions

struct ClassDims {
  int m, n, r, nb;
  int64_t ldx, ldg, ldm;
  int x_bf16, g_bf16;
  int col_fast;        // error-feedback pass: consecutive workgroups walk along a row of tiles (set by its launcher)
};

// A workspace array with one slice per matrix of the class.
struct WsArr {
  float* base;
  int64_t stride;      // elements between consecutive matrices
};

// A workspace array of pre-scaled fp16 operand words, one slice per matrix.
struct HalfArr {
  uint16_t* base;
  int64_t stride;      // elements between consecutive matrices
};

// A launch made conditional, matrix by matrix, on a scale-table word written by an earlier
// kernel of the same stream: matrix z is processed only if
// (scal[z * kScalPerMat + slot] > thr) == (want != 0).  scal == nullptr: unconditional.
struct Pred {
  const float* scal;
  int slot;
  float thr;
  int want;
};

// scal layout per matrix (floats): [1] scale of R, [2] / [3] largest deviation of the
// first-pass Gram matrix of the left / right factor from identity, [8..39] sampled row sums
// of squares of B
constexpr int kScalPerMat = 40;
constexpr int kScalSample = 8;
// info layout per matrix (ints): [0] left-factor breakdown column, [1] right-factor
// breakdown column (1-based, 0 = none), [2] zero-column flag of ColNorm, [3] warning bits
// (results are delivered, but with less accuracy than the precision mode promises)
constexpr int kInfoPerMat = 4;
constexpr int kWarnSlot = 3;
constexpr int kWarnBClipped = 1;       // an entry of B = M + G exceeded the fp16 range under its sampled scale
constexpr int kWarnRClipped = 2;       // the same for R = B^T P
constexpr int kWarnBScaleBlind = 4;    // the sampled rows of B were all zero although B is not
constexpr int kWarnWaitExpired = 8;    // a bounded wait inside the Cholesky kernel ran out
// Second CholeskyQR pass: up to kFirstOrderDeviation (largest entry of the first pass's
// G - I) the pass is the first-order correction I - Phi(E), whose O(E^2) remainder then stays
// near the rounding of the measurement itself; above it, up to kMaxGramDeviation, a second
// factorisation of I + E is run for that matrix; beyond that the matrix is flagged.
constexpr float kFirstOrderDeviation = 1.0e-3f;
constexpr float kMaxGramDeviation = 0.5f;
// smallest ratio of diagonal entries of the first pass's triangular factor (about the
// reciprocal condition number of the factor) that still counts as full rank
constexpr float kMinPivotRatio = 1.0e-3f;

// What steps together in shared launches.
struct Work {
  int64_t elements, matrices;
};

// One launch batch as the launchers see it: shape, the caller's buffers, its workspace arrays and
// the choices made when the handle was created.  Choices depend on the whole matrix set (how many
// workgroups share the chip in a launch), never on how the set is dealt into groups.
struct BatchRef {
  ClassDims d;
  const MatEntry* mats;              // device table, first matrix of the batch
  const MatEntry* host_mats;         // the same entries on the host (read while enqueuing)
  float* scal;
  int* info;
  WsArr pa, pb, ra, rb, part, gram, t1[2], t2[2], w, tmp, colsq;     // t1, t2: [0] left, [1] right factor
  HalfArr ph, pht, rh, qh, qht;
  int splits_proj, splits_back, splits_gram[2], slabs;
  bool small;                        // orthogonalised by the stages for ranks up to 32
  bool beside;                       // small, but sharing launches with a larger rank: factored beside it (launch_cholinv)
  Work work;                         // of all batches that step together with it: the same for all of them
  int64_t peers;                     // matrices of this shape that would make up that work, rounded down
  // left (P, rows m) and right (Q, rows n) side of the orthogonalisation
  int rows(int side) const { return side == 0 ? d.m : d.n; }
  WsArr a0(int side) const { return side == 0 ? pa : ra; }
  WsArr a1(int side) const { return side == 0 ? pb : rb; }
};
typedef const BatchRef* const* BatchList;     // a list of batches; always with its length

// First kernel of a step: writes the table of the caller's buffers, clears the matrices' scale words
// [0..7] and flag words; in fast precision also samples sums of squares of B (for its fp16 scale)
// and writes Q as pre-scaled fp16, transposed [r][n].
hipError_t launch_begin(BatchList b, int n, Prec prec, hipStream_t st);

// the tile rows and columns of the projection / back-projection for this shape, and the workgroups
// of its kernel that fit the chip at a time: what the number of splits is chosen from.  `staged`: those of the
// register-staged kernels for ranks below 192, whose smaller workgroups take fewer splits
void proj_tiling(const ClassDims& d, Prec prec, int64_t peers, const Work& work, bool staged, int* rows, int* cols, int* slots);
void back_tiling(const ClassDims& d, Prec prec, const Work& work, bool staged, int* rows, int* cols, int* slots);
// P_raw = (M + G) Q, split over n: partial sums in `part`, or with one split straight in `pa`
hipError_t launch_proj(BatchList b, int n, Prec prec, hipStream_t st);
// pa = sum of the projection's partials (batches with one split have nothing to add)
hipError_t launch_proj_reduce(BatchList b, int n, hipStream_t st);
// R = (M + G)^T P, split over m: partial sums in `part`, or with one split straight in `ra`; with
// one split the direct-to-LDS kernel also writes R as pre-scaled fp16 and checks its range
hipError_t launch_back(BatchList b, int n, Prec prec, hipStream_t st);
// ra = sum of the partials; in fast precision also R as pre-scaled fp16 (rh)
hipError_t launch_back_reduce(BatchList b, int n, Prec prec, hipStream_t st);

// The orthogonalisation of P_raw (side 0) or R (side 1) by CholeskyQR2, in pieces:
// orth_gram: Gram matrix of a0 in the batch's slices of the class array `gram` (small batches: partial sums
// for the second pass)
hipError_t launch_orth_gram(BatchList b, int n, int side, Prec prec, hipStream_t st);
// where the Gram partials of a0 (pass 0) or of a1 (pass 1) of a small batch lie, splits_gram[side] of r x r
WsArr small_partials(const BatchRef& b, int side, int pass);
// second pass: a1 = a0 W1, Gram of a1, T2 = I + Phi(E), Phi^T (fast) or W2 = I - Phi(E) (exact), max |E|;
// small batches: the factorisation of the first pass (unless `beside`), a1 and its Gram partials
hipError_t launch_orth_second(BatchList b, int n, int side, Prec prec, hipStream_t st);
// r <= 256: Cholesky factor of I + E for the matrices whose deviation is above kFirstOrderDeviation
hipError_t launch_orth_guard(BatchList b, int n, int side, hipStream_t st);
// result = a1 - a1 Phi(E) (fast), a1 W2 (exact), for a flagged matrix the full product a1 W2, to a0 or (side 1)
// the callers' Q, with the fp16 copies of fast precision.  `which`: 0 everything, 1 only the
// first-order correction of the well-conditioned matrices, 2 only the full product of the flagged ones.
// small batches: the whole rest of the second pass.
hipError_t launch_orth_result(BatchList b, int n, int side, Prec prec, int which, hipStream_t st);

// Gram partials of a plain array: part[split][r][r] = A^T A over a row range, six-product operands
hipError_t launch_gram_plain(int nb, int rows, int r, WsArr a, WsArr part, int splits, hipStream_t st);
// out[i] = sum_s part[s * count + i], i < count, per matrix
hipError_t launch_reduce(int nb, WsArr part, int splits, int64_t count, WsArr out, hipStream_t st, Pred pred = Pred{nullptr, 0, 0.f, 0});

// Cholesky factor and its inverse of the SPD r x r matrices `gram` (ld r): gram = T^T T,
// W = T^-1, both upper triangular with zeros below the diagonal.  The matrices need not belong
// to one shape class: the work depends on r only, so one call serves every matrix of that
// rank (`nb` of them).  For r <= 256 one workgroup per matrix does everything, and jobs of
// different ranks share a launch; above, the factorisation is blocked, `gram` is destroyed and
// `tmp` is r x r scratch.  A non-positive or non-finite pivot writes its 1-based column to
// info[mat * kInfoPerMat + info_slot] (first failure wins); the factors of such a matrix are
// unspecified (they may hold NaN).  With `splits` > 1 (r <= 256 only) `gram` holds that many partial
// sums per matrix, `split_stride` elements apart, which the factorisation adds up itself.
struct CholJob {
  int nb, r;
  WsArr gram, t, w, tmp;
  int* info;
  int info_slot;
  Pred pred;
  int splits;
  int64_t split_stride;
};
hipError_t launch_cholinv(const CholJob* jobs, int njobs, hipStream_t st);

// ColNorm: Q[:, c] = R[:, c] / ||R[:, c]||; `part` holds slabs x r partial sums per matrix, `colsq` r
// reciprocal lengths per matrix.
hipError_t launch_colnorm(BatchList b, int n, Prec prec, hipStream_t st);

// M_new = a (M+G) - b P R^T ;  X_new = X - lr P Q^T   (one pass over M, G, X)
// A matrix whose info words report a breakdown keeps its X and gets M_new = a (M + G): its
// factors are unspecified and must not reach the caller's state.  Fast precision also checks every
// entry of B against its sampled fp16 scale and sets the warning bits of `info`.
hipError_t launch_efx(BatchList b, int n, Prec prec, float a_coef, float b_coef, float lr, hipStream_t st);

// ---- optional diagnostics (od_diag.hip) ----
constexpr int kDiagPerMat = 8;     // floats reported per matrix
constexpr int kDaccPerMat = 8;     // fp64 accumulators per matrix: [3] ||R||^2, [4] sum of column lengths of R,
                                   // [5] sum of len * log(len), [7] lambda_max
constexpr int kDiagBlocks = 512;   // most workgroups (partial triples of 4 doubles) per matrix of the norm pass

// dpart[mat][blocks][4] = partial sums of squares of M, G, M + G
hipError_t launch_diag_norms(const ClassDims& d, const MatEntry* mats, double* dpart, int blocks, hipStream_t st);
// column lengths of R (n x r, ld r) -> dacc[mat][3..5]; `part` needs slabs * r floats per matrix
hipError_t launch_diag_cols(int nb, int n, int r, WsArr rr, WsArr part, int slabs, double* dacc, hipStream_t st);
// out[mat] = callers' Q (n x r)
hipError_t launch_gather_q(int nb, int n, int r, const MatEntry* mats, WsArr out, hipStream_t st);
// dacc[mat][7] = largest eigenvalue of the symmetric PSD r x r matrix `gram`: Lanczos iteration up to r = 256, power
// iteration with squared powers beyond; tmp1, tmp2: r x r scratch per matrix, xbuf: 2 r floats per matrix (used for r > 512)
hipError_t launch_power(int nb, int r, WsArr gram, WsArr tmp1, WsArr tmp2, WsArr xbuf, double* dacc, hipStream_t st);
// diag[mat][0..7] = ||B||, ||R||, tracking error, ||M_prev|| / ||G||, <B, P Q^T>, nu, effective rank, ||G||;
// <B, P Q^T> is sum_i t1[i][i] t2[i][i] (QR) or the sum of the column lengths of R (colnorm)
hipError_t launch_diag_final(int nb, int r, const double* dpart, int blocks, const double* dacc, WsArr t1, WsArr t2, int colnorm, float* diag, hipStream_t st);
// q_new (n x r_new) = leading min(r_old, r_new) columns of q_old, then columns of pad (n x (r_new - r_old))
hipError_t launch_resize_q(const float* q_old, int64_t n, int r_old, float* q_new, int r_new, const float* pad, hipStream_t st);

// The next launch_proj / launch_back / launch_efx of this thread records the start time stamp of its
// first and the stop time stamp of its last kernel in the two events (one shot).
void time_next_launch(hipEvent_t start, hipEvent_t stop);

}  // namespace od

// Host side of the Orth-Dion C ABI: argument checks, shape classes, workspace planning and
// the kernel sequence of one step.  No device memory is allocated here; everything lives
// in the caller's workspace.
#include "../../include/orthdion.h"

#include <algorithm>
#include <cmath>
#include <memory>
#include <new>
#include <vector>

#include "od_kernels.h"
#include "od_internal.h"

namespace {

using od::BatchRef;
using od::ClassDims;
using od::HalfArr;
using od::MatEntry;
using od::WsArr;

constexpr size_t kAlign = 256;
// Two groups by default between these numbers of matrix elements.  A set below is a chain of
// short launches, where the fork and join of the second stream cost more than the overlap
// returns.  A set above comes in launch batches of many matrices, whose kernels fill the chip
// by themselves: side by side they mostly compete (measured on 96 matrices of rank 512: 2 to 4 %
// less time per step, and no kernel's time stamps mean anything any more), whereas a few matrices
// of large rank gain 13 %: there the Cholesky chains and the one-matrix launches leave room.
constexpr double kGroupMinElements = 64.0 * 1024 * 1024;
constexpr double kGroupMaxElements = 512.0 * 1024 * 1024;

// Matrices of one shape class step in launch batches of at most this many matrices, or more while
// they hold less than kBatchElements: what a batch's kernels leave behind for the next one (partial
// sums, factors) should still be in the Infinity Cache when it is read.  Measured with half and twice the
// elements, us a step: 100 matrices of 1024 x 1024, r = 128: 1101 | 1059 | 1112; 600 matrices of a 512-wide model,
// r = 64: 3396 | 3369 | 3211; the 96 and 126 matrices of a 2048- and a 768-wide one within 1 %.  64 matrices instead
// of 32 are 4 % faster on 144 and 320 matrices of a 1024-wide model, r = 128 (3262 -> 3129, 7551 -> 7229), and
// nothing elsewhere.
constexpr int kBatchMatrices = 32;
constexpr double kBatchElements = 64.0 * 1024 * 1024;
// In any case this many: a batch's matrices are the y or z extent of its launches, where a device takes 65536.
constexpr int kBatchMost = 32768;
constexpr int kLeanDiagBlocks = 128;  // see the two plans of the workspace in create_impl
// Batches of different shapes share their launches (a cluster) up to this many elements: below it
// the launches of one shape leave most of the chip idle, above it every batch fills the chip by itself.
// Measured with half and twice of it, us a step: 126 matrices of a 768-wide model, r = 192: 1806 | 1651 | 1647; 144
// and 320 of a 1024-wide one, r = 128: 3273 | 3277 | 3163 and 7624 | 7574 | 7223; 600 of a 512-wide one, r = 64:
// 3418 | 3358 | 3228; r = 256 and 512 of a 2048-wide one within 1 %.  So half is too little; twice is 3 to 4 %
// better for sets of many small matrices.
constexpr double kClusterElements = 128.0 * 1024 * 1024;

size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

// A batch: matrices of identical shape and leading dimensions.
struct Batch {
  ClassDims d;
  std::vector<int> members;          // indices into the caller's arrays
  // per-matrix float arrays (offset of matrix 0 in bytes, stride in elements)
  size_t off_pa, off_pb, off_ra, off_rb, off_part, off_gram, off_tp1, off_tp2, off_tq1, off_tq2, off_w,
      off_tmp, off_colsq;
  size_t off_ph, off_pht, off_rh, off_qh, off_qht;   // pre-scaled fp16 copies of the factors (uint16 arrays)
  size_t off_dpart;                  // diagnostics: partial norms, diag_blocks times 4 doubles per matrix
  int diag_blocks;
  int alike;                         // matrices of this shape in the whole set
  int64_t st_p, st_r, st_part, st_rr, st_colsq;
  int splits_proj, splits_back, splits_gram[2], slabs;
  int slot_base;                     // first row of this batch in the scal / info tables
  int rank_class;
  int cluster;                       // batches of one cluster share their launches
  bool small;                        // orthogonalisation by the three stages for ranks up to 32
  bool beside;                       // small, in a cluster that holds a larger rank
  od::Work work;                     // of the cluster (its batches in the same group)
  int64_t peers;                     // matrices of this shape that make up the same work, rounded down
};

// All batches of one rank r.  The r x r work of the orthogonalisations (Cholesky factor and
// inverse) does not depend on m and n, so it is launched once per rank class over all of its
// matrices: the class owns the r x r arrays, every batch a contiguous range of slices.
struct RankClass {
  int r, count, slot_base;
  bool small;                        // see Batch
  int group;                         // which of the two groups a large set of one rank is dealt into
  int64_t st_rr;
  std::vector<int> batches;
  size_t off_gram, off_tp1, off_tp2, off_tq1, off_tq2, off_w, off_tmp;
};

// What runs in lockstep: the rank classes up to 256 of a group together, a larger rank by itself.
// Its batches are enqueued cluster by cluster, piece by piece.
struct Unit {
  int group;
  bool wide_guard;                   // ranks above 256: the class-wide guard of the second pass
  std::vector<int> classes;
  std::vector<std::vector<int>> clusters;   // batches that share launches
};

int pick_splits(int64_t tiles, int64_t nb, int64_t k, int kt_min) {
  int64_t want = (512 + tiles * nb - 1) / (tiles * nb);
  int64_t cap = k / kt_min;
  if (cap < 1) cap = 1;
  if (want > cap) want = cap;
  if (want > 32) want = 32;
  if (want < 1) want = 1;
  return (int)want;
}

// Splits for a kernel whose workgroups run in rounds of `slots` (256 CUs times the workgroups
// that fit one CU).  A workgroup's time is proportional to 1 / splits, so rounds / splits
// measures the launch; the fewest splits (least partial-sum traffic) within 15 % of the best
// are taken; a single one, which leaves no partial sums, also within `single` of it.
int pick_splits_by_rounds(int64_t tiles, int64_t nb, int64_t k, int kt_min, int64_t slots, double single = 1.15) {
  int64_t cap = k / kt_min;
  if (cap < 1) cap = 1;
  if (cap > 32) cap = 32;
  auto cost = [&](int s) { return (double)((tiles * nb * s + slots - 1) / slots) / (double)s; };
  double best = cost(1);
  for (int s = 2; s <= (int)cap; ++s) best = cost(s) < best ? cost(s) : best;
  for (int s = 1; s <= (int)cap; ++s)
    if (cost(s) <= (s == 1 ? single : 1.15) * best) return s;
  return 1;
}

}  // namespace

struct orthdion_ctx {
  std::vector<orthdion_matdesc> mats;
  orthdion_config cfg;
  std::vector<Batch> batches;
  std::vector<RankClass> classes;
  std::vector<Unit> units;
  std::vector<int> batch_of, slot_of;     // per matrix
  size_t off_mats, off_scal, off_info, off_diag, off_dacc, ws_bytes;
  void* last_ws;
  bool diag_on = false, diag_valid = false;
  // optional phase timing with HIP events (host resources only)
  bool prof_on = false;
  unsigned prof_mask = 0;
  int prof_max_steps = 0, prof_steps = 0;
  std::vector<hipEvent_t> prof_events;    // [step][batch][phase][begin/end]
  std::vector<int> prof_recorded;         // [step][batch][phase]: batches the recorded interval covers, 0 = none
  // a second stream for the guard of the second CholeskyQR pass (ranks above 256): its launch
  // chain returns at once for every well-conditioned matrix, and beside the main stream those
  // empty launches cost nothing (host resources; made at the first step that is not being captured)
  hipStream_t side = nullptr;
  hipEvent_t ev_fork = nullptr, ev_join = nullptr;
  bool side_tried = false;
  // Two groups: the batches are dealt to two sets of about equal work, each with rank classes
  // of its own, and the two sets run side by side on the caller's stream and on `group_stream`
  // (see orthdion_step_impl).
  bool two_groups = false;
  hipStream_t group_stream = nullptr;
  hipEvent_t ev_group_fork = nullptr, ev_group_join = nullptr;
};

static bool ensure_side_stream(orthdion_ctx* h, hipStream_t st) {
  if (h->side) return true;
  if (h->side_tried) return false;
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &cs) != hipSuccess) { (void)hipGetLastError(); return false; }
  if (cs != hipStreamCaptureStatusNone) return false;        // nothing is created under capture; a later call may
  h->side_tried = true;
  if (hipStreamCreateWithFlags(&h->side, hipStreamNonBlocking) != hipSuccess) { h->side = nullptr; (void)hipGetLastError(); return false; }
  bool ok = hipStreamCreateWithFlags(&h->group_stream, hipStreamNonBlocking) == hipSuccess;
  if (!ok) h->group_stream = nullptr;
  hipEvent_t* const events[4] = {&h->ev_fork, &h->ev_join, &h->ev_group_fork, &h->ev_group_join};
  for (hipEvent_t* e : events) ok = ok && hipEventCreateWithFlags(e, hipEventDisableTiming) == hipSuccess;
  if (!ok) {
    for (hipEvent_t* e : events) {
      if (*e) (void)hipEventDestroy(*e);
      *e = nullptr;
    }
    if (h->group_stream) (void)hipStreamDestroy(h->group_stream);
    (void)hipStreamDestroy(h->side);
    h->side = nullptr; h->group_stream = nullptr;
    (void)hipGetLastError();
    return false;
  }
  return true;
}

static hipEvent_t* prof_slot(orthdion_ctx* h, int batch, int phase, int end, int covers) {
  if (!h->prof_on || h->prof_steps >= h->prof_max_steps || !(h->prof_mask & (1u << phase))) return nullptr;
  size_t nb = h->batches.size();
  size_t idx = (((size_t)h->prof_steps * nb + (size_t)batch) * ORTHDION_NPHASE + (size_t)phase) * 2 + (size_t)end;
  if (end) h->prof_recorded[idx / 2] = covers;
  return &h->prof_events[idx];
}

static od::Prec resolve_prec(const orthdion_config& c) {
  if (c.precision == ORTHDION_PREC_FAST) return od::PREC_F16;
  if (c.precision == ORTHDION_PREC_EXACT) return od::PREC_BF3;
  return (c.x_dtype == ORTHDION_BF16 && c.g_dtype == ORTHDION_BF16) ? od::PREC_F16 : od::PREC_BF3;
}

static int check_config(const orthdion_config* c) {
  if (c->x_dtype != ORTHDION_F32 && c->x_dtype != ORTHDION_BF16) return ORTHDION_E_INVALID_ARG;
  if (c->g_dtype != ORTHDION_F32 && c->g_dtype != ORTHDION_BF16) return ORTHDION_E_INVALID_ARG;
  if (c->variant != ORTHDION_QR && c->variant != ORTHDION_COLNORM) return ORTHDION_E_INVALID_ARG;
  if (c->ef != ORTHDION_EF_DION && c->ef != ORTHDION_EF_PAPER && c->ef != ORTHDION_EF_POLYAK) return ORTHDION_E_INVALID_ARG;
  if (c->precision != ORTHDION_PREC_AUTO && c->precision != ORTHDION_PREC_FAST && c->precision != ORTHDION_PREC_EXACT)
    return ORTHDION_E_INVALID_ARG;
  if (!std::isfinite(c->mu) || c->mu < 0.f || c->mu > 1.f) return ORTHDION_E_INVALID_ARG;
  if (!std::isfinite(c->lr)) return ORTHDION_E_INVALID_ARG;
  if (c->groups < 0 || c->groups > 2) return ORTHDION_E_INVALID_ARG;
  return ORTHDION_OK;
}

static int check_shape(const orthdion_matdesc& m) {
  if (m.m < 8 || m.n < 8 || m.r < 8) return ORTHDION_E_BAD_SHAPE;
  if (m.m % 8 || m.n % 8 || m.r % 8) return ORTHDION_E_BAD_SHAPE;
  if (m.m >= (1 << 24) || m.n >= (1 << 24)) return ORTHDION_E_BAD_SHAPE;
  if (m.r > m.m || m.r > m.n) return ORTHDION_E_BAD_SHAPE;
  if (m.ldx < m.n || m.ldg < m.n || m.ldm < m.n) return ORTHDION_E_BAD_SHAPE;
  if (m.ldx % 8 || m.ldg % 8 || m.ldm % 8) return ORTHDION_E_BAD_SHAPE;
  return ORTHDION_OK;
}

// Nothing may throw across the C boundary: the entry points that allocate host memory run their
// bodies through this.
template <class F>
static int no_throw(F&& body) {
  try {
    return body();
  } catch (const std::bad_alloc&) {
    return ORTHDION_E_NO_MEMORY;
  } catch (...) {
    return ORTHDION_E_INVALID_ARG;
  }
}

static int create_impl(orthdion_handle* out, const orthdion_matdesc* mats, int32_t nmat, const orthdion_config* cfg);

extern "C" int orthdion_create(orthdion_handle* out, const orthdion_matdesc* mats, int32_t nmat,
                               const orthdion_config* cfg) {
  if (!out) return ORTHDION_E_NULL_PTR;
  *out = nullptr;
  orthdion_handle h = nullptr;
  const int rc = no_throw([&] { return create_impl(&h, mats, nmat, cfg); });
  if (rc != ORTHDION_OK) {
    delete h;
    return rc;
  }
  *out = h;
  return ORTHDION_OK;
}

static int create_impl(orthdion_handle* out, const orthdion_matdesc* mats, int32_t nmat, const orthdion_config* cfg) {
  if (!mats || !cfg) return ORTHDION_E_NULL_PTR;
  if (nmat < 1 || nmat > (1 << 20)) return ORTHDION_E_INVALID_ARG;
  int rc = check_config(cfg);
  if (rc != ORTHDION_OK) return rc;
  for (int i = 0; i < nmat; ++i)
    if ((rc = check_shape(mats[i])) != ORTHDION_OK) return rc;

  orthdion_ctx* h = new (std::nothrow) orthdion_ctx();
  if (!h) return ORTHDION_E_NO_MEMORY;
  *out = h;                        // the caller frees it if anything below fails or throws
  h->mats.assign(mats, mats + nmat);
  h->cfg = *cfg;
  h->last_ws = nullptr;
  h->batch_of.assign(nmat, -1);
  h->slot_of.assign(nmat, -1);

  // shape classes, in order of first appearance, cut into batches
  auto same_shape = [](const ClassDims& d, const orthdion_matdesc& a) {
    return d.m == a.m && d.n == a.n && d.r == a.r && d.ldx == a.ldx && d.ldg == a.ldg && d.ldm == a.ldm;
  };
  double total_elems = 0.0;
  for (int i = 0; i < nmat; ++i) total_elems += (double)mats[i].m * (double)mats[i].n;
  const int by_default = nmat >= 2 && total_elems >= kGroupMinElements && total_elems < kGroupMaxElements ? 2 : 1;
  const int groups = cfg->groups == 0 ? by_default : cfg->groups;
  for (int i = 0; i < nmat; ++i) {
    const orthdion_matdesc& a = mats[i];
    int found = -1;
    for (size_t b = 0; b < h->batches.size(); ++b) {
      const double held = (double)h->batches[b].members.size();
      if (held < kBatchMost && same_shape(h->batches[b].d, a) && (held < kBatchMatrices || (held + 1) * (double)a.m * (double)a.n <= kBatchElements)) found = (int)b;
    }
    if (found < 0) {
      Batch nb = {};
      nb.d.m = (int)a.m; nb.d.n = (int)a.n; nb.d.r = a.r;
      nb.d.ldx = a.ldx; nb.d.ldg = a.ldg; nb.d.ldm = a.ldm;
      nb.d.x_bf16 = cfg->x_dtype == ORTHDION_BF16;
      nb.d.g_bf16 = cfg->g_dtype == ORTHDION_BF16;
      h->batches.push_back(nb);
      found = (int)h->batches.size() - 1;
    }
    h->batch_of[i] = found;
    h->slot_of[i] = (int)h->batches[found].members.size();
    h->batches[found].members.push_back(i);
  }

  for (Batch& b : h->batches) {
    b.alike = 0;
    for (const Batch& o : h->batches)
      if (same_shape(o.d, h->mats[b.members[0]])) b.alike += (int)o.members.size();
  }

  // Two groups: the heaviest batch first, each to the group with less work so far (m n per matrix
  // measures a batch's step).  A set with a single batch stays one group.
  for (Batch& b : h->batches) b.d.nb = (int)b.members.size();
  std::vector<int> dealt(h->batches.size(), 0);
  {
    std::vector<int> order(h->batches.size());
    for (size_t k = 0; k < order.size(); ++k) order[k] = (int)k;
    auto weight = [&](int k) { const ClassDims& d = h->batches[k].d; return (double)d.m * d.n * d.nb; };
    std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return weight(x) > weight(y); });
    double load[2] = {0.0, 0.0};
    for (int k : order) {
      dealt[k] = load[1] < load[0] ? 1 : 0;
      load[dealt[k]] += weight(k);
    }
  }

  // Clusters, in batch order: the ranks up to 256 together, every larger rank by itself.  They do not
  // depend on the groups below (nor does anything chosen from them), so that the groups leave the
  // results alone bit for bit.
  {
    struct Open { int key, id; double elems; };
    std::vector<Open> open;
    const auto side_of = [&](const Batch& b) { return by_default == 2 ? dealt[&b - h->batches.data()] : 0; };
    std::vector<od::Work> shared[2];    // of a cluster's batches in either group
    for (Batch& b : h->batches) {
      const int key = b.d.r <= od::kLeafRank ? 0 : b.d.r;
      const double e = (double)b.d.m * b.d.n * (double)b.members.size();
      size_t k = 0;
      while (k < open.size() && open[k].key != key) ++k;
      if (k == open.size()) open.push_back(Open{key, -1, 0.0});
      if (open[k].id < 0 || open[k].elems + e > kClusterElements) {
        open[k].id = (int)shared[0].size();
        open[k].elems = 0.0;
        shared[0].push_back(od::Work{0, 0});
        shared[1].push_back(od::Work{0, 0});
      }
      open[k].elems += e;
      b.cluster = open[k].id;
      od::Work& w = shared[side_of(b)][b.cluster];
      w.elements += (int64_t)e;
      w.matrices += (int64_t)b.members.size();
    }
    for (Batch& b : h->batches) {
      // Where the library takes two groups, a batch shares its launches and its stream with those of its group
      // only (the other group's run beside them): chosen for all batches of the cluster, the splits halved and one
      // matrix of 8192 columns lost its rotated k order (8192 x 8192, r = 256 and 32: 938 us a step with launches
      // of their own, 1030 so, 941 like this).  By the default, not by the groups of this handle: see above.
      b.work = shared[side_of(b)][b.cluster];
      b.peers = b.work.elements / ((int64_t)b.d.m * b.d.n);
    }
    // Ranks up to 32 have three stages of their own per orthogonalisation instead of eight kernels (one matrix of
    // 8192 x 8192, r = 16: 376 -> 352 us), in fp32, whatever larger ranks share their launches.
    for (Batch& b : h->batches) b.small = b.d.r <= 32;
  }

  // workspace plan
  size_t off = 0;
  h->off_mats = off; off = align_up(off + (size_t)nmat * sizeof(MatEntry));
  h->off_scal = off; off = align_up(off + (size_t)nmat * od::kScalPerMat * sizeof(float));
  h->off_info = off; off = align_up(off + (size_t)nmat * od::kInfoPerMat * sizeof(int));
  h->off_diag = off; off = align_up(off + (size_t)nmat * od::kDiagPerMat * sizeof(float));
  h->off_dacc = off; off = align_up(off + (size_t)nmat * od::kDaccPerMat * sizeof(double));
  std::vector<int> group_of(h->batches.size(), 0);
  if (groups == 2 && h->batches.size() >= 2) {
    group_of = dealt;
    h->two_groups = true;
  }
  // rank classes in order of first appearance (one per rank and group); table rows (slots) run
  // class by class
  for (size_t bi = 0; bi < h->batches.size(); ++bi) {
    Batch& b = h->batches[bi];
    int found = -1;
    for (size_t c = 0; c < h->classes.size(); ++c)
      if (h->classes[c].r == b.d.r && h->classes[c].group == group_of[bi]) found = (int)c;
    if (found < 0) {
      RankClass rc = {};
      rc.r = b.d.r;
      rc.small = b.small;
      rc.group = group_of[bi];
      rc.st_rr = ((int64_t)b.d.r * b.d.r + 63) / 64 * 64;
      h->classes.push_back(rc);
      found = (int)h->classes.size() - 1;
    }
    b.rank_class = found;
    h->classes[found].batches.push_back((int)bi);
    h->classes[found].count += b.d.nb;
  }
  // units: what steps in lockstep
  for (size_t ci = 0; ci < h->classes.size(); ++ci) {
    const RankClass& c = h->classes[ci];
    const bool wide = c.r > od::kLeafRank;
    int found = -1;
    for (size_t u = 0; u < h->units.size() && !wide; ++u)
      if (h->units[u].group == c.group && !h->units[u].wide_guard) found = (int)u;
    if (found < 0) {
      Unit u = {};
      u.group = c.group;
      u.wide_guard = wide;
      h->units.push_back(u);
      found = (int)h->units.size() - 1;
    }
    h->units[found].classes.push_back((int)ci);
  }
  for (size_t bi = 0; bi < h->batches.size(); ++bi) {
    Batch& b = h->batches[bi];
    for (Unit& u : h->units) {
      bool mine = false;
      for (int c : u.classes) mine = mine || c == b.rank_class;
      if (!mine) continue;
      size_t k = 0;
      while (k < u.clusters.size() && h->batches[u.clusters[k][0]].cluster != b.cluster) ++k;
      if (k == u.clusters.size()) u.clusters.push_back({});
      u.clusters[k].push_back((int)bi);
    }
  }
  // Beside a larger rank the factorisation of a small one joins that rank's instead of its own first pass, which
  // is then no longer than the product of the larger rank that it shares a launch with (five small matrices of
  // ranks 24 to 72: 213 -> 208 us a step).  The arithmetic is the same, so the groups may decide this.
  for (const Unit& u : h->units)
    for (const auto& cluster : u.clusters) {
      int widest = 0;
      for (int bi : cluster) widest = std::max(widest, h->batches[bi].d.r);
      for (int bi : cluster) h->batches[bi].beside = h->batches[bi].small && widest > 32;
    }
  int slot_base = 0;
  for (RankClass& c : h->classes) {
    c.slot_base = slot_base;
    for (int bi : c.batches) {
      h->batches[bi].slot_base = slot_base;
      slot_base += h->batches[bi].d.nb;
    }
    auto take_rr = [&]() { size_t o = off; off = align_up(off + (size_t)c.st_rr * c.count * sizeof(float)); return o; };
    c.off_gram = take_rr(); c.off_tp1 = take_rr(); c.off_tp2 = take_rr(); c.off_tq1 = take_rr(); c.off_tq2 = take_rr();
    c.off_w = take_rr(); c.off_tmp = take_rr();
  }
  // The arrays of the batches.  Batches that share their launches now and then take more splits than they
  // would alone (rounds do not divide evenly), up to 30 % more workspace.  Where that would take a set out of
  // reach of orthdion_step_static, the plan without it is used, if it fits.
  const size_t arrays = off;
  auto plan = [&](bool lean) {
    off = arrays;
    for (Batch& b : h->batches) {
      ClassDims& d = b.d;
      const RankClass& rcl = h->classes[b.rank_class];
      const int64_t m = d.m, n = d.n, r = d.r;
      const od::Prec prec = resolve_prec(*cfg);
      auto splits_of = [&](bool back, int64_t peers, bool staged) {
        int rows, cols, slots;
        if (back) od::back_tiling(d, prec, b.work, staged, &rows, &cols, &slots);
        else od::proj_tiling(d, prec, peers, b.work, staged, &rows, &cols, &slots);
        const int64_t out = back ? n : m, k = back ? m : n;
        const int64_t tiles = ((out + rows - 1) / rows) * ((r + cols - 1) / cols);
        // One 8-wave workgroup per CU is scheduled in whole rounds; two smaller ones mix.  Below r = 192 (columns of one tile,
        // little arithmetic) partial sums are a larger part of the traffic, and more than one split has to save a third of
        // the rounds (us a step by the rule of the larger ranks | by this one, with the register-staged kernels: 160 matrices
        // 512 x 512 of r = 128 687 | 625, 672; 134 of r = 72 518 | 487, 501; 66 of r = 160 457 | 435, 500; 18 of
        // 2048 x 2048, r = 160, 805 | 806, 912)
        return slots == 256 ? pick_splits_by_rounds(tiles, peers, k, 256, slots, r < 192 ? 1.45 : 1.15) : pick_splits(tiles, peers, k, 128);
      };
      // the lean plan takes no more splits than the register-staged kernels would
      auto splits_for = [&](bool back, int64_t peers) {
        const int s = splits_of(back, peers, false);
        return lean ? std::min(s, splits_of(back, peers, true)) : s;
      };
      // `lean`: no more splits than in launches of the batch's own, at most kBatchMatrices matrices each
      auto limited = [&](auto&& pick) {
        int s = pick(b.peers);
        // exact precision: sums no longer than in launches of the batch's own (each split is summed in fp32 by itself)
        if (prec == od::PREC_BF3) s = std::max(s, (int)pick(std::min<int64_t>(d.nb, kBatchMatrices)));
        if (lean)
          for (int64_t alone : {std::min(b.alike, kBatchMatrices), b.alike % kBatchMatrices})
            if (alone > 0) s = std::min(s, (int)pick(alone));
        return s;
      };
      b.splits_proj = limited([&](int64_t peers) { return splits_for(false, peers); });
      b.splits_back = limited([&](int64_t peers) { return splits_for(true, peers); });
      // Gram tiles on and above the diagonal (the ones that are computed)
      const int64_t gt1 = (r + 127) / 128;
      const int64_t gt = gt1 * (gt1 + 1) / 2;
      for (int side = 0; side < 2; ++side) {
        const int64_t rows = side == 0 ? m : n;
        // small ranks: one 32 x 32 tile, one thread per row: 256-row slabs (small_gram, small_first_pass);
        // else two workgroups of the Gram kernel fit one CU.  Where that leaves few tiles, the kernel takes 64 x 64
        // ones (gram_pass), and their short loops are split further, down to 128 rows, as long as one workgroup per CU
        // has room (4096 x 4096, r = 256, 14 | 25 splits: 312 | 307 us a step, 2048 x 5632 291 | 287, five small matrices
        // of ranks 24 to 72 210 | 200; without that bound 64 matrices 640 x 640 of r = 72 took 392 instead of 375); never
        // fewer: six ragged ones of r = 136 took 444 instead of 436.  Two splits in place of one, i.e. a launch more that adds
        // them up, pay up to some 50 matrices (48 of 320 x 320, r = 40: one 160, two 157; 64: 179, 184; 128 of 264 x 264:
        // 290, 294), in exact precision, whose loops take longer, as long as there is room (64 and 100 of 256 x 256, r = 40:
        // one 172 and 237, two 164 and 228).
        const int s = limited([&](int64_t peers) { return b.small ? pick_splits(1, peers, rows, 256) : pick_splits_by_rounds(gt, peers, rows, 256, 512); });
        b.splits_gram[side] = s;
        if (b.small || lean) continue;
        // By what steps together, also in exact precision: 32 matrices alone, which its least splits are taken from, leave
        // CUs idle that many do not (fp32, with finer splits for the former | so: 300 matrices 256 x 256 of r = 40 585 | 513,
        // 500 of 384 x 384 1560 | 1382, 1000 of 256 x 256, r = 96, 2060 | 1960).
        const int64_t g64 = (r + 63) / 64, tiles = g64 * (g64 + 1) / 2;
        const int64_t idle = 256 / (tiles * b.peers);       // splits that one workgroup per CU has room for
        const int fine = (int)std::max<int64_t>(s, std::min<int64_t>(idle, pick_splits_by_rounds(tiles, b.peers, rows, 128, 256)));
        if (gt1 * gt1 * fine * b.peers < od::kSmallGramTiles && (s > 1 || fine > 2 || b.peers < 64 || prec == od::PREC_BF3)) b.splits_gram[side] = fine;
      }
      b.slabs = (int)((n + 31) / 32);           // row slabs of the column-norm kernels: many, so the grid fills the chip
      if (b.slabs > 256) b.slabs = 256;
      int64_t part = (int64_t)b.splits_proj * m * r;
      if ((int64_t)b.splits_back * n * r > part) part = (int64_t)b.splits_back * n * r;
      for (int sg : b.splits_gram)
        if ((int64_t)sg * r * r > part) part = (int64_t)sg * r * r;
      if ((int64_t)b.slabs * r > part) part = (int64_t)b.slabs * r;
      // strides rounded so that every matrix slice stays 256-byte aligned
      auto rnd = [](int64_t e) { return (e + 63) / 64 * 64; };
      b.st_p = rnd(m * r); b.st_r = rnd(n * r); b.st_part = rnd(part); b.st_rr = rnd(r * r); b.st_colsq = rnd(r);
      auto take = [&](int64_t stride) { size_t o = off; off = align_up(off + (size_t)stride * d.nb * sizeof(float)); return o; };
      b.off_pa = take(b.st_p); b.off_pb = take(b.st_p);
      b.off_ra = take(b.st_r); b.off_rb = take(b.st_r);
      b.off_part = take(b.st_part);
      // this batch's slices of the class-owned r x r arrays
      const size_t in_class = (size_t)(b.slot_base - rcl.slot_base) * (size_t)rcl.st_rr * sizeof(float);
      b.off_gram = rcl.off_gram + in_class;
      b.off_tp1 = rcl.off_tp1 + in_class; b.off_tp2 = rcl.off_tp2 + in_class;
      b.off_tq1 = rcl.off_tq1 + in_class; b.off_tq2 = rcl.off_tq2 + in_class;
      b.off_w = rcl.off_w + in_class; b.off_tmp = rcl.off_tmp + in_class;
      b.off_colsq = take(b.st_colsq);
      auto take_h = [&](int64_t stride) { size_t o = off; off = align_up(off + (size_t)stride * d.nb * sizeof(uint16_t)); return o; };
      b.off_ph = take_h(b.st_p); b.off_pht = take_h(b.st_p);
      b.off_rh = take_h(b.st_r); b.off_qh = take_h(b.st_r); b.off_qht = take_h(b.st_r);
      // one workgroup per four rows (k_diag_norms): the table stays small beside a small matrix
      b.diag_blocks = (int)std::min<int64_t>(lean ? kLeanDiagBlocks : od::kDiagBlocks, (m + 3) / 4);
      b.off_dpart = off; off = align_up(off + (size_t)d.nb * b.diag_blocks * 4 * sizeof(double));
    }
    return off;
  };
  if (plan(false) > ORTHDION_STATIC_SCRATCH_BYTES && plan(true) > ORTHDION_STATIC_SCRATCH_BYTES) plan(false);
  h->ws_bytes = off;
  return ORTHDION_OK;
}

extern "C" size_t orthdion_workspace_bytes(orthdion_handle h) { return h ? h->ws_bytes : 0; }

extern "C" int32_t orthdion_get_groups(orthdion_handle h) { return h ? (h->two_groups ? 2 : 1) : 0; }

extern "C" int orthdion_set_lr(orthdion_handle h, float lr) {
  if (!h) return ORTHDION_E_NULL_PTR;
  if (!std::isfinite(lr)) return ORTHDION_E_INVALID_ARG;
  h->cfg.lr = lr;
  return ORTHDION_OK;
}

extern "C" int orthdion_set_mu(orthdion_handle h, float mu) {
  if (!h) return ORTHDION_E_NULL_PTR;
  if (!std::isfinite(mu) || mu < 0.f || mu > 1.f) return ORTHDION_E_INVALID_ARG;
  h->cfg.mu = mu;
  return ORTHDION_OK;
}

extern "C" int orthdion_set_variant(orthdion_handle h, orthdion_variant v) {
  if (!h) return ORTHDION_E_NULL_PTR;
  if (v != ORTHDION_QR && v != ORTHDION_COLNORM) return ORTHDION_E_INVALID_ARG;
  h->cfg.variant = v;
  return ORTHDION_OK;
}

#define OD_TRY(expr)                                  \
  do {                                                \
    if ((expr) != hipSuccess) return ORTHDION_E_HIP;  \
  } while (0)

// orth() by CholeskyQR2 comes in pieces (od_kernels.h), so that the r x r stages in its middle, which
// do not depend on the number of rows, can be launched once for every matrix of a rank.

// Cholesky factor and inverse of the first pass for every matrix of a unit; side 0: left factor.
// (Small ranks by themselves factor inside their first pass.)
static int unit_cholinv(const orthdion_ctx* h, const Unit& u, const BatchRef* refs, char* ws, int side, int* info_all, hipStream_t st) {
  od::CholJob jobs[8];
  int n = 0;
  auto add = [&](const od::CholJob& j) -> hipError_t {
    jobs[n++] = j;
    if (n < 8) return hipSuccess;
    n = 0;
    return od::launch_cholinv(jobs, 8, st);
  };
  for (int ci : u.classes) {
    const RankClass& c = h->classes[ci];
    if (c.small) continue;
    od::CholJob j = {};
    j.nb = c.count;
    j.r = c.r;
    j.gram = WsArr{reinterpret_cast<float*>(ws + c.off_gram), c.st_rr};
    j.t = WsArr{reinterpret_cast<float*>(ws + (side == 0 ? c.off_tp1 : c.off_tq1)), c.st_rr};
    j.w = WsArr{reinterpret_cast<float*>(ws + c.off_w), c.st_rr};
    j.tmp = WsArr{reinterpret_cast<float*>(ws + c.off_tmp), c.st_rr};
    j.info = info_all + (size_t)c.slot_base * od::kInfoPerMat;
    j.info_slot = side;
    j.splits = 1;
    OD_TRY(add(j));
  }
  for (const auto& cluster : u.clusters)
    for (int bi : cluster) {
      const BatchRef& b = refs[bi];
      if (!b.beside) continue;
      od::CholJob j = {};
      j.nb = b.d.nb;
      j.r = b.d.r;
      j.gram = od::small_partials(b, side, 0);
      j.t = b.t1[side];
      j.w = b.w;
      j.tmp = b.tmp;
      j.info = b.info;
      j.info_slot = side;
      j.splits = b.splits_gram[side];
      j.split_stride = (int64_t)b.d.r * b.d.r;
      OD_TRY(add(j));
    }
  OD_TRY(od::launch_cholinv(jobs, n, st));
  return ORTHDION_OK;
}

// The guard of the second pass for a class of rank above 256: Cholesky factor and inverse of I + E for
// the matrices whose first pass left a deviation too large for the first-order form (T2 and W2 are
// overwritten); every launch returns at once for the others.
static int class_guard(const RankClass& c, char* ws, int side, float* scal_all, int* info_all, hipStream_t st) {
  od::CholJob j = {};
  j.nb = c.count;
  j.r = c.r;
  j.gram = WsArr{reinterpret_cast<float*>(ws + c.off_gram), c.st_rr};
  j.t = WsArr{reinterpret_cast<float*>(ws + (side == 0 ? c.off_tp2 : c.off_tq2)), c.st_rr};
  j.w = WsArr{reinterpret_cast<float*>(ws + c.off_w), c.st_rr};
  j.tmp = WsArr{reinterpret_cast<float*>(ws + c.off_tmp), c.st_rr};
  j.info = info_all + (size_t)c.slot_base * od::kInfoPerMat;
  j.info_slot = side;
  j.splits = 1;
  j.pred = od::Pred{scal_all + (size_t)c.slot_base * od::kScalPerMat, 2 + side, od::kFirstOrderDeviation, 1};
  OD_TRY(od::launch_cholinv(&j, 1, st));
  return ORTHDION_OK;
}

extern "C" int orthdion_step(orthdion_handle h, void* const* X, const void* const* G, float* const* M,
                             float* const* Q, void* workspace, size_t workspace_bytes, void* stream) {
  return orthdion_step_impl(h, X, G, M, Q, workspace, workspace_bytes, stream, 1);
}

extern "C" int orthdion_step_impl(orthdion_handle h, void* const* X, const void* const* G, float* const* M, float* const* Q,
                                  void* workspace, size_t workspace_bytes, void* stream, int allow_second_stream) {
  if (!h || !X || !G || !M || !Q || !workspace) return ORTHDION_E_NULL_PTR;
  if (workspace_bytes < h->ws_bytes) return ORTHDION_E_WORKSPACE_TOO_SMALL;
  if (reinterpret_cast<uintptr_t>(workspace) % kAlign) return ORTHDION_E_MISALIGNED;
  const int nmat = (int)h->mats.size();
  for (int i = 0; i < nmat; ++i) {
    if (!X[i] || !G[i] || !M[i] || !Q[i]) return ORTHDION_E_NULL_PTR;
    if (reinterpret_cast<uintptr_t>(X[i]) % 16 || reinterpret_cast<uintptr_t>(G[i]) % 16 ||
        reinterpret_cast<uintptr_t>(M[i]) % 16 || reinterpret_cast<uintptr_t>(Q[i]) % 16)
      return ORTHDION_E_MISALIGNED;
  }
  const hipStream_t caller_st = reinterpret_cast<hipStream_t>(stream);
  char* ws = reinterpret_cast<char*>(workspace);
  // Launch errors are read back with hipGetLastError; drop whatever an earlier, unrelated
  // HIP call of this thread left there (e.g. a not-ready event query of the caller).
  (void)hipGetLastError();
  const od::Prec prec = resolve_prec(h->cfg);
  float a_coef, b_coef;
  if (h->cfg.ef == ORTHDION_EF_DION) { a_coef = 1.f; b_coef = 1.f - h->cfg.mu; }
  else if (h->cfg.ef == ORTHDION_EF_PAPER) { a_coef = h->cfg.mu; b_coef = h->cfg.mu; }
  else { a_coef = h->cfg.mu; b_coef = 0.f; }

  int* info_all = reinterpret_cast<int*>(ws + h->off_info);
  float* scal_all = reinterpret_cast<float*>(ws + h->off_scal);
  h->last_ws = workspace;
  const bool diag = h->diag_on;
  h->diag_valid = diag;
  float* diag_all = reinterpret_cast<float*>(ws + h->off_diag);
  double* dacc_all = reinterpret_cast<double*>(ws + h->off_dacc);
  const bool fast = prec == od::PREC_F16;

  // the caller's buffers in slot order, and every batch with its workspace arrays
  const std::unique_ptr<MatEntry[]> entries(new (std::nothrow) MatEntry[nmat]);
  const std::unique_ptr<BatchRef[]> refs(new (std::nothrow) BatchRef[h->batches.size()]);
  const std::unique_ptr<const BatchRef*[]> list(new (std::nothrow) const BatchRef*[h->batches.size()]);
  if (!entries || !refs || !list) return ORTHDION_E_NO_MEMORY;
  for (size_t bi = 0; bi < h->batches.size(); ++bi) {
    const Batch& b = h->batches[bi];
    for (int s = 0; s < b.d.nb; ++s) {
      const int i = b.members[s];
      entries[b.slot_base + s] = MatEntry{X[i], G[i], M[i], Q[i]};
    }
    auto f32 = [&](size_t off, int64_t stride) { return WsArr{reinterpret_cast<float*>(ws + off), stride}; };
    auto f16 = [&](size_t off, int64_t stride) { return HalfArr{reinterpret_cast<uint16_t*>(ws + off), stride}; };
    BatchRef& v = refs[bi];
    v.d = b.d;
    v.mats = reinterpret_cast<const MatEntry*>(ws + h->off_mats) + b.slot_base;
    v.host_mats = entries.get() + b.slot_base;
    v.scal = scal_all + (size_t)b.slot_base * od::kScalPerMat;
    v.info = info_all + (size_t)b.slot_base * od::kInfoPerMat;
    v.pa = f32(b.off_pa, b.st_p); v.pb = f32(b.off_pb, b.st_p);
    v.ra = f32(b.off_ra, b.st_r); v.rb = f32(b.off_rb, b.st_r);
    v.part = f32(b.off_part, b.st_part); v.gram = f32(b.off_gram, b.st_rr);
    v.t1[0] = f32(b.off_tp1, b.st_rr); v.t1[1] = f32(b.off_tq1, b.st_rr);
    v.t2[0] = f32(b.off_tp2, b.st_rr); v.t2[1] = f32(b.off_tq2, b.st_rr);
    v.w = f32(b.off_w, b.st_rr); v.tmp = f32(b.off_tmp, b.st_rr);
    v.colsq = f32(b.off_colsq, b.st_colsq);
    v.ph = f16(b.off_ph, b.st_p); v.pht = f16(b.off_pht, b.st_p);
    v.rh = f16(b.off_rh, b.st_r); v.qh = f16(b.off_qh, b.st_r); v.qht = f16(b.off_qht, b.st_r);
    v.splits_proj = b.splits_proj; v.splits_back = b.splits_back;
    v.splits_gram[0] = b.splits_gram[0]; v.splits_gram[1] = b.splits_gram[1];
    v.slabs = b.slabs;
    v.small = b.small;
    v.beside = b.beside;
    v.work = b.work;
    v.peers = b.peers;
  }

  // `covers`: how many batches (or, for the factorisations, ranks) the interval stands for; it is
  // booked on the first of them
#define OD_PHASE_BEGIN(ph)                                                              \
  do {                                                                                  \
    if (hipEvent_t* e_ = prof_slot(h, bi, ph, 0, covers)) OD_TRY(hipEventRecord(*e_, st)); \
  } while (0)
#define OD_PHASE_END(ph)                                                                \
  do {                                                                                  \
    if (hipEvent_t* e_ = prof_slot(h, bi, ph, 1, covers)) OD_TRY(hipEventRecord(*e_, st)); \
  } while (0)

  // phases of streaming kernels only: the dispatches' own start / stop time stamps
#define OD_PHASE_KERNEL(ph)                                                             \
  do {                                                                                  \
    hipEvent_t* e0_ = prof_slot(h, bi, ph, 0, covers);                                  \
    hipEvent_t* e1_ = prof_slot(h, bi, ph, 1, covers);                                  \
    if (e0_ && e1_) od::time_next_launch(*e0_, *e1_);                                   \
  } while (0)

  hipStream_t st = caller_st;
  // a cluster as the launchers take it
  int bi = 0, covers = 0;
  auto select = [&](const std::vector<int>& cluster) {
    for (size_t k = 0; k < cluster.size(); ++k) list[k] = &refs[cluster[k]];
    bi = cluster[0];
    covers = (int)cluster.size();
    return covers;
  };

  // Alg. 1 lines 1-2, first part: P_raw = (M + G) Q and its Gram matrix
  auto head = [&](const std::vector<int>& cluster) -> int {
    const int n = select(cluster);
    OD_PHASE_BEGIN(ORTHDION_PHASE_STATS);
    OD_TRY(od::launch_begin(list.get(), n, prec, st));
    OD_PHASE_END(ORTHDION_PHASE_STATS);
    if (diag)
      for (int k : cluster)
        OD_TRY(od::launch_diag_norms(refs[k].d, refs[k].mats, reinterpret_cast<double*>(ws + h->batches[k].off_dpart), h->batches[k].diag_blocks, st));
    OD_PHASE_KERNEL(ORTHDION_PHASE_PROJ);
    OD_TRY(od::launch_proj(list.get(), n, prec, st));
    OD_PHASE_BEGIN(ORTHDION_PHASE_PROJ_REDUCE);
    OD_TRY(od::launch_proj_reduce(list.get(), n, st));
    OD_PHASE_END(ORTHDION_PHASE_PROJ_REDUCE);
    OD_PHASE_BEGIN(ORTHDION_PHASE_GRAM_LEFT);
    OD_TRY(od::launch_orth_gram(list.get(), n, 0, prec, st));
    OD_PHASE_END(ORTHDION_PHASE_GRAM_LEFT);
    return ORTHDION_OK;
  };
  // second CholeskyQR pass of the factor of `side`, up to its deviation
  auto second = [&](const std::vector<int>& cluster, int side) -> int {
    const int n = select(cluster), ph = side == 0 ? ORTHDION_PHASE_ORTH_LEFT : ORTHDION_PHASE_ORTH_RIGHT;
    OD_PHASE_BEGIN(ph);
    OD_TRY(od::launch_orth_second(list.get(), n, side, prec, st));
    OD_PHASE_END(ph);
    return ORTHDION_OK;
  };
  // its result; `which` and `on` as launch_orth_result takes them (2: the flagged matrices, on the second stream)
  auto result = [&](const std::vector<int>& cluster, int side, int which, hipStream_t on) -> int {
    const int n = select(cluster), ph = side == 0 ? ORTHDION_PHASE_FINISH_LEFT : ORTHDION_PHASE_FINISH_RIGHT;
    if (which != 2) OD_PHASE_BEGIN(ph);
    OD_TRY(od::launch_orth_guard(list.get(), n, side, on));
    OD_TRY(od::launch_orth_result(list.get(), n, side, prec, which, on));
    if (which != 2) OD_PHASE_END(ph);
    return ORTHDION_OK;
  };
  // line 3 (R = (M + G)^T P), and the head of line 4
  auto back = [&](const std::vector<int>& cluster) -> int {
    const int n = select(cluster);
    OD_PHASE_KERNEL(ORTHDION_PHASE_BACK);
    OD_TRY(od::launch_back(list.get(), n, prec, st));
    OD_PHASE_BEGIN(ORTHDION_PHASE_BACK_REDUCE);
    OD_TRY(od::launch_back_reduce(list.get(), n, prec, st));
    OD_PHASE_END(ORTHDION_PHASE_BACK_REDUCE);
    if (diag)
      for (int k : cluster)
        OD_TRY(od::launch_diag_cols(refs[k].d.nb, refs[k].d.n, refs[k].d.r, refs[k].ra, refs[k].part, refs[k].slabs,
                                    dacc_all + (size_t)h->batches[k].slot_base * od::kDaccPerMat, st));
    if (h->cfg.variant == ORTHDION_QR) {
      OD_PHASE_BEGIN(ORTHDION_PHASE_GRAM_RIGHT);
      OD_TRY(od::launch_orth_gram(list.get(), n, 1, prec, st));
      OD_PHASE_END(ORTHDION_PHASE_GRAM_RIGHT);
    }
    return ORTHDION_OK;
  };
  // nu = sigma_1(Q_new): Gram matrix of the new right factor, then Lanczos or, above r = 256, power iteration; the table's row
  auto diagnose = [&](int k) -> int {
    const BatchRef& v = refs[k];
    const ClassDims& d = v.d;
    const int slot = h->batches[k].slot_base, sg = v.splits_gram[1];
    double* dacc = dacc_all + (size_t)slot * od::kDaccPerMat;
    od::WsArr q = v.rb;
    if (d.nb == 1) q = od::WsArr{v.host_mats[0].Q, 0};      // one matrix: read where it lies
    else OD_TRY(od::launch_gather_q(d.nb, d.n, d.r, v.mats, v.rb, st));
    OD_TRY(od::launch_gram_plain(d.nb, d.n, d.r, q, v.part, sg, st));
    OD_TRY(od::launch_reduce(d.nb, v.part, sg, (int64_t)d.r * d.r, v.gram, st));
    OD_TRY(od::launch_power(d.nb, d.r, v.gram, v.tmp, v.w, v.part, dacc, st));
    OD_TRY(od::launch_diag_final(d.nb, d.r, reinterpret_cast<const double*>(ws + h->batches[k].off_dpart), h->batches[k].diag_blocks, dacc, v.t1[1], v.t2[1],
                                 h->cfg.variant == ORTHDION_COLNORM ? 1 : 0, diag_all + (size_t)slot * od::kDiagPerMat, st));
    return ORTHDION_OK;
  };
  // lines 5-7: parameter update and error feedback in one pass
  auto update = [&](const std::vector<int>& cluster) -> int {
    const int n = select(cluster);
    if (diag)
      for (int k : cluster) {
        const int rc = diagnose(k);
        if (rc != ORTHDION_OK) return rc;
      }
    OD_PHASE_KERNEL(ORTHDION_PHASE_EFX);
    OD_TRY(od::launch_efx(list.get(), n, prec, a_coef, b_coef, h->cfg.lr, st));
    return ORTHDION_OK;
  };

  // Unit by unit; inside a unit the clusters run piece by piece, so that each of the two Cholesky
  // steps is one launch sequence over all matrices of the unit.  Its time is booked on the unit's
  // first batch.
  auto chol = [&](const Unit& u, int side) -> int {
    const int ph = side == 0 ? ORTHDION_PHASE_CHOL_LEFT : ORTHDION_PHASE_CHOL_RIGHT;
    bi = u.clusters[0][0];
    covers = (int)u.classes.size();
    OD_PHASE_BEGIN(ph);
    const int rc = unit_cholinv(h, u, refs.get(), ws, side, info_all, st);
    if (rc != ORTHDION_OK) return rc;
    OD_PHASE_END(ph);
    return ORTHDION_OK;
  };
  // Ranks above 256 in fast precision: the guard (a launch chain over the class that returns at
  // once for every well-conditioned matrix, then the full product of the flagged ones) runs on
  // the second stream beside the first-order result of the others; the streams join before
  // anything reads a factor.  (With two groups side by side the guard stays on its group's
  // stream: the other group fills the chip meanwhile.)
  auto finish = [&](const Unit& u, int side, bool fork_guard) -> int {
    int rc;
    for (const auto& c : u.clusters)
      if ((rc = second(c, side)) != ORTHDION_OK) return rc;
    const RankClass& cls = h->classes[u.classes[0]];
    const bool forked = fork_guard && allow_second_stream && fast && u.wide_guard && ensure_side_stream(h, st);
    if (forked) {
      OD_TRY(hipEventRecord(h->ev_fork, st));
      OD_TRY(hipStreamWaitEvent(h->side, h->ev_fork, 0));
      if ((rc = class_guard(cls, ws, side, scal_all, info_all, h->side)) != ORTHDION_OK) return rc;
      for (const auto& c : u.clusters)
        if ((rc = result(c, side, 2, h->side)) != ORTHDION_OK) return rc;
      OD_TRY(hipEventRecord(h->ev_join, h->side));
      for (const auto& c : u.clusters)
        if ((rc = result(c, side, 1, st)) != ORTHDION_OK) return rc;
      OD_TRY(hipStreamWaitEvent(st, h->ev_join, 0));
      return ORTHDION_OK;
    }
    const int ph = side == 0 ? ORTHDION_PHASE_GUARD_LEFT : ORTHDION_PHASE_GUARD_RIGHT;
    bi = u.clusters[0][0];
    covers = (int)u.classes.size();
    OD_PHASE_BEGIN(ph);
    if (u.wide_guard && (rc = class_guard(cls, ws, side, scal_all, info_all, st)) != ORTHDION_OK) return rc;
    OD_PHASE_END(ph);
    return ORTHDION_OK;
  };

  // Two groups: the classes of group 1 go to the handle's group stream, which starts after
  // everything enqueued on the caller's stream so far and is joined before the call returns, so
  // the caller sees a single stream.  The groups share no matrix and no workspace slice;
  // whatever one group cannot fill the chip with (its Cholesky chains, the small reductions and
  // corrections, the last round of every launch) the other group's kernels run beside.
  const bool side_by_side = h->two_groups && allow_second_stream && ensure_side_stream(h, caller_st);
  if (side_by_side) {
    OD_TRY(hipEventRecord(h->ev_group_fork, caller_st));
    OD_TRY(hipStreamWaitEvent(h->group_stream, h->ev_group_fork, 0));
  }
  const bool qr = h->cfg.variant == ORTHDION_QR;
  for (const Unit& u : h->units) {
    int rc;
    st = (side_by_side && u.group == 1) ? h->group_stream : caller_st;
    // whether the results are enqueued by finish() itself (the guard on the second stream)
    const bool forks = !side_by_side && allow_second_stream && fast && u.wide_guard && ensure_side_stream(h, st);
    for (const auto& c : u.clusters)
      if ((rc = head(c)) != ORTHDION_OK) return rc;
    if ((rc = chol(u, 0)) != ORTHDION_OK) return rc;
    if ((rc = finish(u, 0, forks)) != ORTHDION_OK) return rc;
    for (const auto& c : u.clusters) {
      if (!forks && (rc = result(c, 0, 0, st)) != ORTHDION_OK) return rc;
      if ((rc = back(c)) != ORTHDION_OK) return rc;
    }
    if (qr) {
      if ((rc = chol(u, 1)) != ORTHDION_OK) return rc;
      if ((rc = finish(u, 1, forks)) != ORTHDION_OK) return rc;
    }
    for (const auto& c : u.clusters) {
      if (!qr) {
        const int n = select(c);
        OD_PHASE_BEGIN(ORTHDION_PHASE_FINISH_RIGHT);
        OD_TRY(od::launch_colnorm(list.get(), n, prec, st));
        OD_PHASE_END(ORTHDION_PHASE_FINISH_RIGHT);
      } else if (!forks && (rc = result(c, 1, 0, st)) != ORTHDION_OK) {
        return rc;
      }
      if ((rc = update(c)) != ORTHDION_OK) return rc;
    }
  }
  st = caller_st;
  if (side_by_side) {
    OD_TRY(hipEventRecord(h->ev_group_join, h->group_stream));
    OD_TRY(hipStreamWaitEvent(caller_st, h->ev_group_join, 0));
  }
  if (h->prof_on && h->prof_steps < h->prof_max_steps) h->prof_steps++;
  return ORTHDION_OK;
}

extern "C" int orthdion_profile_begin(orthdion_handle h, uint32_t phase_mask, int32_t max_steps) {
  if (!h) return ORTHDION_E_NULL_PTR;
  if (max_steps < 1 || max_steps > 100000 || h->prof_on) return ORTHDION_E_INVALID_ARG;
  size_t count = (size_t)max_steps * h->batches.size() * ORTHDION_NPHASE * 2;
  const int rc_alloc = no_throw([&] {
    h->prof_events.assign(count, nullptr);
    h->prof_recorded.assign(count / 2, 0);
    return (int)ORTHDION_OK;
  });
  if (rc_alloc != ORTHDION_OK) return rc_alloc;
  for (int s = 0; s < max_steps; ++s)
    for (size_t b = 0; b < h->batches.size(); ++b)
      for (int ph = 0; ph < ORTHDION_NPHASE; ++ph)
        if (phase_mask & (1u << ph))
          for (int e = 0; e < 2; ++e) {
            size_t idx = (((size_t)s * h->batches.size() + b) * ORTHDION_NPHASE + (size_t)ph) * 2 + (size_t)e;
            if (hipEventCreate(&h->prof_events[idx]) != hipSuccess) return ORTHDION_E_HIP;
          }
  h->prof_mask = phase_mask;
  h->prof_max_steps = max_steps;
  h->prof_steps = 0;
  h->prof_on = true;
  return ORTHDION_OK;
}

extern "C" int orthdion_profile_end(orthdion_handle h, float* ms_per_phase, int32_t* count_per_phase) {
  if (!h || !ms_per_phase || !count_per_phase) return ORTHDION_E_NULL_PTR;
  if (!h->prof_on) return ORTHDION_E_INVALID_ARG;
  int rc = ORTHDION_OK;
  for (int ph = 0; ph < ORTHDION_NPHASE; ++ph) { ms_per_phase[ph] = 0.f; count_per_phase[ph] = 0; }
  const size_t nb = h->batches.size();
  for (int s = 0; s < h->prof_steps; ++s)
    for (size_t b = 0; b < nb; ++b)
      for (int ph = 0; ph < ORTHDION_NPHASE; ++ph) {
        if (!(h->prof_mask & (1u << ph))) continue;
        size_t idx = (((size_t)s * nb + b) * ORTHDION_NPHASE + (size_t)ph) * 2;
        if (!h->prof_recorded[idx / 2]) continue;      // e.g. the Cholesky of a class: first batch only
        float ms = 0.f;
        if (hipEventSynchronize(h->prof_events[idx + 1]) != hipSuccess ||
            hipEventElapsedTime(&ms, h->prof_events[idx], h->prof_events[idx + 1]) != hipSuccess) {
          rc = ORTHDION_E_HIP;
          continue;
        }
        ms_per_phase[ph] += ms;
        count_per_phase[ph] += h->prof_recorded[idx / 2];
      }
  for (hipEvent_t e : h->prof_events)
    if (e) (void)hipEventDestroy(e);
  h->prof_events.clear();
  h->prof_on = false;
  return rc;
}

extern "C" int orthdion_get_info(orthdion_handle h, int32_t* info_host, void* stream) {
  if (!h || !info_host) return ORTHDION_E_NULL_PTR;
  if (!h->last_ws) return ORTHDION_E_NO_STEP;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const int nmat = (int)h->mats.size();
  std::vector<int> raw;
  const int rc_alloc = no_throw([&] { raw.resize((size_t)nmat * od::kInfoPerMat); return (int)ORTHDION_OK; });
  if (rc_alloc != ORTHDION_OK) return rc_alloc;
  const char* ws = reinterpret_cast<const char*>(h->last_ws);
  OD_TRY(hipMemcpyAsync(raw.data(), ws + h->off_info, raw.size() * sizeof(int), hipMemcpyDeviceToHost, st));
  OD_TRY(hipStreamSynchronize(st));
  for (int i = 0; i < nmat; ++i) {
    const Batch& b = h->batches[h->batch_of[i]];
    const int* w = raw.data() + (size_t)(b.slot_base + h->slot_of[i]) * od::kInfoPerMat;
    int v = 0;
    if (w[0] != 0) v = w[0];
    else if (w[1] != 0) v = -w[1];
    else if (w[2] != 0) v = -w[2];
    info_host[i] = v;
  }
  return ORTHDION_OK;
}

extern "C" int orthdion_get_warnings(orthdion_handle h, uint32_t* warn_host, void* stream) {
  if (!h || !warn_host) return ORTHDION_E_NULL_PTR;
  if (!h->last_ws) return ORTHDION_E_NO_STEP;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const int nmat = (int)h->mats.size();
  std::vector<int> raw;
  const int rc_alloc = no_throw([&] { raw.resize((size_t)nmat * od::kInfoPerMat); return (int)ORTHDION_OK; });
  if (rc_alloc != ORTHDION_OK) return rc_alloc;
  const char* ws = reinterpret_cast<const char*>(h->last_ws);
  OD_TRY(hipMemcpyAsync(raw.data(), ws + h->off_info, raw.size() * sizeof(int), hipMemcpyDeviceToHost, st));
  OD_TRY(hipStreamSynchronize(st));
  for (int i = 0; i < nmat; ++i) {
    const Batch& b = h->batches[h->batch_of[i]];
    warn_host[i] = (uint32_t)raw[(size_t)(b.slot_base + h->slot_of[i]) * od::kInfoPerMat + od::kWarnSlot];
  }
  return ORTHDION_OK;
}

extern "C" int orthdion_set_diagnostics(orthdion_handle h, int32_t enable) {
  if (!h) return ORTHDION_E_NULL_PTR;
  for (const Batch& b : h->batches)
    if (enable && b.d.r > 2048) return ORTHDION_E_BAD_SHAPE;     // power iteration keeps a vector of r floats in LDS
  h->diag_on = enable != 0;
  return ORTHDION_OK;
}

extern "C" int orthdion_get_diagnostics(orthdion_handle h, float* out_host, void* stream) {
  if (!h || !out_host) return ORTHDION_E_NULL_PTR;
  if (!h->last_ws || !h->diag_valid) return ORTHDION_E_NO_STEP;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const int nmat = (int)h->mats.size();
  std::vector<float> raw;
  const int rc_alloc = no_throw([&] { raw.resize((size_t)nmat * od::kDiagPerMat); return (int)ORTHDION_OK; });
  if (rc_alloc != ORTHDION_OK) return rc_alloc;
  const char* ws = reinterpret_cast<const char*>(h->last_ws);
  OD_TRY(hipMemcpyAsync(raw.data(), ws + h->off_diag, raw.size() * sizeof(float), hipMemcpyDeviceToHost, st));
  OD_TRY(hipStreamSynchronize(st));
  for (int i = 0; i < nmat; ++i) {
    const Batch& b = h->batches[h->batch_of[i]];
    const float* w = raw.data() + (size_t)(b.slot_base + h->slot_of[i]) * od::kDiagPerMat;
    for (int k = 0; k < od::kDiagPerMat; ++k) out_host[(size_t)i * ORTHDION_NDIAG + k] = w[k];
  }
  return ORTHDION_OK;
}

extern "C" int orthdion_rank_policy(float e_t, float ema_prev, int32_t r_min, int32_t r_max, float alpha, float gamma,
                                    float* ema_out, int32_t* r_next) {
  if (!ema_out || !r_next) return ORTHDION_E_NULL_PTR;
  if (r_min < 8 || r_max < r_min || r_min % 8 || r_max % 8) return ORTHDION_E_INVALID_ARG;
  if (!std::isfinite(e_t) || !std::isfinite(ema_prev) || e_t < 0.f || ema_prev < 0.f) return ORTHDION_E_INVALID_ARG;
  if (!(alpha >= 0.f && alpha <= 1.f) || !(gamma > 0.f) || !std::isfinite(gamma)) return ORTHDION_E_INVALID_ARG;
  // Alg. 2 in double precision: EMA, buffer multiplier, ceiling, clip, multiple of 8
  const double ema = (double)alpha * (double)e_t + (1.0 - (double)alpha) * (double)ema_prev;
  double target = std::ceil((double)gamma * ema);
  if (target < (double)r_min) target = (double)r_min;
  if (target > (double)r_max) target = (double)r_max;
  int32_t nxt = ((int32_t)target + 7) / 8 * 8;
  if (nxt < r_min) nxt = r_min;
  if (nxt > r_max) nxt = r_max;
  *ema_out = (float)ema;
  *r_next = nxt;
  return ORTHDION_OK;
}

extern "C" int orthdion_resize_q(const float* q_old, int64_t n, int32_t r_old, float* q_new, int32_t r_new,
                                 const float* pad, void* stream) {
  if (!q_old || !q_new) return ORTHDION_E_NULL_PTR;
  if (n < 8 || n % 8 || n >= (1 << 24) || r_old < 8 || r_new < 8 || r_old % 8 || r_new % 8 || r_old > n || r_new > n)
    return ORTHDION_E_BAD_SHAPE;
  if (r_new > r_old && !pad) return ORTHDION_E_NULL_PTR;
  if (reinterpret_cast<uintptr_t>(q_old) % 16 || reinterpret_cast<uintptr_t>(q_new) % 16 ||
      reinterpret_cast<uintptr_t>(pad) % 16)
    return ORTHDION_E_MISALIGNED;
  (void)hipGetLastError();
  OD_TRY(od::launch_resize_q(q_old, n, r_old, q_new, r_new, pad, reinterpret_cast<hipStream_t>(stream)));
  return ORTHDION_OK;
}

extern "C" int orthdion_workspace_layout(orthdion_handle h, int32_t index, size_t* off_p, size_t* off_r,
                                         size_t* off_tp1, size_t* off_tp2, size_t* off_tq1, size_t* off_tq2) {
  if (!h) return ORTHDION_E_NULL_PTR;
  if (index < 0 || index >= (int)h->mats.size()) return ORTHDION_E_INVALID_ARG;
  const Batch& b = h->batches[h->batch_of[index]];
  const size_t s = (size_t)h->slot_of[index];
  if (off_p) *off_p = b.off_pa + s * b.st_p * sizeof(float);
  if (off_r) *off_r = b.off_ra + s * b.st_r * sizeof(float);
  if (off_tp1) *off_tp1 = b.off_tp1 + s * b.st_rr * sizeof(float);
  if (off_tp2) *off_tp2 = b.off_tp2 + s * b.st_rr * sizeof(float);
  if (off_tq1) *off_tq1 = b.off_tq1 + s * b.st_rr * sizeof(float);
  if (off_tq2) *off_tq2 = b.off_tq2 + s * b.st_rr * sizeof(float);
  return ORTHDION_OK;
}

extern "C" const char* orthdion_strerror(int status) {
  switch (status) {
    case ORTHDION_OK: return "ok";
    case ORTHDION_E_INVALID_ARG: return "invalid argument";
    case ORTHDION_E_NULL_PTR: return "null pointer";
    case ORTHDION_E_BAD_SHAPE: return "unsupported shape: m, n, r, ld must be multiples of 8 with 8 <= r <= min(m, n) and ld >= n";
    case ORTHDION_E_WORKSPACE_TOO_SMALL: return "workspace too small";
    case ORTHDION_E_MISALIGNED: return "device pointer not sufficiently aligned";
    case ORTHDION_E_HIP: return "HIP call failed";
    case ORTHDION_E_NO_STEP: return "no step has been enqueued on this handle";
    case ORTHDION_E_NO_MEMORY: return "out of host memory";
    default: return "unknown status";
  }
}

extern "C" int orthdion_destroy(orthdion_handle h) {
  if (!h) return ORTHDION_E_NULL_PTR;
  for (hipEvent_t e : h->prof_events)
    if (e) (void)hipEventDestroy(e);
  if (h->ev_fork) (void)hipEventDestroy(h->ev_fork);
  if (h->ev_join) (void)hipEventDestroy(h->ev_join);
  if (h->ev_group_fork) (void)hipEventDestroy(h->ev_group_fork);
  if (h->ev_group_join) (void)hipEventDestroy(h->ev_group_join);
  if (h->side) (void)hipStreamDestroy(h->side);
  if (h->group_stream) (void)hipStreamDestroy(h->group_stream);
  delete h;
  return ORTHDION_OK;
}

// The C ABI of libmagnus (declared in include/magnus.h).
//
// Host side of the hot path: argument validation, per-exponential Leja
// planning (planner.h), buffer rotation for the Newton recurrence and its
// substeps, and the two fourth-order Magnus steps of Section 2 (Cf4, M4)
// built from chained exponentials.  All device work is in kernels.hip.
#include <hip/hip_runtime.h>

#include <cmath>
#include <complex>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <set>
#include <string>
#include <tuple>
#include <utility>
#include <vector>

#include "../../include/magnus.h"
#include "kernels.h"
#include "planner.h"

using magnus::ColParam;
using magnus::CsrDev;
using magnus::ExpPlan;
using magnus::IterArgs;
using magnus::MultiArgs;
using magnus::PersistArgs;
using magnus::PersistExp;
using magnus::PersistProblem;
using magnus::Slot;

namespace {

thread_local std::string g_err;

int fail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return code;
}

#define HIP_TRY(expr)                                                                    \
  do {                                                                                   \
    hipError_t e_ = (expr);                                                              \
    if (e_ != hipSuccess) return fail(MAGNUS_EHIP, "%s: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

// Workspace vectors per state.
enum Vec { kA = 0, kB, kS0, kS1, kS2, kU, kV, kY, kNumVec };

// Device table of per-state Leja parameters (ColParam entries) filled once per call segment.
constexpr size_t kTableCap = 1 << 18;
// Per-call headers of the persistent small-state kernel.
constexpr size_t kArenaBytes = 8u << 20;
// States of at most this many entries run whole propagations in one workgroup.
constexpr int64_t kSmallDim = magnus::kPersistMaxDim;
// Row mappings magnus_autotune times (variant codes 1..kTuneVariants).
constexpr int kTuneVariants = 7;

}  // namespace

struct magnus_ctx {
  int device = 0;
  int64_t max_dim = 0;
  int32_t max_batch = 0;
  double2* vecs = nullptr;     // kNumVec vectors of max_dim * max_batch entries
  Slot* slots = nullptr;       // one control block per state of a batch
  int nslots = 0;
  int sticky_status = 0;       // status bits of slots reset inside the current call
  ColParam* table = nullptr;   // kTableCap entries
  unsigned char* arena = nullptr;  // kArenaBytes
  // coded CSR terms (kernels_coded.hip): the form that the current call's terms
  // were rewritten in, for the Hamiltonian at coded_h while the call runs
  magnus::CodedDev coded{};
  size_t coded_slices = 0, coded_blocks = 0;  // what its buffers hold (reserve_coded)
  bool coded_tried = false;                   // whether they have been asked for
  magnus::CodeTerms coded_terms{};
  const magnus_hamiltonian* coded_h = nullptr;
  bool coded_pairs = false;      // the states of the current call's batch run as interleaved pairs
  magnus::PairArgs pair_last{};  // every problem's last launch of pairs, for the check of their norms
  bool pair_pending = false;
  double2* split = nullptr;      // shares of a dense group's products (split_entries of them)
  long long split_entries = 0;
  double* dots = nullptr;        // per-workgroup sums of dot products, and a result (inside partials)
  int coding = 1;   // MAGNUS_CODED: 0 reads the CSR arrays in every iteration, 2 codes the terms of every call
  // term pairs found to fit the coded form when they were scanned: only a
  // guess at what pays, since every call codes the arrays as they are then and
  // reads a block that does not fit from them
  std::set<std::tuple<const void*, const void*, const void*, const void*, int64_t>> codable;
  int persist = 1;  // MAGNUS_PERSIST: 0 never, 1 by size and state count, 2 every state of at most kSmallDim
  int fuse = 1;     // MAGNUS_FUSE: 0 a decide kernel after every iteration, 1 stop tests fused on small grids
  magnus::IterArgs fz_last{};  // the arguments of a final check of the last fused iteration
  bool fz_pending = false;     // a fused iteration ran since the last final check
  // graph replay of single-state steps (MAGNUS_GRAPH: 0 off, 1 on): one Magnus
  // step captured on cap_stream, replayed once per step with the step's Leja
  // coefficients read from a device table indexed by the counter *gctr
  int graph = 0;         // off by default: replays measured slower than launches once the stop tests are fused
  int graph_chunk = 0;  // MAGNUS_GRAPH_STEPS: steps per uploaded table chunk (0: as many as fit)
  int ragged_joint = 1; // MAGNUS_RAGGED_JOINT: 0 runs a ragged batch's large problems one after another
  int* gctr = nullptr;
  hipStream_t cap_stream = nullptr;
  hipGraph_t graph_g = nullptr;
  hipGraphExec_t graph_x = nullptr;
  hipEvent_t graph_done = nullptr;  // recorded after the last replay of the current graph
  Slot* seen = nullptr;             // pinned: the slots as of seen_at (copy_slots)
  hipEvent_t seen_at = nullptr;
  std::vector<magnus::IterCoef> graph_table;  // host side of the last uploaded table chunk
  double2* assembled = nullptr;  // magnus_reserve_dense
  int64_t assembled_dim = 0;
  double2* comm = nullptr;       // magnus_dense_commutator: K = i[H1, H2], row stride comm_dim
  int64_t comm_dim = 0;
  const void* comm_h1 = nullptr;  // the dense pair K belongs to (value pointers, dim, ld)
  const void* comm_h2 = nullptr;
  int64_t comm_n = 0, comm_ld = 0;
  // magnus_csr_commutator: K = i[H1, H2] as CSR (row stride-free arrays of
  // kc_rows + 1, kc_cap entries) for the pair of CSR terms recognised by kc_key
  int* kc_rp = nullptr;
  int* kc_ci = nullptr;
  double2* kc_val = nullptr;
  int64_t kc_rows = 0, kc_cap = 0, kc_nnz = 0;
  std::tuple<const void*, const void*, const void*, const void*, int64_t> kc_key{nullptr, nullptr, nullptr, nullptr, 0};
  bool kc_codable = false;  // H1, H2 and K were found to fit the coded form (a guess at what pays, as codable)
  // magnus_csr_m6_prepare: P_a = -i[H_a, K] (a = 1, 2) as CSR for the pair K
  // belongs to (valid while pm_key equals kc_key; null where no iteration reads
  // them), their enclosures, and kM6Vecs work vectors of pm_ws_dim entries for the M6 iteration
  int* pm_rp[2] = {nullptr, nullptr};
  int* pm_ci[2] = {nullptr, nullptr};
  double2* pm_val[2] = {nullptr, nullptr};
  int64_t pm_rows[2] = {0, 0}, pm_cap[2] = {0, 0}, pm_nnz[2] = {0, 0};
  double pm_lo[2] = {0.0, 0.0}, pm_hi[2] = {0.0, 0.0};
  double2* pm_ws = nullptr;
  int64_t pm_ws_dim = 0;
  std::tuple<const void*, const void*, const void*, const void*, int64_t> pm_key{nullptr, nullptr, nullptr, nullptr, 0};
  // magnus_dense_m6_prepare: the nested commutators of M6, kM6Mats matrices of
  // m6_dim^2 entries, with Gershgorin enclosures, for the pair K belongs to
  double2* m6 = nullptr;
  int64_t m6_dim = 0;
  bool m6_ready = false;
  double m6_lo[7] = {0, 0, 0, 0, 0, 0, 0}, m6_hi[7] = {0, 0, 0, 0, 0, 0, 0};
  double* partials = nullptr;  // npartials doubles
  size_t npartials = 0;
  int64_t max_grid = 0;
  double* scan = nullptr;      // per-workgroup outputs of the Gershgorin scans
  int64_t scan_len = 0;
  std::set<std::tuple<const void*, const void*, const void*, int64_t, int64_t>> validated;
  std::mutex mu;
  // kernel timing: (kind, start, stop) per recorded launch, events reused from a pool
  int csr_variant = 0;  // MAGNUS_CSR_VARIANT: 0 by size (variant_rows), 1 eight lanes per row (nonzero
                        // streaming from 2^16 rows on), 2-4 row-per-lane (64/32/128 rows), 5-6 wave tiles
                        // (8/16 rows), 7 streamed wave tiles
  // magnus_autotune results, per CSR term pair (H1 row_ptr, dim): the variant code
  // of the single-state iteration and the states per multi-state pass
  std::map<std::pair<const void*, int64_t>, int> tuned_variant, tuned_group;
  // and where these were faster than iterations on the coded terms (single states; batches)
  std::set<std::pair<const void*, int64_t>> uncoded_single, uncoded_batch;
  // magnus_autotune results for dense terms, per (H1 values, dim): rows per
  // wave of the GEMV iteration and the FP64-MFMA tile of group iterations
  std::map<std::pair<const void*, int64_t>, int> tuned_dense_rpw, tuned_mfma;
  int dense_rpw_env = 0;   // MAGNUS_DENSE_RPW: 1, 2 or 4 rows per wave of the GEMV iteration (0: tuned or 2)
  int persist_cache = 1;   // MAGNUS_PERSIST_CACHE: 0 keeps the small-state kernel's term 1 out of LDS
  int fuse_assembly = 1;   // MAGNUS_ASSEMBLE_FUSED: 0 assembles a dense exponent in a pass of its own
  int mfma_tile_env = -1;  // MAGNUS_MFMA_TILE: 0..6 forces an FP64-MFMA tile shape (-1: tuned or the size rule)
  int timing = 0;  // 0 off, k >= 1: every k-th launch of each kernel class is bracketed
  int64_t timing_seq[MAGNUS_KERNEL_CSR_LEJA3 + 1] = {};  // launches of each class since enabling
  std::vector<std::tuple<int, hipEvent_t, hipEvent_t>> records;
  std::vector<hipEvent_t> pool;
  size_t pool_used = 0;

  double2* vec(int k) { return vecs + (size_t)k * (size_t)max_dim * (size_t)max_batch; }
};

namespace {

bool is_fin(double x) { return std::isfinite(x); }

int check_term(const magnus_term& t, int64_t dim, const char* name) {
  if (t.format != MAGNUS_CSR && t.format != MAGNUS_DENSE)
    return fail(MAGNUS_EINVAL, "%s: unknown format %d", name, t.format);
  if (t.dim != dim) return fail(MAGNUS_EINVAL, "%s: dim %lld != %lld", name, (long long)t.dim, (long long)dim);
  if (t.format == MAGNUS_CSR) {
    if (t.nnz < 0 || t.nnz > INT32_MAX) return fail(MAGNUS_EINVAL, "%s: nnz %lld out of range", name, (long long)t.nnz);
    // a term without entries (the zero matrix) may pass null column and value arrays
    if (!t.row_ptr || (t.nnz > 0 && (!t.col_idx || !t.val)))
      return fail(MAGNUS_EINVAL, "%s: null CSR array", name);
  } else {
    if (!t.val) return fail(MAGNUS_EINVAL, "%s: null val", name);
    if (t.ld < dim) return fail(MAGNUS_EINVAL, "%s: ld %lld < dim", name, (long long)t.ld);
  }
  if (!is_fin(t.lam_min) || !is_fin(t.lam_max) || t.lam_min > t.lam_max)
    return fail(MAGNUS_EDOMAIN, "%s: spectral enclosure [%g, %g] invalid", name, t.lam_min, t.lam_max);
  return MAGNUS_OK;
}

int check_ham(magnus_ctx* ctx, const magnus_hamiltonian* h, int need_k) {
  if (!ctx) return fail(MAGNUS_EINVAL, "null context");
  if (!h) return fail(MAGNUS_EINVAL, "null hamiltonian");
  const int64_t dim = h->H1.dim;
  if (dim < 1) return fail(MAGNUS_EINVAL, "dim %lld < 1", (long long)dim);
  if (dim > ctx->max_dim) return fail(MAGNUS_ENOMEM, "dim %lld exceeds workspace max_dim %lld", (long long)dim, (long long)ctx->max_dim);
  if (dim > INT32_MAX / 2) return fail(MAGNUS_EINVAL, "dim %lld too large", (long long)dim);
  int rc = check_term(h->H1, dim, "H1");
  if (rc) return rc;
  rc = check_term(h->H2, dim, "H2");
  if (rc) return rc;
  if (h->H1.format != h->H2.format) return fail(MAGNUS_EINVAL, "H1 and H2 must share a format");
  if (h->H1.format == MAGNUS_DENSE && h->H1.ld != h->H2.ld)
    return fail(MAGNUS_EINVAL, "dense H1 and H2 must share the row stride ld");
  if (need_k && (!is_fin(h->k_min) || !is_fin(h->k_max) || h->k_min > h->k_max))
    return fail(MAGNUS_EDOMAIN, "commutator enclosure [%g, %g] invalid", h->k_min, h->k_max);
  return MAGNUS_OK;
}

int check_opts(const magnus_leja_opts* o) {
  if (!o) return fail(MAGNUS_EINVAL, "null options");
  if (!(o->tol > 0.0) || !is_fin(o->tol)) return fail(MAGNUS_EDOMAIN, "tol %g must be positive and finite", o->tol);
  if (o->max_degree < 1 || o->max_degree > MAGNUS_MAX_DEGREE)
    return fail(MAGNUS_EINVAL, "max_degree %d outside 1..%d", o->max_degree, MAGNUS_MAX_DEGREE);
  if (o->max_substeps < 1) return fail(MAGNUS_EINVAL, "max_substeps %d < 1", o->max_substeps);
  if (o->tol_mode != 0 && o->tol_mode != 1) return fail(MAGNUS_EINVAL, "tol_mode %d", o->tol_mode);
  return MAGNUS_OK;
}

void release_coded(magnus_ctx* ctx) {
  if (ctx->coded.dict) (void)hipFree(ctx->coded.dict);  // (the first of its arrays)
  ctx->coded = magnus::CodedDev{};
}

// The buffers of the coded form, when CSR terms are first looked at for it: 153
// bytes per row of max_dim, and 8 KiB per block of rows (of 64 up to 65,536 rows,
// then 1,024 blocks), in one allocation (magnus_spectral_bounds of a new context,
// 65,536 / 262,144 rows, 112 / 302 us; with six 134 / 338).  Without them every
// call reads the CSR arrays.
void reserve_coded(magnus_ctx* ctx) {
  if (ctx->coded_tried || !ctx->coding || ctx->max_dim > magnus::kCodeMaxDim) return;
  ctx->coded_tried = true;
  const int64_t n = ctx->max_dim;
  const size_t slices = ctx->coded_slices = ((size_t)n + 63) / 64 * 4;
  const size_t blocks = ctx->coded_blocks = (size_t)std::min<int64_t>(magnus::kFuseMaxGrid, (n + 63) / 64);
  size_t bytes = 0;
  auto place = [&](size_t size) { return std::exchange(bytes, bytes + (size + 255) / 256 * 256); };
  const size_t dict = place(sizeof(magnus::CodeEntry) * (magnus::kCodeMax + 1) * blocks);
  const size_t codes = place(sizeof(unsigned) * 64 * magnus::kCodeAhead * slices);
  const size_t more = place(sizeof(unsigned) * 64 * magnus::kCodeMore * slices);
  const size_t head = place(sizeof(unsigned) * magnus::kCodeHead * slices);
  const size_t block = place(sizeof(int) * blocks);
  const size_t diag = place(sizeof(double) * magnus::kCodeTerms * (size_t)n);
  char* at = nullptr;
  if (hipMalloc(&at, bytes) != hipSuccess) {
    (void)hipGetLastError();  // (the next launch would report it)
    return;
  }
  magnus::CodedDev& C = ctx->coded;
  C.dict = reinterpret_cast<magnus::CodeEntry*>(at + dict);
  C.codes = reinterpret_cast<unsigned*>(at + codes);
  C.more = reinterpret_cast<unsigned*>(at + more);
  C.head = reinterpret_cast<unsigned*>(at + head);
  C.block = reinterpret_cast<int*>(at + block);
  C.diag = reinterpret_cast<double*>(at + diag);
  C.diag_stride = n;
}

int launch_probe(magnus_ctx* ctx, const magnus_hamiltonian* h, bool with_k, int* bad_dev, const double* flags,
                 int nflags, hipStream_t s);
bool coding_possible(const magnus_ctx* ctx, const magnus_hamiltonian* h);

// Structural check (and Gershgorin enclosure) of n <= 2 CSR terms of one
// dimension, run once per term, with one wait for all of them.  *valid: the terms
// found sound, in order, before the first that is not (MAGNUS_EINVAL then).  The
// two terms of `both` are coded as well, to say in *fits whether all blocks of rows
// fit the form (behind the scans on the stream, by a kernel that looks at their flags
// before it reads the arrays).
int csr_scan(magnus_ctx* ctx, const magnus_term* const* t, int n, hipStream_t s, double* lo, double* hi,
             int* valid = nullptr, const magnus_hamiltonian* both = nullptr, bool* fits = nullptr) {
  if (valid) *valid = 0;
  if (fits) *fits = false;
  if (both) reserve_coded(ctx);
  const bool probe = both && fits && coding_possible(ctx, both);
  const int dim = (int)t[0]->dim;
  const int grid = magnus::csr_gershgorin_grid(dim);
  const size_t len = 3 * (size_t)grid * n;
  if ((int64_t)len + 1 > ctx->scan_len) return fail(MAGNUS_ENOMEM, "scan buffer too small");
  auto key = [](const magnus_term& x) {
    return std::make_tuple((const void*)x.row_ptr, (const void*)x.col_idx, x.val, x.dim, x.nnz);
  };
  {
    // a term scanned again (its arrays may have been rewritten) counts as valid only if this scan passes
    std::lock_guard<std::mutex> g(ctx->mu);
    for (int k = 0; k < n; ++k) ctx->validated.erase(key(*t[k]));
  }
  hipError_t e = hipSuccess;
  for (int k = 0; k < n && e == hipSuccess; ++k) {
    const CsrDev d{t[k]->row_ptr, t[k]->col_idx, reinterpret_cast<const double2*>(t[k]->val)};
    e = magnus::launch_csr_gershgorin(d, dim, t[k]->nnz, ctx->scan + (size_t)k * 3 * grid, grid, s);
  }
  int* bad_dev = reinterpret_cast<int*>(ctx->scan + len);
  if (e == hipSuccess && probe)
    if (int rc = launch_probe(ctx, both, false, bad_dev, ctx->scan, grid * n, s)) return rc;
  std::vector<double> h(len + 1);
  if (e == hipSuccess) e = hipMemcpyAsync(h.data(), ctx->scan, sizeof(double) * h.size(), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) return fail(MAGNUS_EHIP, "CSR scan: %s", hipGetErrorString(e));
  for (int k = 0; k < n; ++k) {
    double a = INFINITY, b = -INFINITY;
    bool bad = false;
    for (const double* r = h.data() + (size_t)k * 3 * grid; r < h.data() + (size_t)(k + 1) * 3 * grid; r += 3) {
      a = std::fmin(a, r[0]);
      b = std::fmax(b, r[1]);
      bad = bad || r[2] != 0.0;
    }
    if (bad) return fail(MAGNUS_EINVAL, "malformed CSR (row_ptr not monotone / not 0..nnz, or column out of range)");
    lo[k] = a;
    hi[k] = b;
    if (valid) *valid = k + 1;
    std::lock_guard<std::mutex> g(ctx->mu);
    ctx->validated.insert(key(*t[k]));
  }
  if (probe) {
    int bad = 0;
    memcpy(&bad, &h[len], sizeof bad);
    *fits = bad == 0;
  }
  return MAGNUS_OK;
}

int probe_coding(magnus_ctx* ctx, const magnus_hamiltonian* h, bool with_k, bool* fits, hipStream_t s);
void note_codable(magnus_ctx* ctx, const magnus_hamiltonian* h, bool fits);

int ensure_valid(magnus_ctx* ctx, const magnus_hamiltonian* h, hipStream_t s) {
  const magnus_term* unseen[2];
  int n = 0;
  for (const magnus_term* t : {&h->H1, &h->H2}) {
    if (t->format != MAGNUS_CSR) continue;
    auto key = std::make_tuple((const void*)t->row_ptr, (const void*)t->col_idx, t->val, t->dim, t->nnz);
    std::lock_guard<std::mutex> g(ctx->mu);
    if (!ctx->validated.count(key)) unseen[n++] = t;
  }
  if (n == 0) return MAGNUS_OK;
  double lo[2], hi[2];
  bool fits = false;
  if (int rc = csr_scan(ctx, unseen, n, s, lo, hi, nullptr, n == 2 ? h : nullptr, &fits)) return rc;
  if (n == 1)
    if (int rc = probe_coding(ctx, h, false, &fits, s)) return rc;
  note_codable(ctx, h, fits);
  return MAGNUS_OK;
}

int dense_scan(magnus_ctx* ctx, const magnus_term& t, hipStream_t s, double* lo, double* hi) {
  const int dim = (int)t.dim;
  const int grid = magnus::dense_gershgorin_grid(dim);
  if (2 * (int64_t)grid > ctx->scan_len) return fail(MAGNUS_ENOMEM, "scan buffer too small");
  double* dout = ctx->scan;
  hipError_t e = magnus::launch_dense_gershgorin(reinterpret_cast<const double2*>(t.val), dim, t.ld, dout, grid, s);
  std::vector<double> h(2 * (size_t)grid);
  if (e == hipSuccess) e = hipMemcpyAsync(h.data(), dout, sizeof(double) * h.size(), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) return fail(MAGNUS_EHIP, "dense scan: %s", hipGetErrorString(e));
  double a = INFINITY, b = -INFINITY;
  for (int g = 0; g < grid; ++g) { a = std::fmin(a, h[2 * g]); b = std::fmax(b, h[2 * g + 1]); }
  *lo = a;
  *hi = b;
  return MAGNUS_OK;
}

// Host-side record of the work a call enqueued.
struct Acc {
  int64_t exponentials = 0, substeps = 0, planned = 0;
  int64_t extra_iters = 0;  // iterations already counted by nested calls
  int32_t max_m = 0, max_s = 0;
  double max_bound = 0.0;
  int products_per_iter = 2;
};

struct ExpOp {
  const magnus_hamiltonian* h;
  double a, b, kappa;
  const double2* assembled = nullptr;  // dense: the exponent assembled (row stride dim), used with a = 1
  bool has_interval = false;           // spectral enclosure given (else Weyl from a, b, kappa)
  double lo = 0.0, hi = 0.0;
  const double* m6c = nullptr;         // CSR Method M6: the ten coefficients of the exponent (matrix-free)
  // dense: the first iteration also writes the assembled exponent
  // fuse_out = fa H1 + fb H2 (+ fk K), the matrix `assembled` points to
  bool fuse_assembly = false;
  double fa = 0.0, fb = 0.0, fk = 0.0;
  const double2* fK = nullptr;
  double2* fuse_out = nullptr;
};

// Whether the context holds K = i[H1, H2] of this pair of CSR terms.
bool csr_comm_ready(const magnus_ctx* ctx, const magnus_hamiltonian* h) {
  return ctx->kc_rp && h->H1.format == MAGNUS_CSR &&
         ctx->kc_key == std::make_tuple((const void*)h->H1.row_ptr, h->H1.val, (const void*)h->H2.row_ptr, h->H2.val,
                                        h->H1.dim);
}

// Whether the context holds K and P_1, P_2 of Method M6 for this pair of CSR terms.
bool csr_m6_ready(const magnus_ctx* ctx, const magnus_hamiltonian* h) {
  return csr_comm_ready(ctx, h) && ctx->pm_key == ctx->kc_key && ctx->pm_ws && ctx->pm_ws_dim >= h->H1.dim;
}

// Whether the context holds K = i[H1, H2] of this pair of dense terms.
bool dense_comm_ready(const magnus_ctx* ctx, const magnus_hamiltonian* h) {
  return ctx->comm && ctx->comm_h1 == h->H1.val && ctx->comm_h2 == h->H2.val && ctx->comm_n == h->H1.dim &&
         ctx->comm_ld == h->H1.ld;
}

auto pair_key(const magnus_hamiltonian* h) {
  return std::make_tuple((const void*)h->H1.row_ptr, h->H1.val, (const void*)h->H2.row_ptr, h->H2.val, h->H1.dim);
}

CsrDev csr_dev(const magnus_term& t) {
  return CsrDev{t.row_ptr, t.col_idx, reinterpret_cast<const double2*>(t.val)};
}

// Whether the context can hold CSR terms of this dimension in coded form.
bool coding_possible(const magnus_ctx* ctx, const magnus_hamiltonian* h) {
  return ctx->coding && ctx->coded.codes && h->H1.format == MAGNUS_CSR && h->H1.dim <= magnus::kCodeMaxDim;
}

// Code the terms once, counting the blocks of rows that do not fit in *bad_dev
// (flags: as launch_code_build).
int launch_probe(magnus_ctx* ctx, const magnus_hamiltonian* h, bool with_k, int* bad_dev, const double* flags,
                 int nflags, hipStream_t s) {
  ctx->coded_h = nullptr;
  const int dim = (int)h->H1.dim;
  magnus::CodeTerms T{2, {csr_dev(h->H1), csr_dev(h->H2)}};
  if (with_k) T.m[T.n++] = CsrDev{ctx->kc_rp, ctx->kc_ci, ctx->kc_val};
  ctx->coded.rows = magnus::code_rows(dim);
  HIP_TRY(magnus::launch_step_set(bad_dev, 0, s));
  HIP_TRY(magnus::launch_code_build(T, dim, ctx->coded, bad_dev, s, flags, nflags));
  return MAGNUS_OK;
}

// Whether every block of rows fits the coded form (where the terms have just
// been scanned or assembled; synchronous, as those are).
int probe_coding(magnus_ctx* ctx, const magnus_hamiltonian* h, bool with_k, bool* fits, hipStream_t s) {
  *fits = false;
  ctx->coded_h = nullptr;
  reserve_coded(ctx);
  if (!coding_possible(ctx, h)) return MAGNUS_OK;
  int bad = 0;
  int* bad_dev = ctx->gctr + 1;
  if (int rc = launch_probe(ctx, h, with_k, bad_dev, nullptr, 0, s)) return rc;
  HIP_TRY(hipMemcpyAsync(&bad, bad_dev, sizeof(int), hipMemcpyDeviceToHost, s));
  HIP_TRY(hipStreamSynchronize(s));
  *fits = bad == 0;
  return MAGNUS_OK;
}

void note_codable(magnus_ctx* ctx, const magnus_hamiltonian* h, bool fits) {
  if (fits) ctx->codable.insert(pair_key(h));
  else ctx->codable.erase(pair_key(h));
}

// The norm partials of pairs lie behind those of single states (two halves by
// iteration parity each): 4 doubles per pair and block of rows.
size_t pair_partials_at(const magnus_ctx* ctx) { return 4 * (size_t)ctx->max_grid; }
bool pair_partials_fit(const magnus_ctx* ctx, int64_t pair_blocks) {
  return pair_partials_at(ctx) + 8 * (size_t)pair_blocks <= ctx->npartials;
}

// Whether an M6 iteration on the CSR arrays takes two passes over H1, H2, K, P1
// and P2 rather than three over H1, H2 and K: by the entries of a row in P1 and P2
// (p) and in the others (h).  Measured, us per iteration, two passes / three:
// chains (p = 2.0 h to 2.7 h) n = 6 13.6 / 17.6, n = 8 17.2 / 19.3, n = 10
// 21.1 / 21.6, n = 11 23.3 / 22.4, n = 12 26.2 / 22.5; rings (1.1 h to 1.5 h) n = 8
// 15.0 / 19.9, n = 12 19.4 / 21.0; long-range couplings n = 8 (2.2 h) 15.2 / 19.5,
// n = 12 (3.2 h) 23.2 / 21.9.  From 2^14 rows on, where it is the entries read that
// count: the chain with coupling 1, whose P cancel (1.1 h), n = 15 29.2 / 35.1,
// n = 16 48.4 / 56.8, n = 17 94.7 / 95.4, n = 18, past what the MALL holds,
// 219 / 171; rings n = 14 (1.6 h) 29.9 / 24.4, n = 16 (1.7 h) 71.5 / 56.1.  Rows
// that are one round of loads either way (p = 8): 60,001 random rows 30.6 / 38.0.
bool m6_two_passes(const magnus_ctx* ctx, const magnus_hamiltonian* h) {
  if (!ctx->pm_rp[0] || !ctx->pm_rp[1]) return false;  // (released by the preparation)
  const int64_t dim = h->H1.dim;
  const double rows = (double)dim, all = (double)(h->H1.nnz + h->H2.nnz + ctx->kc_nnz);
  const double ps = (double)(ctx->pm_nnz[0] + ctx->pm_nnz[1]);
  if (ps <= 10.0 * rows || (dim <= 512 && ps <= 64.0 * rows)) return true;
  if (dim < 16384) return ps <= 2.25 * all;
  return ps <= 1.25 * all && 20.0 * (all + ps) <= 200e6;
}

// Exponentials from which coding pays.  It costs 10 to 20 us up to 2^16 rows (21 at
// the chain of 16 sites, 53 at 18, 200 at 20), and an exponential takes four
// iterations or more.  One state, us per step of two exponentials on the CSR
// arrays / on the coded terms, terms of 7 / 15 / 21 / 31 entries a row:
//   12,000 rows  55 / 56, 57 / 58, 60 / 59, 62 / 60 (and less gain below)
//   16,384 rows  55 / 56, 56 / 57, 60 / 59, 63 / 59: pays from 18 and 9 exponentials on
//   24,000 rows  60 / 60, 62 / 61, 65 / 63, 69 / 64: from 9 and 5
//   28,672 rows  61 / 61, 65 / 61, 70 / 63, 74 / 64: from 6, 2 and 2
//   40,009 rows  65 / 66, 71 / 67, 78 / 69, 84 / 70: from 3, 2 and 2
//   49,153 rows  92 / 68, 99 / 70, 105 / 71, 126 / 72: from the first
// M6's three passes: chains, n = 12 22 / 20, n = 16 58 / 30 us per iteration (below
// 2^14 rows two passes on the arrays come first where they are taken: rings of 10
// and 12 sites 17.4 / 18.3 and 19.4 / 18.5 coded).  A gradient, six exponentials a
// step, two of them pairs: 1,024 to 49,153 rows of 7 / 21 entries 1.24 to 1.4 /
// 1.6 to 1.8 times as fast, from the first step on.  Pairs: from the second
// exponential on where they are the faster (pairs_slower).
enum class CodeUse { kSingle, kM6, kGradient };
int64_t coding_pays(const magnus_hamiltonian* h, int npairs, CodeUse use) {
  const int64_t dim = h->H1.dim;
  if (dim > 49152 && npairs == 0) return 1;
  if (dim >= 65536 || use == CodeUse::kGradient) return 1;
  if (npairs > 0) return 2;
  if (use == CodeUse::kM6) return dim >= 16384 ? 2 : 6;
  const double per_row = (double)(h->H1.nnz + h->H2.nnz) / (double)dim;
  if (dim >= 28672) return per_row >= 12 ? 3 : INT64_MAX;
  return dim < 16384 || per_row < 20 ? INT64_MAX : per_row < 28 ? 12 : 6;
}

// Whether groups of states on the CSR arrays are faster than pairs on the coded
// terms: short rows, and groups of a power of two states.  Measured, groups' time
// over pairs', terms of 3 / 5 / 7 entries a row, by the states times their rows
// (calls of 2, 4 and 8 exponentials where they differ):
//   60,000          0.97 / 0.99 / 1.0, 1.0 / 1.03 / 1.03 and 1.0 / 1.04 / 1.08
//   90,000..131,070 0.90 / 0.93 / 0.94, 0.93 / 0.96 / 0.99 and 0.95 / 0.97 (two and
//                   four states) 1.02 (more) / 1.02
//   2^18            batches of 16 0.94 / 0.96 / 0.96, of 4 0.89 / 0.91 / 0.95
//   640,000         batches of 16 0.81 / 0.86 / 0.92; 1,440,000 0.90 / 0.97 / 1.01
//   3,200,000       batches of 16 1.1 / 1.2 / 1.27
// Two states, 8 exponentials: 300,000 0.83 / 0.89 / 0.98, 330,000 0.95 / 1.03 / 1.18,
// 360,000 0.96 / 1.06 / 1.23, 640,000 0.88 / 1.02, 1,200,000 0.86 / 0.99 (2 exponentials
// 360,000 0.90 / 0.98 / 1.12).  Batches of 3, 6, 7, 12 and 20 1.0 to 2.1 (5 at 150,000
// 0.93 / 0.96 / 1.0).  9 / 11 / 15 entries a row, 2 exponentials, batches of 4, 8 and
// 16 at 130,000 0.97 / 1.0 / 1.03, 160,000 to 320,000 0.88 to 0.98 / 0.88 to 0.97 / 0.90
// to 1.0, 360,000 1.05 / 1.03 / 1.1 (4 exponentials 0.93 to 1.0 / 0.90 to 0.97 / 0.94 to
// 1.0, 8 and more even), two states and more entries 1.0 to 2.
bool pairs_slower(const magnus_hamiltonian* h, int batch, int64_t exponentials) {
  const int64_t dim = h->H1.dim, nnz = h->H1.nnz + h->H2.nnz, states = dim * std::min(batch, 32);
  if ((batch < 32 && (batch & (batch - 1))) || states < 62000) return false;
  if (nnz >= 8 * dim)
    return nnz < 14 * dim && batch > 2 && exponentials < 4 && states >= 1 << 17 && states <= 340000;
  const bool least = 2 * nnz < 9 * dim, few = nnz < 6 * dim;
  if (states < 1 << 17) return exponentials < 8 || least || (few && batch <= 4);
  if (batch == 2 && !least) return states <= (few ? 360000 : 310000);
  return states <= (few ? 3000000 : 1 << 20);
}

// Whether magnus_autotune found a mapping of the CSR arrays (for batches a group
// size) faster than the iterations on the coded terms.
bool tuned_uncoded(const magnus_ctx* ctx, const magnus_hamiltonian* h, bool batch) {
  return (batch ? ctx->uncoded_batch : ctx->uncoded_single).count({(const void*)h->H1.row_ptr, h->H1.dim}) > 0;
}

// Rows per block of the coded terms for a batch.
int batch_rows(const magnus_hamiltonian* h, int batch) {
  return magnus::code_pair_rows((int)h->H1.dim, std::min(batch / 2, 16), 64, h->H1.nnz + h->H2.nnz, batch % 2 != 0);
}

// At the start of a call on CSR terms: rewrite the terms in coded form
// when the call's iterations pay for that.  `with_k`: its iterations apply the
// assembled commutator too.
// batch > 1: as many states run in groups, on coded terms as pairs (and perhaps one more).
int begin_coded(magnus_ctx* ctx, const magnus_hamiltonian* h, bool with_k, int64_t exponentials, int batch,
                hipStream_t s, CodeUse use = CodeUse::kSingle) {
  ctx->coded_h = nullptr;
  ctx->coded_pairs = false;
  const int npairs = std::min(batch / 2, 16);
  if (!coding_possible(ctx, h) || ctx->csr_variant) return MAGNUS_OK;
  const int64_t dim = h->H1.dim;
  const int rows = npairs > 0 ? batch_rows(h, batch) : magnus::code_rows((int)dim);
  if (npairs > 0 && (!ctx->fuse || !pair_partials_fit(ctx, (int64_t)magnus::code_grid((int)dim, rows) * npairs)))
    return MAGNUS_OK;
  if (ctx->coding < 2) {
    if (with_k ? !ctx->kc_codable : !ctx->codable.count(pair_key(h))) return MAGNUS_OK;
    if (exponentials < coding_pays(h, npairs, use) || (npairs > 0 && pairs_slower(h, batch, exponentials))) return MAGNUS_OK;
    if (use == CodeUse::kM6 && dim < 16384 && m6_two_passes(ctx, h)) return MAGNUS_OK;
    // (the tuner times none of M6's iterations)
    if (use != CodeUse::kM6 && tuned_uncoded(ctx, h, npairs > 0)) return MAGNUS_OK;
  }
  magnus::CodeTerms T{2, {csr_dev(h->H1), csr_dev(h->H2)}};
  if (with_k) T.m[T.n++] = CsrDev{ctx->kc_rp, ctx->kc_ci, ctx->kc_val};
  ctx->coded.rows = rows;
  HIP_TRY(magnus::launch_code_build(T, (int)dim, ctx->coded, nullptr, s));
  ctx->coded_terms = T;
  ctx->coded_h = h;
  ctx->coded_pairs = npairs > 0;
  return MAGNUS_OK;
}

// Row mapping of the single-state CSR iteration for a variant code (the
// MAGNUS_CSR_VARIANT numbering; 0 = the size heuristic).
int variant_rows(int code, int64_t dim, bool two_pass = false) {
  switch (code) {
    // (nonzero streaming, us per iteration: 65,536 rows of 6 entries 9.6, direct 12.0,
    // wave tiles 13.0; 131,071 rows 18.1, 22.1, 19.2)
    case 1: return dim >= 65536 ? 64 : magnus::kRowsDirect + 32;
    case 2: return magnus::kRowLane;
    case 3: return -32;
    case 4: return -128;
    case 5: return magnus::kWaveTile + 8;
    case 6: return magnus::kWaveTile + 16;
    case 7: return magnus::kStreamTile;
    // Measured, us per iteration with the stop test (made by the iteration on
    // grids of at most csr2_fuse_grid workgroups, else by a decide kernel after
    // it), random terms.  Eight lanes per row (direct) against a row per lane in
    // blocks of 32 or 64 rows, 6 / 24 / 38 entries a row: 20,000 rows
    // 6.1 / 8.0 / 10.2 against 6.9 / 8.2 / 10.5; chains of 13 and 14 sites
    // 5.2 / 5.9 against 6.3 / 6.8.  From 28,672 to 49,152 rows the blocks of 64
    // rows fill the chip in one round, three to a CU: 33,000 rows 8.6 / 10.6 / 14.6
    // (direct) against 7.3 / 10.1 / 15.3, 49,152 rows 10.4 / 14.5 / 20.9 against
    // 8.5 / 12.9 / 18.3.  Past them direct again: 50,021 rows 11.1 / 15.7 / 22.2
    // against 11.7 / 17.2 / 24.8, 65,536 rows 12.0 / 18.0 / 24.9 against
    // 13.0 / 20.3 / 26.9 with wave tiles of 16 rows, but two passes per iteration
    // (a commutator applied to vectors) on spin models 23.9 against 22.5.  Past
    // 65,536 rows the wave tiles: 70,000 rows 14.3 / 21.9 / 30.3 (direct) against
    // 14.1 / 21.4 / 28.1, 90,000 16.4 / 24.6 / 35.3 against 14.8 / 24.6 / 33.2,
    // 131,071 22.1 / 34.2 / 49.0 against 19.2 / 34.9 / 46.5.  Streamed tiles from
    // 2^17 rows on (at 131,071 rows 19.5 / 27.9 / 43.5).
    default:
      return dim >= 131072                        ? magnus::kStreamTile
             : dim >= (two_pass ? 65536 : 65537) ? magnus::kWaveTile + 16
             : dim > 49152                        ? magnus::kRowsDirect + 32
             : dim >= 28672                       ? -64
                                                  : magnus::kRowsDirect + 32;
  }
}

int rows_per_block(const magnus_ctx* ctx, const magnus_hamiltonian* h, bool two_pass = false) {
  if (ctx->csr_variant) return variant_rows(ctx->csr_variant, h->H1.dim, two_pass);
  auto it = ctx->tuned_variant.find({(const void*)h->H1.row_ptr, h->H1.dim});
  return variant_rows(it == ctx->tuned_variant.end() ? 0 : it->second, h->H1.dim, two_pass);
}

// Tuned dense choices (the defaults until magnus_autotune ran on these terms).
int dense_rpw(const magnus_ctx* ctx, const magnus_hamiltonian* h) {
  if (ctx->dense_rpw_env > 0) return ctx->dense_rpw_env;
  auto it = ctx->tuned_dense_rpw.find({h->H1.val, h->H1.dim});
  return it == ctx->tuned_dense_rpw.end() ? 2 : it->second;
}
// Untuned FP64-MFMA tile: the LDS-DMA tiles, 64 x 64 once its grid has a
// workgroup for every compute unit, else 32 x 64.  Measured (autotuner, us per
// launch, 32 x 64 / 64 x 64): 512 x 16 states 39.5 / 63.4, 1024 x 128 78.9 /
// 126.6, 2048 x 256 156.0 / 245.6, 4096 x 128 310.4 / 488.0, 4096 x 256
// 536.8 / 482.9, 8192 x 64 580.2 / 945.6, 8192 x 256 2,060.6 / 1,908.8; the
// register-staged tiles were slower at every one of these shapes.
int mfma_tile(const magnus_ctx* ctx, const magnus_hamiltonian* h, int B) {
  if (ctx->mfma_tile_env >= 0) return ctx->mfma_tile_env;
  auto it = ctx->tuned_mfma.find({h->H1.val, h->H1.dim});
  if (it != ctx->tuned_mfma.end()) return it->second;
  const long long blocks = (h->H1.dim + 63) / 64 * ((B + 63) / 64);
  return blocks >= 256 ? 6 : 5;
}

// Workgroups per block of that tile (1: the tile as it is), whose shares and
// norm partials (two per state and 16 rows) must fit the workspace.
int mfma_split(const magnus_ctx* ctx, int dim, int B, int tile) {
  if ((size_t)magnus::dense_mfma_row_blocks(dim, 2) * (size_t)B * 2 > ctx->npartials) return 1;
  return magnus::dense_mfma_split(dim, B, tile, ctx->split_entries);
}

hipEvent_t next_event(magnus_ctx* ctx) {
  if (ctx->pool_used == ctx->pool.size()) {
    hipEvent_t e;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    ctx->pool.push_back(e);
  }
  return ctx->pool[ctx->pool_used++];
}

// Launch f() on stream s, bracketed by events when the context records timings.
template <class F>
hipError_t timed(magnus_ctx* ctx, int kind, hipStream_t s, F f) {
  if (!ctx->timing) return f();
  if (ctx->timing_seq[kind]++ % ctx->timing != 0) return f();
  hipEvent_t a = next_event(ctx), b = next_event(ctx);
  if (!a || !b) return hipErrorOutOfMemory;
  hipError_t e = hipEventRecord(a, s);
  if (e == hipSuccess) e = f();
  if (e == hipSuccess) e = hipEventRecord(b, s);
  if (e == hipSuccess) ctx->records.emplace_back(kind, a, b);
  return e;
}

// The last fused iteration's partials are checked for non-finite norms by a
// small kernel, enqueued before anything else writes the partials buffer or
// the control slots (another kind of launch, the end of the call).
int flush_fused_check(magnus_ctx* ctx, hipStream_t s) {
  if (!ctx->fz_pending) return MAGNUS_OK;
  ctx->fz_pending = false;
  HIP_TRY(magnus::launch_leja_final_check(ctx->fz_last, s));
  return MAGNUS_OK;
}

// Likewise for every problem's last launch of pairs (at the end of a group of states, and of the call).
int flush_pair_check(magnus_ctx* ctx, hipStream_t s) {
  if (!ctx->pair_pending) return MAGNUS_OK;
  ctx->pair_pending = false;
  HIP_TRY(magnus::launch_coded_pairs_check(ctx->pair_last, s));
  return MAGNUS_OK;
}

// Launch one Leja iteration (both passes for a commutator exponent).
// Stop test of iteration i: fused into the iteration kernel on grids of at
// most kFuseMaxGrid workgroups (every workgroup reduces iteration i-1's
// partials, which alternate between two halves of the partials buffer),
// else a decide kernel after each iteration.  Sets a->fused.
int setup_stop_test(magnus_ctx* ctx, const ExpPlan& P, int i, int grid, IterArgs* a, hipStream_t s,
                    int limit = magnus::kFuseMaxGrid) {
  a->iter = i;
  a->fused = 0;
  if (!ctx->fuse || grid > limit) return flush_fused_check(ctx, s);
  const size_t half = 2 * (size_t)ctx->max_grid;
  a->fused = 1;
  a->partials = ctx->partials + (size_t)(i & 1) * half;
  a->prev_partials = ctx->partials + (size_t)((i - 1) & 1) * half;
  a->prev_grid = grid;
  a->prev_dabs = i >= 2 ? std::abs(P.d[i - 1]) : 0.0;
  // the call's last fused iteration is checked for non-finite norms at its end
  ctx->fz_last = *a;
  ctx->fz_last.iter = i + 1;
  ctx->fz_last.prev_partials = a->partials;
  ctx->fz_pending = true;
  return MAGNUS_OK;
}

// One Leja iteration of Method M6 on CSR terms, the exponent's nested
// commutators applied to vectors by products with H1, H2 and K alone, or with
// P1 and P2 too.
int m6_csr_iteration(magnus_ctx* ctx, const ExpOp& op, const ExpPlan& P, int i, IterArgs& a, hipStream_t s) {
  const magnus_hamiltonian* h = op.h;
  const int dim = (int)h->H1.dim;
  const bool coded = ctx->coded_h == h && ctx->coded_terms.n == 3;
  magnus::CodeTerms T =
      coded ? ctx->coded_terms
            : magnus::CodeTerms{3, {csr_dev(h->H1), csr_dev(h->H2), CsrDev{ctx->kc_rp, ctx->kc_ci, ctx->kc_val}}};
  magnus::M6Args M{};
  for (int k = 0; k < 10; ++k) M.c[k] = op.m6c[k];
  for (int k = 0; k < 4; ++k) M.a[k] = ctx->pm_ws + (size_t)k * (size_t)ctx->pm_ws_dim;
  for (int k = 0; k < 3; ++k) M.v[k] = ctx->pm_ws + (size_t)(4 + k) * (size_t)ctx->pm_ws_dim;
  M.scale = P.scale;
  const int grid = coded ? magnus::code_grid(dim, ctx->coded.rows) : magnus::m6_grid(dim);
  if (int rc = setup_stop_test(ctx, P, i, grid, &a, s)) return rc;
  const bool two = !coded && m6_two_passes(ctx, h);
  if (two)
    for (int k = 0; k < 2; ++k) T.m[T.n++] = CsrDev{ctx->pm_rp[k], ctx->pm_ci[k], ctx->pm_val[k]};
  auto pass = [&](int stage) {
    return coded ? magnus::launch_coded_m6(stage, T, dim, ctx->coded, M, a, s)
           : two ? magnus::launch_m6_two(stage, T, dim, M, a, s)
                 : magnus::launch_m6(stage, T, dim, M, a, s);
  };
  HIP_TRY(pass(0));
  if (!two) HIP_TRY(pass(1));
  HIP_TRY(timed(ctx, MAGNUS_KERNEL_CSR_LEJA, s, [&] { return pass(two ? 1 : 2); }));
  if (!a.fused) HIP_TRY(magnus::launch_leja_decide(a, grid, s));
  return MAGNUS_OK;
}

// Table column of one iteration launch in a captured step (graph replay).
struct TableRef {
  const magnus::IterCoef* col;  // record of this iteration in step 0
  int stride;                   // records per step
  const int* step;              // device step counter
};

// One Leja iteration on the coded terms (both passes for a commutator applied to vectors).
int launch_coded(magnus_ctx* ctx, const ExpOp& op, const ExpPlan& P, int i, const double2* win, IterArgs a,
                 hipStream_t s) {
  const int dim = (int)op.h->H1.dim;
  const int grid = magnus::code_grid(dim, ctx->coded.rows);
  a.x1 = a.x2 = win;
  if (int rc = setup_stop_test(ctx, P, i, grid, &a, s)) return rc;
  const bool fused = a.fused;
  magnus::CodeTerms T = ctx->coded_terms;
  const bool with_k = op.kappa != 0.0 && T.n == 3;
  if (!with_k) T.n = 2;
  if (op.kappa != 0.0 && !with_k) {
    // as on the streamed tiles: pass 1 writes U = a1 w + i k H2 w and V = a2 w - i k H1 w, pass 2 is H1 U + H2 V
    IterArgs p1 = a;
    p1.wout = ctx->vec(kU);
    p1.pacc = ctx->vec(kV);
    HIP_TRY(timed(ctx, MAGNUS_KERNEL_CSR_SPLIT, s, [&] {
      return magnus::launch_coded_iter(magnus::kSplitComm, T, dim, ctx->coded, p1, 0.0, s);
    }));
    if (fused) {
      a.fused = 0;
      a.check_stop = 1;
    }
    a.x1 = ctx->vec(kU);
    a.x2 = ctx->vec(kV);
    a.a1 = a.a2 = 1.0;
    a.unit_a = 1;
  }
  const int kind = op.kappa == 0.0 ? MAGNUS_KERNEL_CSR_LEJA : with_k ? MAGNUS_KERNEL_CSR_LEJA3 : MAGNUS_KERNEL_CSR_COMM;
  HIP_TRY(timed(ctx, kind, s, [&] {
    return magnus::launch_coded_iter(magnus::kLeja, T, dim, ctx->coded, a, P.scale * op.kappa, s);
  }));
  if (!fused) HIP_TRY(magnus::launch_leja_decide(a, grid, s));
  return MAGNUS_OK;
}

int launch_iteration(magnus_ctx* ctx, const ExpOp& op, const ExpPlan& P, int i, const double2* win,
                     double2* wout, double2* pacc, double tol_sub, int early, hipStream_t s,
                     const TableRef* tab = nullptr) {
  const magnus_hamiltonian* h = op.h;
  const int dim = (int)h->H1.dim;
  const auto& xi = magnus::leja_points();
  IterArgs a{};
  if (tab) {
    a.coef = tab->col;
    a.coef_stride = tab->stride;
    a.step = tab->step;
  }
  a.slot = ctx->slots;
  a.partials = ctx->partials;
  a.a1 = P.scale * op.a;
  a.a2 = P.scale * op.b;
  a.kap = P.scale * op.kappa;
  a.sigma = P.scale * P.c + xi[i - 1];
  a.d = make_double2(P.d[i].real(), P.d[i].imag());
  a.d0 = make_double2(P.d[0].real(), P.d[0].imag());
  a.dabs = std::abs(P.d[i]);
  a.d0abs = std::abs(P.d[0]);
  a.tol = tol_sub;
  a.early = early;
  a.first = (i == 1);
  a.check_stop = (i != 1);
  a.iter = i;
  a.wcur = win;
  a.wout = wout;
  a.pacc = pacc;
  if (op.m6c) return m6_csr_iteration(ctx, op, P, i, a, s);
  if (h->H1.format == MAGNUS_DENSE) {
    if (op.kappa != 0.0) return fail(MAGNUS_EINVAL, "dense commutator exponents run assembled");
    a.x1 = win;
    a.x2 = win;
    const int rpw = dense_rpw(ctx, h);
    const int grid = magnus::dense2_grid(dim);
    if (int rc = setup_stop_test(ctx, P, i, grid, &a, s)) return rc;
    const bool fused = a.fused;
    HIP_TRY(timed(ctx, MAGNUS_KERNEL_DENSE_LEJA, s, [&] {
      if (op.fuse_assembly && i == 1) {
        const magnus::DenseAssembly D{reinterpret_cast<const double2*>(h->H1.val),
                                      reinterpret_cast<const double2*>(h->H2.val),
                                      op.fK,
                                      h->H1.ld,
                                      op.fa,
                                      op.fb,
                                      op.fk,
                                      op.fuse_out};
        return magnus::launch_dense_assemble_iter(D, dim, a, s, rpw);
      }
      if (op.assembled) return magnus::launch_dense2_iter(op.assembled, nullptr, dim, dim, a, s, rpw);
      return magnus::launch_dense2_iter(reinterpret_cast<const double2*>(h->H1.val),
                                        reinterpret_cast<const double2*>(h->H2.val), dim, h->H1.ld, a, s, rpw);
    }));
    if (!fused) HIP_TRY(magnus::launch_leja_decide(a, grid, s));
    return MAGNUS_OK;
  }
  if (ctx->coded_h == h) return launch_coded(ctx, op, P, i, win, a, s);
  CsrDev t1{h->H1.row_ptr, h->H1.col_idx, reinterpret_cast<const double2*>(h->H1.val)};
  CsrDev t2{h->H2.row_ptr, h->H2.col_idx, reinterpret_cast<const double2*>(h->H2.val)};
  if (op.kappa == 0.0) {
    a.x1 = win;
    a.x2 = win;
    const int rpb = rows_per_block(ctx, h);
    const int grid = magnus::csr2_grid(dim, rpb);
    if (int rc = setup_stop_test(ctx, P, i, grid, &a, s, magnus::csr2_fuse_grid(rpb))) return rc;
    const bool fused = a.fused;
    HIP_TRY(timed(ctx, MAGNUS_KERNEL_CSR_LEJA, s,
                  [&] { return magnus::launch_csr2_iter(magnus::kLeja, t1, t2, dim, a, rpb, s); }));
    if (!fused) HIP_TRY(magnus::launch_leja_decide(a, grid, s));
    return MAGNUS_OK;
  }
  if (csr_comm_ready(ctx, h)) {
    // assembled commutator: one pass over H1, H2 and K
    CsrDev t3{ctx->kc_rp, ctx->kc_ci, ctx->kc_val};
    a.x1 = win;
    a.x2 = win;
    const int rpb = magnus::csr3_rows(dim, rows_per_block(ctx, h));
    const int grid = magnus::csr2_grid(dim, rpb);
    if (int rc = setup_stop_test(ctx, P, i, grid, &a, s, magnus::csr2_fuse_grid(rpb))) return rc;
    const bool fused = a.fused;
    HIP_TRY(timed(ctx, MAGNUS_KERNEL_CSR_LEJA3, s,
                  [&] { return magnus::launch_csr3_iter(t1, t2, t3, dim, a, P.scale * op.kappa, rpb, s); }));
    if (!fused) HIP_TRY(magnus::launch_leja_decide(a, grid, s));
    return MAGNUS_OK;
  }
  // Commutator exponents take two passes per iteration.  The first pass
  // makes the stop test (fused or not); with the fused test the second pass
  // only reads the verdict the first one recorded, and it writes the
  // partials the next iteration's first pass reduces.
  double2* U = ctx->vec(kU);
  double2* V = ctx->vec(kV);
  const int rpb = rows_per_block(ctx, h, true);
  const int grid = magnus::csr2_grid(dim, rpb);
  if (int rc = setup_stop_test(ctx, P, i, grid, &a, s, magnus::csr2_fuse_grid(rpb))) return rc;
  const bool fused = a.fused;
  IterArgs p1 = a;
  p1.x1 = win;
  p1.x2 = win;
  p1.wout = U;
  p1.pacc = V;
  if (fused) {
    a.fused = 0;
    a.check_stop = 1;
  }
  if (rpb == magnus::kStreamTile) {
    // streamed commutator: pass 1 writes U = a1 w + i k H2 w and V = a2 w - i k H1 w,
    // pass 2 is the two-term iteration on H1 U + H2 V
    HIP_TRY(timed(ctx, MAGNUS_KERNEL_CSR_SPLIT, s,
                  [&] { return magnus::launch_csr2_iter(magnus::kSplitComm, t1, t2, dim, p1, rpb, s); }));
    a.x1 = U;
    a.x2 = V;
    a.a1 = 1.0;
    a.a2 = 1.0;
    a.unit_a = 1;
    HIP_TRY(timed(ctx, MAGNUS_KERNEL_CSR_COMM, s,
                  [&] { return magnus::launch_csr2_iter(magnus::kLeja, t1, t2, dim, a, rpb, s); }));
    if (!fused) HIP_TRY(magnus::launch_leja_decide(a, grid, s));
    return MAGNUS_OK;
  }
  // commutator: pass 1 writes U = H1 w, V = H2 w; pass 2 applies H1 V and H2 U
  HIP_TRY(timed(ctx, MAGNUS_KERNEL_CSR_SPLIT, s,
                [&] { return magnus::launch_csr2_iter(magnus::kSplit, t1, t2, dim, p1, rpb, s); }));
  a.x1 = V;
  a.x2 = U;
  HIP_TRY(timed(ctx, MAGNUS_KERNEL_CSR_COMM, s,
                [&] { return magnus::launch_csr2_iter(magnus::kLejaComm, t1, t2, dim, a, rpb, s); }));
  if (!fused) HIP_TRY(magnus::launch_leja_decide(a, grid, s));
  return MAGNUS_OK;
}

// The launches of one planned exponential: P.lp.s substeps of P.lp.m
// iterations, the Newton sums in kS0/kS1 (or dst), w in kA/kB.  With a table
// (capture of a replayed step) iteration i of substep sub reads record
// tab->col + sub * m + i - 1 of the step.
int enqueue_exponential(magnus_ctx* ctx, const ExpOp& it, const ExpPlan& P, const double2* src, double2* dst,
                        double tol_sub, int early, const TableRef* tab, hipStream_t s) {
  const int64_t dim = it.h->H1.dim;
  const int m = P.lp.m, ns = P.lp.s;
  const double2* cur = src;
  ExpOp op = it;  // a fused assembly happens in the first iteration only
  for (int sub = 0; sub < ns; ++sub) {
    const bool last = (sub == ns - 1);
    double2* Pbuf;
    if (last && dst != cur) Pbuf = dst;
    else Pbuf = (cur == ctx->vec(kS0)) ? ctx->vec(kS1) : ctx->vec(kS0);
    for (int i = 1; i <= m; ++i) {
      const double2* win = (i == 1) ? cur : ((i - 1) % 2 == 1 ? ctx->vec(kA) : ctx->vec(kB));
      double2* wout = (i % 2 == 1) ? ctx->vec(kA) : ctx->vec(kB);
      TableRef t{};
      if (tab) t = TableRef{tab->col + (size_t)sub * m + (i - 1), tab->stride, tab->step};
      int rc = launch_iteration(ctx, op, P, i, win, wout, Pbuf, tol_sub, early, s, tab ? &t : nullptr);
      if (rc) return rc;
      op.fuse_assembly = false;
    }
    cur = Pbuf;
  }
  if (cur != dst) HIP_TRY(magnus::launch_copy(cur, dst, dim, s));
  return MAGNUS_OK;
}

// dst = exp(-i tau (a H1 + b H2 + kappa K)) src for one state.  dst may equal
// src and may be kS2; it must not be another workspace vector.
int run_exponential(magnus_ctx* ctx, const ExpOp& op, double tau, const double2* src, double2* dst,
                    double tol_e, const magnus_leja_opts* o, Acc* acc, hipStream_t s) {
  const int64_t dim = op.h->H1.dim;
  if (tau == 0.0) {
    if (src != dst) HIP_TRY(magnus::launch_copy(src, dst, dim, s));
    acc->exponentials += 1;
    return MAGNUS_OK;
  }
  double lo = op.lo, hi = op.hi;
  if (!op.has_interval)
    magnus::weyl_interval(op.a, op.h->H1.lam_min, op.h->H1.lam_max, op.b, op.h->H2.lam_min, op.h->H2.lam_max,
                          op.kappa, op.h->k_min, op.h->k_max, &lo, &hi);
  ExpPlan P;
  if (!magnus::plan_exponential(tau, lo, hi, tol_e, o->max_degree, o->max_substeps, &P))
    return fail(MAGNUS_ENOCONV, "no degree <= %d with <= %d substeps reaches tol %g (theta %g)",
                o->max_degree, o->max_substeps, tol_e, 0.5 * std::fabs(tau) * 0.5 * (hi - lo));
  const int m = P.lp.m, ns = P.lp.s;
  const double tol_sub = tol_e / (2.0 * ns);
  // Dense terms: assemble the exponent once (48 dim^2 bytes) when that is
  // cheaper than reading both terms in every iteration (16 dim^2 bytes more
  // each), and always for a commutator exponent (K itself is assembled).
  ExpOp it = op;
  if (!op.assembled && op.h->H1.format == MAGNUS_DENSE &&
      (op.kappa != 0.0 || (ctx->assembled_dim >= dim && m * ns >= 4))) {
    if (op.kappa != 0.0 && !dense_comm_ready(ctx, op.h))
      return fail(MAGNUS_EINVAL, "dense commutator exponents need magnus_dense_commutator for this pair of terms");
    if (ctx->assembled_dim < dim) return fail(MAGNUS_ENOMEM, "no assembly buffer (magnus_reserve_dense)");
    it = ExpOp{op.h, 1.0, 0.0, 0.0, ctx->assembled};
    if (ctx->fuse_assembly) {  // assembled by the first iteration as it goes
      it.fuse_assembly = true;
      it.fa = op.a;
      it.fb = op.b;
      it.fk = op.kappa;
      it.fK = op.kappa != 0.0 ? ctx->comm : nullptr;
      it.fuse_out = ctx->assembled;
    } else {
      HIP_TRY(magnus::launch_dense_assemble(reinterpret_cast<const double2*>(op.h->H1.val),
                                            reinterpret_cast<const double2*>(op.h->H2.val), op.h->H1.ld, (int)dim,
                                            op.a, op.b, op.kappa != 0.0 ? ctx->comm : nullptr, op.kappa,
                                            ctx->assembled, s));
    }
  }
  int rc = enqueue_exponential(ctx, it, P, src, dst, tol_sub, o->early_termination, nullptr, s);
  if (rc) return rc;
  acc->exponentials += 1;
  acc->substeps += ns;
  acc->planned += (int64_t)m * ns;
  acc->max_m = std::max(acc->max_m, m);
  acc->max_s = std::max(acc->max_s, ns);
  acc->max_bound = std::max(acc->max_bound, P.lp.bound);
  return MAGNUS_OK;
}

int begin_call(magnus_ctx* ctx, hipStream_t s) {
  HIP_TRY(hipSetDevice(ctx->device));
  ctx->sticky_status = 0;
  ctx->fz_pending = false;
  ctx->pair_pending = false;
  ctx->coded_h = nullptr;
  ctx->coded_pairs = false;
  HIP_TRY(magnus::launch_slot_reset(ctx->slots, ctx->nslots, s));
  return MAGNUS_OK;
}

// Sum of the per-state counters and the union of the status bits.
int read_slots(magnus_ctx* ctx, hipStream_t s, long long* iters, int* status) {
  std::vector<Slot> hs(ctx->nslots);
  HIP_TRY(hipMemcpyAsync(hs.data(), ctx->slots, sizeof(Slot) * hs.size(), hipMemcpyDeviceToHost, s));
  HIP_TRY(hipStreamSynchronize(s));
  *iters = 0;
  *status = 0;
  for (const Slot& x : hs) {
    *iters += x.iters_total;
    *status |= x.status;
  }
  return MAGNUS_OK;
}

// The slots as they are here in the stream, for await_slots; what is enqueued
// between the two runs while the host waits for what came before.  Without pinned
// memory the wait is here.
int copy_slots(magnus_ctx* ctx, hipStream_t s) {
  if (!ctx->seen && hipHostMalloc(&ctx->seen, sizeof(Slot) * ctx->nslots, 0) != hipSuccess) {
    (void)hipGetLastError();
    ctx->seen = nullptr;
    long long iters = 0;
    int status = 0;
    if (int rc = read_slots(ctx, s, &iters, &status)) return rc;
    return status & 1 ? fail(MAGNUS_ENAN, "non-finite vector norm met during the call") : MAGNUS_OK;
  }
  if (!ctx->seen_at) HIP_TRY(hipEventCreateWithFlags(&ctx->seen_at, hipEventDisableTiming));
  HIP_TRY(hipMemcpyAsync(ctx->seen, ctx->slots, sizeof(Slot) * ctx->nslots, hipMemcpyDeviceToHost, s));
  HIP_TRY(hipEventRecord(ctx->seen_at, s));
  return MAGNUS_OK;
}

int await_slots(magnus_ctx* ctx) {
  if (!ctx->seen) return MAGNUS_OK;
  HIP_TRY(hipEventSynchronize(ctx->seen_at));
  for (int k = 0; k < ctx->nslots; ++k)
    if (ctx->seen[k].status & 1) return fail(MAGNUS_ENAN, "non-finite vector norm met during the call");
  return MAGNUS_OK;
}

int end_call(magnus_ctx* ctx, const Acc& acc, double tol_e, magnus_stats* st, hipStream_t s) {
  if (int rc = flush_fused_check(ctx, s)) return rc;
  if (int rc = flush_pair_check(ctx, s)) return rc;
  if (!st) return MAGNUS_OK;
  long long iters = 0;
  int status = 0;
  int rc = read_slots(ctx, s, &iters, &status);
  if (rc) return rc;
  st->exponentials = acc.exponentials;
  st->substeps = acc.substeps;
  st->planned_iters = acc.planned;
  st->iters = iters + acc.extra_iters;
  status |= ctx->sticky_status;
  st->hv_products = st->iters * acc.products_per_iter;
  st->max_degree_used = acc.max_m;
  st->max_substeps_used = acc.max_s;
  st->max_err_bound = acc.max_bound;
  st->tol_per_exp = tol_e;
  if (status & 1) return fail(MAGNUS_ENAN, "non-finite vector norm met during the call");
  return MAGNUS_OK;
}

double per_exp_tol(const magnus_leja_opts* o, int64_t exps_per_state) {
  if (o->tol_mode == 1 && exps_per_state > 0) return o->tol / (double)exps_per_state;
  return o->tol;
}

// H2 coefficient of exponential k of a product-of-exponentials step.
double scheme_b(const magnus::Scheme& S, int k, const double* f) {
  double b = 0.0;
  for (int j = 0; j < S.q; ++j) b += S.w[k][j] * f[j];
  return b;
}

// One step of a product-of-exponentials method (Cf4, Cf4:3, M2) on one state,
// f = the step's field samples; the factors act in the order of the scheme
// (for Cf4 the right factor exp(tau(alpha2 A1 + alpha1 A2)) first).
int cf_state(magnus_ctx* ctx, const magnus_hamiltonian* h, const magnus::Scheme& S, double tau, const double* f,
             const double2* in, double2* out, double tol_e, const magnus_leja_opts* o, Acc* acc, hipStream_t s) {
  double2* mids[2] = {ctx->vec(kS2), ctx->vec(kU)};
  const double2* src = in;
  for (int k = 0; k < S.nexp; ++k) {
    double2* dst = (k == S.nexp - 1) ? out : mids[k & 1];
    int rc = run_exponential(ctx, ExpOp{h, S.rho[k], scheme_b(S, k, f), 0.0}, tau, src, dst, tol_e, o, acc, s);
    if (rc) return rc;
    src = dst;
  }
  return MAGNUS_OK;
}

// One step of Method M4 on one state: exp(-i tau (H1 + fbar H2 + kappa K)).
int m4_state(magnus_ctx* ctx, const magnus_hamiltonian* h, double tau, double f1, double f2,
             const double2* in, double2* out, double tol_e, const magnus_leja_opts* o, Acc* acc,
             hipStream_t s) {
  const double fbar = 0.5 * (f1 + f2);
  const double kappa = magnus::kSqrt3 * tau * (f2 - f1) / 12.0;
  return run_exponential(ctx, ExpOp{h, 1.0, fbar, kappa}, tau, in, out, tol_e, o, acc, s);
}

// Whether the context holds the M6 commutators of this pair of dense terms.
bool dense_m6_ready(const magnus_ctx* ctx, const magnus_hamiltonian* h) {
  return ctx->m6_ready && dense_comm_ready(ctx, h);
}

// One step of Method M6 on one state, dense terms.  With A_j = -i(H1 + f_j H2)
// the exponent's B_1 = -i tau Hm (Hm = H1 + f_2 H2) and B_2 = -i b2 H2,
// B_3 = -i b3 H2 with b2 = sqrt(15)/3 tau (f3 - f1), b3 = 10/3 tau (f3 - 2 f2 + f1).
// Expanding the nested commutators of the M6 exponent in H1, H2 makes it a
// linear combination, with step-dependent scalars, of ten fixed Hermitian
// matrices: H1, H2, K = i[H1,H2], P_a = -i[H_a,K], U_ab = i[H_a,P_b]
// (U_12 = U_21 by the Jacobi identity) and R_a = -i[K,P_a].  The step
// assembles -i tau (sum_t c_t M_t) once and runs one Leja exponential on it.
int m6_state(magnus_ctx* ctx, const magnus_hamiltonian* h, double tau, const double* f, const double2* in,
             double2* out, double tol_e, const magnus_leja_opts* o, Acc* acc, hipStream_t s) {
  const int64_t dim = h->H1.dim;
  const double f1 = f[0], f2 = f[1], f3 = f[2];
  const double r15 = 3.8729833462074168852;
  const double b2 = r15 / 3.0 * tau * (f3 - f1);
  const double b3 = 10.0 / 3.0 * tau * (f3 - 2.0 * f2 + f1);
  // coefficients of H1, H2, K, P1, P2, U11, U12, U22, R1, R2 in the exponent / (-i tau)
  const double c[10] = {1.0,
                        f2 + b3 / (12.0 * tau),
                        b2 / 12.0,
                        -tau * b3 / 360.0,
                        (-(2.0 * tau * b3 * f2 / 3.0) - b3 * b3 / 30.0 + b2 * b2) / 240.0,
                        tau * tau * b2 / 720.0,
                        (2.0 * tau * tau * b2 * f2 / 3.0 + tau * b2 * b3 / 60.0) / 240.0,
                        (tau * tau * b2 * f2 * f2 / 3.0 + tau * b2 * b3 * f2 / 60.0) / 240.0,
                        -tau * tau * b2 * b2 / 14400.0,
                        -tau * tau * b2 * b2 * f2 / 14400.0};
  double mlo[10] = {h->H1.lam_min, h->H2.lam_min, h->k_min, ctx->m6_lo[0], ctx->m6_lo[1], ctx->m6_lo[2],
                    ctx->m6_lo[3], ctx->m6_lo[4], ctx->m6_lo[5], ctx->m6_lo[6]};
  double mhi[10] = {h->H1.lam_max, h->H2.lam_max, h->k_max, ctx->m6_hi[0], ctx->m6_hi[1], ctx->m6_hi[2],
                    ctx->m6_hi[3], ctx->m6_hi[4], ctx->m6_hi[5], ctx->m6_hi[6]};
  if (h->H1.format == MAGNUS_CSR) {
    // P_a from their Gershgorin discs; the nested commutators i[A, B] are
    // applied matrix-free, enclosed by +-2 rho(A) rho(B) (rho: the larger end
    // of an enclosure in absolute value)
    auto rho = [](double lo_, double hi_) { return std::fmax(std::fabs(lo_), std::fabs(hi_)); };
    const double rh1 = rho(h->H1.lam_min, h->H1.lam_max), rh2 = rho(h->H2.lam_min, h->H2.lam_max);
    const double rk = rho(h->k_min, h->k_max);
    const double rp1 = rho(ctx->pm_lo[0], ctx->pm_hi[0]), rp2 = rho(ctx->pm_lo[1], ctx->pm_hi[1]);
    const double nested[5] = {2 * rh1 * rp1, 2 * rh1 * rp2, 2 * rh2 * rp2, 2 * rk * rp1, 2 * rk * rp2};
    mlo[3] = ctx->pm_lo[0];
    mhi[3] = ctx->pm_hi[0];
    mlo[4] = ctx->pm_lo[1];
    mhi[4] = ctx->pm_hi[1];
    for (int t = 0; t < 5; ++t) {
      mlo[5 + t] = -nested[t];
      mhi[5 + t] = nested[t];
    }
  }
  // Weyl: the spectrum of a sum of Hermitian matrices lies in the sum of their enclosures
  double lo = 0.0, hi = 0.0;
  for (int t = 0; t < 10; ++t) {
    lo += std::fmin(c[t] * mlo[t], c[t] * mhi[t]);
    hi += std::fmax(c[t] * mlo[t], c[t] * mhi[t]);
  }
  if (h->H1.format == MAGNUS_CSR) {
    ExpOp op{h, 0.0, 0.0, 0.0};
    op.has_interval = true;
    op.lo = lo;
    op.hi = hi;
    op.m6c = c;
    return run_exponential(ctx, op, tau, in, out, tol_e, o, acc, s);
  }
  magnus::AssembleTerms T{};
  T.nterms = 10;
  for (int t = 0; t < 10; ++t) {
    T.c[t] = c[t];
    if (t < 2) {
      T.m[t] = reinterpret_cast<const double2*>(t == 0 ? h->H1.val : h->H2.val);
      T.ld[t] = h->H1.ld;
    } else {
      T.m[t] = t == 2 ? ctx->comm : ctx->m6 + (size_t)(t - 3) * (size_t)ctx->m6_dim * (size_t)ctx->m6_dim;
      T.ld[t] = dim;
    }
  }
  if (ctx->assembled_dim < dim) return fail(MAGNUS_ENOMEM, "no assembly buffer (magnus_reserve_dense)");
  HIP_TRY(magnus::launch_assemble_terms(T, (int)dim, ctx->assembled, s));
  ExpOp op{h, 1.0, 0.0, 0.0, ctx->assembled};
  op.has_interval = true;
  op.lo = lo;
  op.hi = hi;
  return run_exponential(ctx, op, tau, in, out, tol_e, o, acc, s);
}

// ---------------------------------------------------------------------------
// Several states per iteration (interleaved workspace, one CSR pass for all).
// ---------------------------------------------------------------------------

// One exponential of a group of B states: exp(-i tau (a_b H1 + b_b H2)) for
// state b.  All states share the substep count s and run max_b m_b
// iterations; a state whose own degree m_b is smaller gets d_i = 0 beyond it.
struct MultiExp {
  int B = 0, s = 1, m = 1;
  int dense_terms = 0;           // dense: 1 (assembled, with acoef/bcoef below) or 2
  double ca = 0.0, cb = 0.0;     // coefficients of the assembled exponent
  size_t table_off = 0;          // first ColParam of this exponential ([i-1][b])
  double tau = 0.0;
  int frechet = 0;               // block vector of [[H, H2], [0, H]] (B == 2)
  const double2* src = nullptr;  // interleaved, dim * B
  double2* dst = nullptr;
};

int plan_multi(const magnus_hamiltonian* h, const double* acoef, const double* bcoef, int B, double tau,
               double tol_e, const magnus_leja_opts* o, int frechet, std::vector<ColParam>* table,
               MultiExp* out, Acc* acc, bool assembled = false) {
  std::vector<double> lo(B), hi(B);
  int s = 1;
  for (int b = 0; b < B; ++b) {
    magnus::weyl_interval(acoef[b], h->H1.lam_min, h->H1.lam_max, bcoef[b], h->H2.lam_min, h->H2.lam_max, 0.0, 0.0,
                          0.0, &lo[b], &hi[b]);
    if (b > 0 && lo[b] == lo[b - 1] && hi[b] == hi[b - 1]) continue;  // planned as the state before
    magnus::LejaPlan t;
    if (!magnus::plan_substeps(tau, lo[b], hi[b], tol_e, o->max_degree, o->max_substeps, &t))
      return fail(MAGNUS_ENOCONV, "no degree <= %d with <= %d substeps reaches tol %g", o->max_degree,
                  o->max_substeps, tol_e);
    s = std::max(s, t.s);
  }
  std::vector<ExpPlan> P(B);
  int m = 1;
  double worst = 0.0;
  for (int b = 0; b < B; ++b) {
    const double coupling =
        frechet ? std::fmax(std::fabs(h->H2.lam_min), std::fabs(h->H2.lam_max)) : 0.0;
    if (b > 0 && lo[b] == lo[b - 1] && hi[b] == hi[b - 1]) P[b] = P[b - 1];
    else if (!magnus::plan_exponential_fixed_s(tau, lo[b], hi[b], tol_e, s, o->max_degree, &P[b], coupling))
      return fail(MAGNUS_ENOCONV, "no degree <= %d reaches tol %g with %d substeps", o->max_degree, tol_e, s);
    m = std::max(m, P[b].lp.m);
    worst = std::max(worst, P[b].lp.bound);
  }
  std::vector<double> d0abs(B);
  for (int b = 0; b < B; ++b) d0abs[b] = std::abs(P[b].d[0]);
  const auto& xi = magnus::leja_points();
  out->B = B;
  out->s = s;
  out->m = m;
  out->tau = tau;
  out->frechet = frechet;
  out->table_off = table->size();
  for (int i = 1; i <= m; ++i)
    for (int b = 0; b < B; ++b) {
      const ExpPlan& p = P[b];
      ColParam c{};
      c.a1 = assembled ? p.scale : p.scale * acoef[b];
      c.a2 = assembled ? 0.0 : p.scale * bcoef[b];
      c.sigma = p.scale * p.c + xi[i - 1];
      const std::complex<double> d = i <= p.lp.m ? p.d[i] : std::complex<double>(0.0, 0.0);
      c.dre = d.real();
      c.dim = d.imag();
      c.dabs = std::abs(d);
      c.d0re = p.d[0].real();
      c.d0im = p.d[0].imag();
      c.d0abs = d0abs[b];
      c.coup = frechet ? p.scale : 0.0;
      table->push_back(c);
    }
  acc->exponentials += B;
  acc->substeps += (int64_t)s * B;
  acc->planned += (int64_t)m * s * B;
  acc->max_m = std::max(acc->max_m, m);
  acc->max_s = std::max(acc->max_s, s);
  acc->max_bound = std::max(acc->max_bound, worst);
  return MAGNUS_OK;
}

int upload_table(magnus_ctx* ctx, const std::vector<ColParam>& table, hipStream_t s) {
  if (table.empty()) return MAGNUS_OK;
  if (table.size() > kTableCap) return fail(MAGNUS_ENOMEM, "parameter table of %zu entries exceeds %zu", table.size(), kTableCap);
  HIP_TRY(hipMemcpyAsync(ctx->table, table.data(), sizeof(ColParam) * table.size(), hipMemcpyHostToDevice, s));
  return MAGNUS_OK;
}

// Pairs of states of one problem on its coded terms: npairs pairs back to back
// in every buffer, w in w0 / w1, the Newton sums of substeps in s0 / s1.
struct PairWork {
  const magnus_hamiltonian* h;
  magnus::CodedDev C;
  int npairs;
  double2 *w0, *w1, *s0, *s1;
  int slot0;    // first control slot
  size_t poff;  // offset of its norm partials in a half
};

// The iterations of one planned exponential of every problem (E[q] of problem
// q), one launch per iteration for all of them.
int launch_pairs_exp(magnus_ctx* ctx, const std::vector<PairWork>& R, const std::vector<MultiExp>& E, double tol_e,
                     int early, bool frechet, hipStream_t s) {
  const size_t np = R.size();
  std::vector<const double2*> cur(np);
  std::vector<double2*> pbuf(np);
  int max_s = 1;
  size_t half = 0;
  for (size_t q = 0; q < np; ++q) {
    cur[q] = E[q].src;
    max_s = std::max(max_s, E[q].s);
    half = std::max(half, R[q].poff + 4 * (size_t)R[q].npairs * magnus::code_grid((int)R[q].h->H1.dim, R[q].C.rows));
  }
  double* base = ctx->partials + pair_partials_at(ctx);
  if (pair_partials_at(ctx) + 2 * half > ctx->npartials) return fail(MAGNUS_ENOMEM, "per-workgroup partial sums exceed the context's buffer");
  for (int sub = 0; sub < max_s; ++sub) {
    int max_m = 0;
    for (size_t q = 0; q < np; ++q) {
      if (sub >= E[q].s) continue;
      const bool last = sub == E[q].s - 1;
      if (last && E[q].dst != cur[q]) pbuf[q] = E[q].dst;
      else pbuf[q] = cur[q] == R[q].s0 ? R[q].s1 : R[q].s0;
      max_m = std::max(max_m, E[q].m);
    }
    for (int i = 1; i <= max_m; ++i) {
      magnus::PairArgs A{};
      size_t who[magnus::kMaxPairProblems];
      for (size_t q = 0; q < np; ++q) {
        if (sub >= E[q].s || i > E[q].m) continue;
        who[A.np] = q;
        magnus::PairProblem& P = A.p[A.np++];
        P.t1 = csr_dev(R[q].h->H1);
        P.t2 = csr_dev(R[q].h->H2);
        P.C = R[q].C;
        P.dim = (int)R[q].h->H1.dim;
        P.npairs = R[q].npairs;
        P.x = (i == 1) ? cur[q] : ((i - 1) % 2 == 1 ? R[q].w0 : R[q].w1);
        P.wout = (i % 2 == 1) ? R[q].w0 : R[q].w1;
        P.pacc = pbuf[q];
        P.slots = ctx->slots + R[q].slot0;
        P.partials = base + (size_t)(i & 1) * half + R[q].poff;
        P.prev_partials = base + (size_t)((i - 1) & 1) * half + R[q].poff;
        P.prm = ctx->table + E[q].table_off + (size_t)(i - 1) * E[q].B;
        P.prev = i > 1 ? P.prm - E[q].B : P.prm;
        P.first = (i == 1);
        P.iter = i;
        P.early = early;
        P.tol = tol_e / (2.0 * E[q].s);
      }
      HIP_TRY(timed(ctx, MAGNUS_KERNEL_CSR_MULTI, s, [&] { return magnus::launch_coded_pairs(frechet, A, s); }));
      // a problem with fewer iterations is not in the last launch: each keeps its own
      ctx->pair_last.np = (int)np;
      for (int k = 0; k < A.np; ++k) ctx->pair_last.p[who[k]] = A.p[k];
      ctx->pair_pending = true;
    }
    for (size_t q = 0; q < np; ++q)
      if (sub < E[q].s) cur[q] = pbuf[q];
  }
  for (size_t q = 0; q < np; ++q)
    if (cur[q] != E[q].dst) HIP_TRY(magnus::launch_copy(cur[q], E[q].dst, (long long)R[q].h->H1.dim * E[q].B, s));
  return MAGNUS_OK;
}

// States into and out of the layout a group's iterations use: interleaved, or
// interleaved pairs when the group runs on coded terms.
int pack_group(magnus_ctx* ctx, const magnus_hamiltonian* h, const double2* src, double2* dst, int B, hipStream_t s) {
  if (ctx->coded_h == h && ctx->coded_pairs) HIP_TRY(magnus::launch_pack_pairs(src, dst, (int)h->H1.dim, B / 2, s));
  else HIP_TRY(magnus::launch_pack(src, dst, (int)h->H1.dim, B, s));
  return MAGNUS_OK;
}
int unpack_group(magnus_ctx* ctx, const magnus_hamiltonian* h, const double2* src, double2* dst, int B, hipStream_t s) {
  if (ctx->coded_h == h && ctx->coded_pairs) {
    if (int rc = flush_pair_check(ctx, s)) return rc;
    HIP_TRY(magnus::launch_unpack_pairs(src, dst, (int)h->H1.dim, B / 2, s));
  } else {
    HIP_TRY(magnus::launch_unpack(src, dst, (int)h->H1.dim, B, s));
  }
  return MAGNUS_OK;
}

// Launch the iterations of one planned multi-state exponential.
int launch_multi(magnus_ctx* ctx, const magnus_hamiltonian* h, const MultiExp& E, double tol_e, int early,
                 hipStream_t s) {
  if (int rc = flush_fused_check(ctx, s)) return rc;
  if (ctx->coded_h == h && ctx->coded_pairs && !E.frechet) {
    const PairWork W{h, ctx->coded, E.B / 2, ctx->vec(kA), ctx->vec(kB), ctx->vec(kS0), ctx->vec(kS1), 0, 0};
    return launch_pairs_exp(ctx, {W}, {E}, tol_e, early, false, s);
  }
  if (int rc = flush_pair_check(ctx, s)) return rc;
  const int dim = (int)h->H1.dim;
  const int B = E.B;
  const size_t n = (size_t)dim * B;
  CsrDev t1{h->H1.row_ptr, h->H1.col_idx, reinterpret_cast<const double2*>(h->H1.val)};
  CsrDev t2{h->H2.row_ptr, h->H2.col_idx, reinterpret_cast<const double2*>(h->H2.val)};
  const bool dense = h->H1.format == MAGNUS_DENSE;
  const int tile = dense && !E.frechet ? mfma_tile(ctx, h, B) : 0;
  const int split = dense && !E.frechet ? mfma_split(ctx, dim, B, tile) : 1;
  const int grid = dense ? (E.frechet ? magnus::dense_frechet_grid(dim) : magnus::dense_mfma_row_blocks(dim, split))
                         : magnus::csr2_multi_grid(dim, B);
  const int mode = E.frechet ? magnus::kMultiFrechet : magnus::kMultiLeja;
  if (grid <= 0 || (size_t)grid * (size_t)B * 2 > ctx->npartials)
    return fail(MAGNUS_ENOMEM, "per-workgroup partial sums (%d x %d) exceed the context's buffer", grid, B);
  const double2* D1 = reinterpret_cast<const double2*>(h->H1.val);
  const double2* D2 = reinterpret_cast<const double2*>(h->H2.val);
  long long ldd = h->H1.ld;
  if (dense && E.dense_terms == 1) {
    HIP_TRY(magnus::launch_dense_assemble(D1, D2, h->H1.ld, dim, E.ca, E.cb, nullptr, 0.0, ctx->assembled, s));
    D1 = ctx->assembled;
    ldd = dim;
  }
  const double tol_sub = tol_e / (2.0 * E.s);
  const double2* cur = E.src;
  for (int sub = 0; sub < E.s; ++sub) {
    const bool last = (sub == E.s - 1);
    double2* Pbuf;
    if (last && E.dst != cur) Pbuf = E.dst;
    else Pbuf = (cur == ctx->vec(kS0)) ? ctx->vec(kS1) : ctx->vec(kS0);
    for (int i = 1; i <= E.m; ++i) {
      MultiArgs a{};
      a.x = (i == 1) ? cur : ((i - 1) % 2 == 1 ? ctx->vec(kA) : ctx->vec(kB));
      a.wout = (i % 2 == 1) ? ctx->vec(kA) : ctx->vec(kB);
      a.pacc = Pbuf;
      a.slots = ctx->slots;
      a.partials = ctx->partials;
      a.prm = ctx->table + E.table_off + (size_t)(i - 1) * B;
      a.B = B;
      a.first = (i == 1);
      a.check_stop = (i != 1);
      a.early = early;
      a.tol = tol_sub;
      a.joint = E.frechet;
      if (dense && E.frechet)
        HIP_TRY(timed(ctx, MAGNUS_KERNEL_DENSE_LEJA, s,
                      [&] { return magnus::launch_dense_frechet(D1, D2, dim, h->H1.ld, a, s); }));
      else if (dense)
        HIP_TRY(timed(ctx, MAGNUS_KERNEL_DENSE_MFMA, s,
                      [&] { return magnus::launch_dense_mfma(E.dense_terms, D1, D2, ldd, dim, a, s, tile, split, ctx->split); }));
      else
        HIP_TRY(timed(ctx, MAGNUS_KERNEL_CSR_MULTI, s, [&] { return magnus::launch_csr2_multi(mode, t1, t2, dim, a, s); }));
      HIP_TRY(magnus::launch_multi_decide(a, grid, s));
    }
    cur = Pbuf;
  }
  if (cur != E.dst) HIP_TRY(magnus::launch_copy(cur, E.dst, (long long)n, s));
  return MAGNUS_OK;
}

// Largest supported group size for the remaining states.
int group_size(int remaining, int cap = 32) {
  for (int g : {32, 16, 8, 4, 2})
    if (g <= cap && remaining >= g) return g;
  return 1;
}

bool multi_ok(const magnus_hamiltonian* h, double kappa) { return kappa == 0.0; }

// Dense groups take every remaining state at once; CSR groups 32, 16, 8, 4, 2
// (at most the autotuned group size).
int group_for(magnus_ctx* ctx, const magnus_hamiltonian* h, int remaining) {
  if (h->H1.format == MAGNUS_DENSE) return remaining > 1 ? remaining : 1;
  // on coded terms: any number of pairs, up to 32 states as below (a group shares its largest substep count)
  if (ctx->coded_h == h && ctx->coded_pairs) return remaining > 1 ? std::min(remaining & ~1, 32) : 1;
  auto it = ctx->tuned_group.find({(const void*)h->H1.row_ptr, h->H1.dim});
  return group_size(remaining, it == ctx->tuned_group.end() ? 32 : it->second);
}

// Plan one group exponential, assembling the dense exponent when all states share it.
int plan_group(magnus_ctx* ctx, const magnus_hamiltonian* h, const double* acoef, const double* bcoef, int B,
               double tau, double tol_e, const magnus_leja_opts* o, std::vector<ColParam>* table, MultiExp* E,
               Acc* acc) {
  bool shared = true;
  for (int b = 1; b < B; ++b) shared = shared && acoef[b] == acoef[0] && bcoef[b] == bcoef[0];
  const bool dense = h->H1.format == MAGNUS_DENSE;
  const bool assemble = dense && shared && ctx->assembled && ctx->assembled_dim >= h->H1.dim;
  int rc = plan_multi(h, acoef, bcoef, B, tau, tol_e, o, 0, table, E, acc, assemble);
  if (rc) return rc;
  E->dense_terms = dense ? (assemble ? 1 : 2) : 0;
  E->ca = acoef[0];
  E->cb = bcoef[0];
  return MAGNUS_OK;
}

// dst[c] = exp(-i tau (a H1 + b_c H2)) src[c] for the states c0..c0+B-1
// (b-major caller layout in and out).
int multi_expmv_group(magnus_ctx* ctx, const magnus_hamiltonian* h, int B, const double* acoef,
                      const double* bcoef, double tau, const double2* src, double2* dst, double tol_e,
                      const magnus_leja_opts* o, Acc* acc, hipStream_t s) {
  double2* Y = ctx->vec(kY);
  int rc = pack_group(ctx, h, src, Y, B, s);
  if (rc) return rc;
  std::vector<ColParam> table;
  MultiExp E;
  rc = plan_group(ctx, h, acoef, bcoef, B, tau, tol_e, o, &table, &E, acc);
  if (rc) return rc;
  if ((rc = upload_table(ctx, table, s))) return rc;
  E.src = Y;
  E.dst = Y;
  if ((rc = launch_multi(ctx, h, E, tol_e, o->early_termination, s))) return rc;
  return unpack_group(ctx, h, Y, dst, B, s);
}

// Product-of-exponentials steps for a group of B states held interleaved in
// kY, f values per state: fn(c, n, j) = f(t_n + c_j tau) of state c.
template <class F>
int multi_cf_steps(magnus_ctx* ctx, const magnus_hamiltonian* h, const magnus::Scheme& S, int B, double tau,
                   int64_t n0, int64_t n1, F fn, double tol_e, const magnus_leja_opts* o, Acc* acc,
                   hipStream_t s) {
  double2* Y = ctx->vec(kY);
  double2* mids[2] = {ctx->vec(kS2), ctx->vec(kU)};
  std::vector<double> av(B), bv(B), fv(S.q);
  // steps are planned and uploaded in segments that fit the parameter table
  int64_t n = n0;
  while (n < n1) {
    std::vector<ColParam> table;
    std::vector<MultiExp> exps;
    int64_t k = n;
    for (; k < n1; ++k) {
      const size_t mark = table.size();
      Acc trial = *acc;
      std::vector<MultiExp> step(S.nexp);
      const double2* src = Y;
      for (int e = 0; e < S.nexp; ++e) {
        for (int c = 0; c < B; ++c) {
          for (int j = 0; j < S.q; ++j) fv[j] = fn(c, k, j);
          av[c] = S.rho[e];
          bv[c] = scheme_b(S, e, fv.data());
        }
        int rc = plan_group(ctx, h, av.data(), bv.data(), B, tau, tol_e, o, &table, &step[e], &trial);
        if (rc) return rc;
        step[e].src = src;
        step[e].dst = (e == S.nexp - 1) ? Y : mids[e & 1];
        src = step[e].dst;
      }
      if (table.size() > kTableCap) {
        if (k == n) return fail(MAGNUS_ENOMEM, "one step needs more than the parameter table holds");
        table.resize(mark);
        break;
      }
      *acc = trial;
      for (const MultiExp& E : step) exps.push_back(E);
    }
    int rc = upload_table(ctx, table, s);
    if (rc) return rc;
    for (const MultiExp& E : exps)
      if ((rc = launch_multi(ctx, h, E, tol_e, o->early_termination, s))) return rc;
    n = k;
  }
  return MAGNUS_OK;
}

// ---------------------------------------------------------------------------
// Ragged batches: the large problems of equal group size B advance together,
// one launch per Leja iteration serving every problem (and one decision
// launch for all their columns), each group with its own terms, degrees,
// workspace slice, control slots and partial sums.
// ---------------------------------------------------------------------------
struct RagProblem {
  const magnus_problem* P;
  magnus::CodedDev C;  // its coded terms, when the problems run as pairs
  int c0, B;      // its states in the problem: a group of B from the c0-th on
  size_t voff;    // offset of its slice inside every workspace vector
  int slot0;      // its first control slot
  size_t poff;    // offset of its partial sums
  double2* v(magnus_ctx* ctx, int k) const { return ctx->vec(k) + voff; }
  double2* psi() const { return reinterpret_cast<double2*>(P->psi) + (size_t)c0 * P->h.H1.dim; }
};

// One exponential of every problem (E[q] planned for problem q).
int launch_ragged_exp(magnus_ctx* ctx, const std::vector<RagProblem>& R, const std::vector<MultiExp>& E, int B,
                      double tol_e, int early, hipStream_t s) {
  if (int rc = flush_fused_check(ctx, s)) return rc;
  const size_t np = R.size();
  std::vector<const double2*> cur(np);
  std::vector<double2*> pbuf(np);
  int max_s = 1;
  for (size_t q = 0; q < np; ++q) {
    cur[q] = E[q].src;
    max_s = std::max(max_s, E[q].s);
  }
  for (int sub = 0; sub < max_s; ++sub) {
    int max_m = 0;
    for (size_t q = 0; q < np; ++q) {
      if (sub >= E[q].s) continue;
      const bool last = sub == E[q].s - 1;
      if (last && E[q].dst != cur[q]) pbuf[q] = E[q].dst;
      else pbuf[q] = cur[q] == R[q].v(ctx, kS0) ? R[q].v(ctx, kS1) : R[q].v(ctx, kS0);
      max_m = std::max(max_m, E[q].m);
    }
    for (int i = 1; i <= max_m; ++i) {
      magnus::RaggedArgs r{};
      for (size_t q = 0; q < np; ++q) {
        if (sub >= E[q].s || i > E[q].m) continue;
        const magnus_hamiltonian& h = R[q].P->h;
        magnus::RaggedProblem& rp = r.p[r.np++];
        rp.t1 = CsrDev{h.H1.row_ptr, h.H1.col_idx, reinterpret_cast<const double2*>(h.H1.val)};
        rp.t2 = CsrDev{h.H2.row_ptr, h.H2.col_idx, reinterpret_cast<const double2*>(h.H2.val)};
        rp.dim = (int)h.H1.dim;
        MultiArgs& a = rp.a;
        a.x = (i == 1) ? cur[q] : ((i - 1) % 2 == 1 ? R[q].v(ctx, kA) : R[q].v(ctx, kB));
        a.wout = (i % 2 == 1) ? R[q].v(ctx, kA) : R[q].v(ctx, kB);
        a.pacc = pbuf[q];
        a.slots = ctx->slots + R[q].slot0;
        a.partials = ctx->partials + R[q].poff;
        a.prm = ctx->table + E[q].table_off + (size_t)(i - 1) * B;
        a.B = B;
        a.first = (i == 1);
        a.check_stop = (i != 1);
        a.early = early;
        a.tol = tol_e / (2.0 * E[q].s);
        a.joint = 0;
      }
      HIP_TRY(timed(ctx, MAGNUS_KERNEL_CSR_MULTI, s, [&] { return magnus::launch_csr2_ragged(r, B, s); }));
    }
    for (size_t q = 0; q < np; ++q)
      if (sub < E[q].s) cur[q] = pbuf[q];
  }
  for (size_t q = 0; q < np; ++q)
    if (cur[q] != E[q].dst)
      HIP_TRY(magnus::launch_copy(cur[q], E[q].dst, (long long)R[q].P->h.H1.dim * B, s));
  return MAGNUS_OK;
}

// Code the terms of a ragged batch's large problems and lay out their slices of
// the workspace, when they can run together as pairs: CSR terms found to fit the
// form, one even batch, everything within the context's buffers.  A problem's
// states go in groups of at most 32, as in propagate: a group shares its largest
// substep count, and one step's parameters of all groups fit the table (8 groups,
// 3 exponentials of 32 states and degree 64).  *out stays empty otherwise.
static_assert((size_t)magnus::kMaxPairProblems * magnus::kMaxCols * 3 * MAGNUS_MAX_DEGREE <= kTableCap,
              "a step's parameters");
int code_ragged(magnus_ctx* ctx, const magnus_problem* probs, const std::vector<int>& big, const magnus::Scheme& S,
                int64_t nsteps, int small_states, std::vector<RagProblem>* out, hipStream_t s) {
  const int batch = probs[big[0]].batch;
  const int groups = (batch + magnus::kMaxCols - 1) / magnus::kMaxCols;
  if (!ctx->fuse || ctx->csr_variant || batch < 2 || batch % 2 || batch > ctx->max_batch ||
      big.size() * (size_t)groups > (size_t)magnus::kMaxPairProblems)
    return MAGNUS_OK;
  const int npairs = batch / 2;
  // several rows of slices to a wave where problems of several sizes share a launch
  const int min_rows = big.size() > 1 ? 256 : 64;
  size_t slices = 0, blocks = 0, rows = 0, voff = 0, poff = 0;
  int slot0 = small_states;
  std::vector<RagProblem> R;
  for (int i : big) {
    const magnus_problem& P = probs[i];
    const magnus_hamiltonian* h = &P.h;
    if (P.batch != batch || !coding_possible(ctx, h)) return MAGNUS_OK;
    if (ctx->coding < 2 && (!ctx->codable.count(pair_key(h)) || (h->H1.dim < 65536 && S.nexp * nsteps < 2) ||
                            tuned_uncoded(ctx, h, true)))
      return MAGNUS_OK;
    const int dim = (int)h->H1.dim;
    magnus::CodedDev C = ctx->coded;
    C.rows = magnus::code_pair_rows(dim, npairs, min_rows, h->H1.nnz + h->H2.nnz, false);
    C.codes += slices * 64 * magnus::kCodeAhead;
    C.more += slices * 64 * magnus::kCodeMore;
    C.head += slices * magnus::kCodeHead;
    C.dict += blocks * (magnus::kCodeMax + 1);
    C.block += blocks;
    C.diag += rows;
    const size_t grid = (size_t)magnus::code_grid(dim, C.rows);
    for (int c0 = 0; c0 < batch; c0 += magnus::kMaxCols) {
      const int B = std::min(magnus::kMaxCols, batch - c0);
      R.push_back(RagProblem{&P, C, c0, B, voff, slot0, poff});
      voff += (size_t)dim * B;
      poff += 2 * (size_t)B * grid;
      slot0 += B;
    }
    slices += ((size_t)dim + 63) / 64 * 4;
    blocks += grid;
    rows += (size_t)dim;
  }
  if (slices > ctx->coded_slices || blocks > ctx->coded_blocks || rows > (size_t)ctx->max_dim ||
      voff > (size_t)ctx->max_dim * (size_t)ctx->max_batch || pair_partials_at(ctx) + 2 * poff > ctx->npartials ||
      slot0 > ctx->nslots)
    return MAGNUS_OK;
  for (const RagProblem& q : R) {
    if (q.c0 > 0) continue;  // a problem's groups share its coded terms
    const magnus::CodeTerms T{2, {csr_dev(q.P->h.H1), csr_dev(q.P->h.H2)}};
    HIP_TRY(magnus::launch_code_build(T, (int)q.P->h.H1.dim, q.C, nullptr, s));
  }
  *out = std::move(R);
  return MAGNUS_OK;
}

// Product-of-exponentials steps of the ragged batch's large problems, packed
// into their workspace slices (interleaved groups, all of the same size; or pairs).
int ragged_joint_steps(magnus_ctx* ctx, std::vector<RagProblem>& R, const magnus::Scheme& S, double tau,
                       int64_t nsteps, double tol_e, const magnus_leja_opts* o, Acc* acc, hipStream_t s) {
  const bool pairs = R[0].C.codes != nullptr;
  std::vector<PairWork> W;
  for (const RagProblem& q : R) {
    const int dim = (int)q.P->h.H1.dim;
    if (pairs) {
      HIP_TRY(magnus::launch_pack_pairs(q.psi(), q.v(ctx, kY), dim, q.B / 2, s));
      W.push_back(PairWork{&q.P->h, q.C, q.B / 2, q.v(ctx, kA), q.v(ctx, kB), q.v(ctx, kS0), q.v(ctx, kS1), q.slot0, q.poff});
    } else {
      HIP_TRY(magnus::launch_pack(q.psi(), q.v(ctx, kY), dim, q.B, s));
    }
  }
  std::vector<double> av(magnus::kMaxCols), bv(magnus::kMaxCols), fv(S.q);
  int64_t n = 0;
  while (n < nsteps) {
    std::vector<ColParam> table;
    std::vector<std::vector<MultiExp>> steps;  // [step * nexp + e][problem]
    int64_t k = n;
    for (; k < nsteps; ++k) {
      const size_t mark = table.size();
      Acc trial = *acc;
      std::vector<std::vector<MultiExp>> st(S.nexp, std::vector<MultiExp>(R.size()));
      for (size_t q = 0; q < R.size(); ++q) {
        const magnus_problem& P = *R[q].P;
        const int B = R[q].B;
        const double2* src = R[q].v(ctx, kY);
        double2* mids[2] = {R[q].v(ctx, kS2), R[q].v(ctx, kU)};
        for (int e = 0; e < S.nexp; ++e) {
          for (int c = 0; c < B; ++c) {
            const double* f = P.f_nodes + ((P.batch_f == 1 ? 0 : (int64_t)(R[q].c0 + c)) * nsteps + k) * S.q;
            for (int j = 0; j < S.q; ++j) fv[j] = f[j];
            av[c] = S.rho[e];
            bv[c] = scheme_b(S, e, fv.data());
          }
          MultiExp& E = st[e][q];
          int rc = plan_multi(&P.h, av.data(), bv.data(), B, tau, tol_e, o, 0, &table, &E, &trial);
          if (rc) return rc;
          E.src = src;
          E.dst = (e == S.nexp - 1) ? R[q].v(ctx, kY) : mids[e & 1];
          src = E.dst;
        }
      }
      if (table.size() > kTableCap) {
        if (k == n) return fail(MAGNUS_ENOMEM, "one step needs more than the parameter table holds");
        table.resize(mark);
        break;
      }
      *acc = trial;
      for (auto& e : st) steps.push_back(std::move(e));
    }
    int rc = upload_table(ctx, table, s);
    if (rc) return rc;
    for (const auto& E : steps) {
      rc = pairs ? launch_pairs_exp(ctx, W, E, tol_e, o->early_termination, false, s)
                 : launch_ragged_exp(ctx, R, E, R[0].B, tol_e, o->early_termination, s);
      if (rc) return rc;
    }
    n = k;
  }
  for (const RagProblem& q : R) {
    const int dim = (int)q.P->h.H1.dim;
    if (pairs) HIP_TRY(magnus::launch_unpack_pairs(q.v(ctx, kY), q.psi(), dim, q.B / 2, s));
    else HIP_TRY(magnus::launch_unpack(q.v(ctx, kY), q.psi(), dim, q.B, s));
  }
  return flush_pair_check(ctx, s);
}

// ---------------------------------------------------------------------------
// Whole Cf4 propagations of small states, one workgroup per state.
// ---------------------------------------------------------------------------
struct SmallState {
  int prob;
  double2* psi;
  const double* fn;  // this state's field samples, [nsteps][q]
};

// One workgroup's iteration time grows with the dimension, while the
// per-iteration grid launches of the other paths cost about the same for any
// dimension up to a few thousand rows; the persistent launch pays off when its
// states are small or many.  Measured crossover (MI355X, Cf4 on spin chains,
// state-steps/s persistent vs grid): 1024 rows win from one state on; 2048
// rows lose at one state (5.1k vs 7.5k) and win at four (19k vs 14k); 4096
// rows lose up to 16 states (38k vs 40k) and win at 64 (151k vs 59k).
int64_t small_cap(const magnus_ctx* ctx, int64_t nstates) {
  if (ctx->persist == 0) return 0;
  if (ctx->persist >= 2 || nstates >= 32) return kSmallDim;
  return nstates >= 4 ? 2048 : 1024;
}

bool small_candidate(const magnus_hamiltonian* h) { return h->H1.format == MAGNUS_CSR && h->H1.dim <= kSmallDim; }

// Whether the one-workgroup kernels are expected to hold these terms' rows in
// registers: 24 entries a row of real or imaginary values, which terms that fit
// the coded form with 20 a row between them have (only a guess at what is
// fastest: the kernel looks at every row).
bool rows_in_registers(const magnus_ctx* ctx, const magnus_hamiltonian* h) {
  return h->H1.dim <= magnus::kPersistStepDim && h->H1.nnz + h->H2.nnz <= 20 * h->H1.dim &&
         ctx->codable.count(pair_key(h));
}

// Whether the kernels for states of up to 1,024 rows can keep term 1 in LDS.
bool term1_in_lds(const magnus_ctx* ctx, const magnus_hamiltonian* h) {
  return ctx->persist_cache && h->H1.dim <= magnus::kPersistStepDim && h->H1.nnz <= magnus::kPersistCache;
}

// One state of which a workgroup would read more than 12,000 entries from memory
// in every iteration takes the grid path (us per iteration in one workgroup / on
// the grid; rows of equal length, 1,024 of them, term 1 in LDS: 10,240 entries
// 4.5 / 5.3, 14,336 5.7 / 5.5; 700 rows read whole: 14,000 5.2 / 5.4; random rows,
// whose longest a workgroup waits for, meet at 8,000 and 10,000 entries).
bool small_ok(magnus_ctx* ctx, const magnus_hamiltonian* h, int64_t nstates) {
  if (!small_candidate(h) || h->H1.dim > small_cap(ctx, nstates)) return false;
  if (nstates > 1 || ctx->persist >= 2 || rows_in_registers(ctx, h)) return true;
  return h->H2.nnz + (term1_in_lds(ctx, h) ? 0 : h->H1.nnz) <= 12000;
}

// exp(-i tau (a H1 + b H2)) for the one-workgroup kernels: its header, and its iterations appended to the table.
int persist_exponential(const magnus_hamiltonian* h, double ca, double cb, double tau, double tol_e,
                        const magnus_leja_opts* o, PersistExp* E, std::vector<ColParam>* table, Acc* acc) {
  const auto& xi = magnus::leja_points();
  double lo, hi;
  magnus::weyl_interval(ca, h->H1.lam_min, h->H1.lam_max, cb, h->H2.lam_min, h->H2.lam_max, 0.0, 0.0, 0.0, &lo, &hi);
  ExpPlan P;
  if (!magnus::plan_exponential(tau, lo, hi, tol_e, o->max_degree, o->max_substeps, &P))
    return fail(MAGNUS_ENOCONV, "no degree <= %d with <= %d substeps reaches tol %g", o->max_degree, o->max_substeps,
                tol_e);
  E->m = P.lp.m;
  E->s = P.lp.s;
  E->table_off = (long long)table->size();
  E->tol_sub = tol_e / (2.0 * P.lp.s);
  const double d0abs = std::abs(P.d[0]);
  for (int i = 1; i <= P.lp.m; ++i) {
    ColParam c{};
    c.a1 = P.scale * ca;
    c.a2 = P.scale * cb;
    c.sigma = P.scale * P.c + xi[i - 1];
    c.dre = P.d[i].real();
    c.dim = P.d[i].imag();
    c.dabs = std::abs(P.d[i]);
    c.d0re = P.d[0].real();
    c.d0im = P.d[0].imag();
    c.d0abs = d0abs;
    table->push_back(c);
  }
  acc->exponentials += 1;
  acc->substeps += P.lp.s;
  acc->planned += (int64_t)P.lp.m * P.lp.s;
  acc->max_m = std::max(acc->max_m, P.lp.m);
  acc->max_s = std::max(acc->max_s, P.lp.s);
  acc->max_bound = std::max(acc->max_bound, P.lp.bound);
  return MAGNUS_OK;
}

// Steps n0..n1-1 of every state in one launch.
int persist_segment(magnus_ctx* ctx, const std::vector<const magnus_hamiltonian*>& hs,
                    const std::vector<SmallState>& st, const magnus::Scheme& S, double tau, int64_t n0, int64_t n1,
                    double tol_e, const magnus_leja_opts* o, Acc* acc, hipStream_t s) {
  if (int rc = flush_fused_check(ctx, s)) return rc;
  const int nst = (int)st.size();
  const int nexp = (int)(S.nexp * (n1 - n0));
  if (nst > ctx->nslots) return fail(MAGNUS_ENOMEM, "%d small states exceed %d control slots", nst, ctx->nslots);
  int64_t maxdim = 1;
  for (auto* h : hs) maxdim = std::max<int64_t>(maxdim, h->H1.dim);
  if (maxdim > magnus::kPersistMaxDim) return fail(MAGNUS_EINVAL, "dimension %lld too large for the small-state kernel", (long long)maxdim);
  std::vector<ColParam> table;
  std::vector<PersistExp> exps((size_t)nst * nexp);
  for (int b = 0; b < nst; ++b) {
    const magnus_hamiltonian* h = hs[st[b].prob];
    for (int64_t n = n0; n < n1; ++n) {
      const double* f = st[b].fn + S.q * n;
      for (int half = 0; half < S.nexp; ++half) {
        if (int rc = persist_exponential(h, S.rho[half], scheme_b(S, half, f), tau, tol_e, o,
                                         &exps[(size_t)b * nexp + S.nexp * (n - n0) + half], &table, acc))
          return rc;
      }
    }
  }
  if (table.size() > kTableCap) return fail(MAGNUS_ENOMEM, "parameter table overflow");
  // headers: problems | state_prob | state pointers | exponentials
  std::vector<PersistProblem> probs(hs.size());
  for (size_t i = 0; i < hs.size(); ++i) {
    const magnus_hamiltonian* h = hs[i];
    probs[i].t1 = CsrDev{h->H1.row_ptr, h->H1.col_idx, reinterpret_cast<const double2*>(h->H1.val)};
    probs[i].t2 = CsrDev{h->H2.row_ptr, h->H2.col_idx, reinterpret_cast<const double2*>(h->H2.val)};
    probs[i].dim = (int)h->H1.dim;
  }
  std::vector<int> sp(nst);
  std::vector<double2*> ptrs(nst);
  for (int b = 0; b < nst; ++b) {
    sp[b] = st[b].prob;
    ptrs[b] = st[b].psi;
  }
  auto align = [](size_t x) { return (x + 255) & ~size_t(255); };
  const size_t o_prob = 0;
  const size_t o_sp = align(o_prob + sizeof(PersistProblem) * probs.size());
  const size_t o_ptr = align(o_sp + sizeof(int) * sp.size());
  const size_t o_exp = align(o_ptr + sizeof(double2*) * ptrs.size());
  const size_t total = o_exp + sizeof(PersistExp) * exps.size();
  if (total > kArenaBytes) return fail(MAGNUS_ENOMEM, "call headers of %zu bytes exceed the arena", total);
  std::vector<unsigned char> host(total);
  memcpy(host.data() + o_prob, probs.data(), sizeof(PersistProblem) * probs.size());
  memcpy(host.data() + o_sp, sp.data(), sizeof(int) * sp.size());
  memcpy(host.data() + o_ptr, ptrs.data(), sizeof(double2*) * ptrs.size());
  memcpy(host.data() + o_exp, exps.data(), sizeof(PersistExp) * exps.size());
  HIP_TRY(hipMemcpyAsync(ctx->arena, host.data(), total, hipMemcpyHostToDevice, s));
  int rc = upload_table(ctx, table, s);
  if (rc) return rc;
  PersistArgs a{};
  a.probs = reinterpret_cast<const PersistProblem*>(ctx->arena + o_prob);
  a.state_prob = reinterpret_cast<const int*>(ctx->arena + o_sp);
  a.state = reinterpret_cast<double2* const*>(ctx->arena + o_ptr);
  a.table = ctx->table;
  a.exps = reinterpret_cast<const PersistExp*>(ctx->arena + o_exp);
  a.nexp = nexp;
  a.slots = ctx->slots;
  a.early = o->early_termination;
  // term 1 in LDS: one workgroup per CU then, so only while the states fit the chip
  a.cache1 = nst <= 256;
  a.in_regs = 1;
  for (const magnus_hamiltonian* h : hs) {
    a.cache1 = a.cache1 && term1_in_lds(ctx, h);
    a.in_regs = a.in_regs && rows_in_registers(ctx, h);
  }
  HIP_TRY(timed(ctx, MAGNUS_KERNEL_PERSIST, s, [&] { return magnus::launch_persist_propagate(a, nst, (int)maxdim, s); }));
  return MAGNUS_OK;
}

// All steps of a set of small-state problems, split into segments whose
// tables fit (and at the given stop points).
int persist_steps(magnus_ctx* ctx, const std::vector<const magnus_hamiltonian*>& hs,
                  const std::vector<SmallState>& st, const magnus::Scheme& S, double tau, int64_t n0, int64_t n1,
                  double tol_e, const magnus_leja_opts* o, Acc* acc, hipStream_t s) {
  const int64_t per_step = (int64_t)st.size() * S.nexp * std::max(1, o->max_degree) * 2;
  int64_t L = std::max<int64_t>(1, (int64_t)kTableCap / std::max<int64_t>(per_step, 1));
  L = std::min<int64_t>(L, (int64_t)(kArenaBytes / 2) / ((int64_t)sizeof(PersistExp) * S.nexp * (int64_t)st.size() + 1));
  L = std::max<int64_t>(L, 1);
  for (int64_t n = n0; n < n1; n += L) {
    int rc = persist_segment(ctx, hs, st, S, tau, n, std::min(n1, n + L), tol_e, o, acc, s);
    if (rc) return rc;
  }
  return MAGNUS_OK;
}

// Plan of one exponential of a replayed step with s substeps: the plan the
// launch-by-launch path makes when it chooses s itself, else the smallest
// degree for s substeps.
bool graph_step_plan(double tau, double lo, double hi, double tol_e, int s, const magnus_leja_opts* o, ExpPlan* P) {
  if (magnus::plan_exponential(tau, lo, hi, tol_e, o->max_degree, o->max_substeps, P) && P->lp.s == s) return true;
  return magnus::plan_exponential_fixed_s(tau, lo, hi, tol_e, s, o->max_degree, P);
}

// ---------------------------------------------------------------------------
// Graph replay of a single CSR state's steps.  The launches of one Magnus step
// (every exponential's substeps and iterations, with the stop tests fused)
// are captured once per call and replayed once per step; each launch reads
// its Leja coefficients from a device table column indexed by a step counter
// that the graph advances at its end.  Every step has the same launch
// structure: per exponential k the largest substep count s_k and degree m_k
// over the call's steps, iterations past a step's own degree inactive.
// ---------------------------------------------------------------------------
struct GraphPlan {
  int nexp = 0;
  std::vector<int> s, m;    // per exponential
  std::vector<int> off;     // first record of exponential k in a step
  int stride = 0;           // records per step
  std::vector<double> lo, hi;  // enclosure of exponential k of step n at [n * nexp + k]
  std::vector<ExpOp> ops;      // exponent of exponential k of step n
};

// Records of the graph's step table that fit the context's table memory.
int64_t graph_table_cap(const magnus_ctx*) {
  return (int64_t)(kTableCap * sizeof(ColParam) / sizeof(magnus::IterCoef));
}

// Whether every iteration launch of this state's exponentials makes its own
// stop test (the condition for capturing a step: no decide kernels).
bool graph_eligible(magnus_ctx* ctx, const magnus_hamiltonian* h, const magnus::Scheme& S) {
  if (!ctx->graph || !ctx->fuse || ctx->timing || h->H1.format != MAGNUS_CSR || S.sixth) return false;
  const int dim = (int)h->H1.dim;
  if (ctx->coded_h == h) return magnus::code_grid(dim, ctx->coded.rows) <= magnus::kFuseMaxGrid;
  int rpb = rows_per_block(ctx, h, S.commutator);
  if (S.commutator && csr_comm_ready(ctx, h)) rpb = magnus::csr3_rows(dim, rows_per_block(ctx, h));
  return magnus::csr2_grid(dim, rpb) <= magnus::csr2_fuse_grid(rpb);
}

template <class F>
int graph_plan(magnus_ctx* ctx, const magnus_hamiltonian* h, const magnus::Scheme& S, double tau, int64_t nsteps,
               F fval, double tol_e, const magnus_leja_opts* o, GraphPlan* G) {
  G->nexp = S.commutator ? 1 : S.nexp;
  const int ne = G->nexp;
  G->s.assign(ne, 1);
  G->m.assign(ne, 1);
  G->lo.resize((size_t)nsteps * ne);
  G->hi.resize((size_t)nsteps * ne);
  G->ops.resize((size_t)nsteps * ne);
  for (int64_t n = 0; n < nsteps; ++n) {
    double f[3] = {0, 0, 0};
    for (int j = 0; j < S.q; ++j) f[j] = fval(n, j);
    for (int k = 0; k < ne; ++k) {
      ExpOp op;
      if (S.commutator) {
        op = ExpOp{h, 1.0, 0.5 * (f[0] + f[1]), magnus::kSqrt3 * tau * (f[1] - f[0]) / 12.0};
      } else {
        op = ExpOp{h, S.rho[k], scheme_b(S, k, f), 0.0};
      }
      double lo, hi;
      magnus::weyl_interval(op.a, h->H1.lam_min, h->H1.lam_max, op.b, h->H2.lam_min, h->H2.lam_max, op.kappa,
                            h->k_min, h->k_max, &lo, &hi);
      ExpPlan P;
      if (!magnus::plan_exponential(tau, lo, hi, tol_e, o->max_degree, o->max_substeps, &P))
        return fail(MAGNUS_ENOCONV, "no degree <= %d with <= %d substeps reaches tol %g", o->max_degree,
                    o->max_substeps, tol_e);
      G->s[k] = std::max(G->s[k], P.lp.s);
      const size_t q = (size_t)n * ne + k;
      G->ops[q] = op;
      G->lo[q] = lo;
      G->hi[q] = hi;
    }
  }
  for (int64_t n = 0; n < nsteps; ++n)
    for (int k = 0; k < ne; ++k) {
      ExpPlan P;
      const size_t q = (size_t)n * ne + k;
      if (!graph_step_plan(tau, G->lo[q], G->hi[q], tol_e, G->s[k], o, &P))
        return fail(MAGNUS_ENOCONV, "no degree <= %d reaches tol %g with %d substeps", o->max_degree, tol_e, G->s[k]);
      G->m[k] = std::max(G->m[k], P.lp.m);
    }
  G->off.assign(ne, 0);
  G->stride = 0;
  for (int k = 0; k < ne; ++k) {
    G->off[k] = G->stride;
    G->stride += G->s[k] * G->m[k];
  }
  if (G->stride > graph_table_cap(ctx)) return fail(MAGNUS_ENOMEM, "step table too large for graph replay");
  return MAGNUS_OK;
}

// Coefficient records of steps [n0, n1) in the layout a captured step reads
// (record off[k] + sub * m[k] + i - 1 of each step).
int graph_fill(const GraphPlan& G, double tau, int64_t n0, int64_t n1, double tol_e, const magnus_leja_opts* o,
               Acc* acc, std::vector<magnus::IterCoef>* out) {
  const auto& xi = magnus::leja_points();
  const int ne = G.nexp;
  out->assign((size_t)(n1 - n0) * G.stride, magnus::IterCoef{});
  for (int64_t n = n0; n < n1; ++n)
    for (int k = 0; k < ne; ++k) {
      const size_t q = (size_t)n * ne + k;
      ExpPlan P;
      if (!graph_step_plan(tau, G.lo[q], G.hi[q], tol_e, G.s[k], o, &P))
        return fail(MAGNUS_ENOCONV, "no degree <= %d reaches tol %g", o->max_degree, tol_e);
      const ExpOp& op = G.ops[q];
      const int m = P.lp.m, ns = G.s[k];
      for (int sub = 0; sub < ns; ++sub)
        for (int i = 1; i <= m; ++i) {
          magnus::IterCoef& c = (*out)[(size_t)(n - n0) * G.stride + G.off[k] + (size_t)sub * G.m[k] + (i - 1)];
          c.a1 = P.scale * op.a;
          c.a2 = P.scale * op.b;
          c.kap = P.scale * op.kappa;
          c.sigma = P.scale * P.c + xi[i - 1];
          c.dre = P.d[i].real();
          c.dim = P.d[i].imag();
          c.d0re = P.d[0].real();
          c.d0im = P.d[0].imag();
          c.dabs = std::abs(P.d[i]);
          c.d0abs = std::abs(P.d[0]);
          c.prev_dabs = i >= 2 ? std::abs(P.d[i - 1]) : 0.0;
          c.tol = tol_e / (2.0 * ns);
          c.active = 1;
        }
      acc->exponentials += 1;
      acc->substeps += ns;
      acc->planned += (int64_t)m * ns;
      acc->max_m = std::max(acc->max_m, m);
      acc->max_s = std::max(acc->max_s, ns);
      acc->max_bound = std::max(acc->max_bound, P.lp.bound);
    }
  return MAGNUS_OK;
}

void graph_release(magnus_ctx* ctx) {
  if (ctx->graph_x) (void)hipGraphExecDestroy(ctx->graph_x);
  if (ctx->graph_g) (void)hipGraphDestroy(ctx->graph_g);
  ctx->graph_x = nullptr;
  ctx->graph_g = nullptr;
}

// Capture the launches of one step of state y (in place) on the context's
// capture stream: the exponentials in the scheme's order, each launch bound
// to its table column, then the step counter's advance.
int graph_capture(magnus_ctx* ctx, const magnus_hamiltonian* h, const magnus::Scheme& S, const GraphPlan& G,
                  double2* y, double tol_e, int early) {
  if (ctx->graph_x) {
    // the previous call's replays must have finished before its graph goes
    HIP_TRY(hipEventSynchronize(ctx->graph_done));
    graph_release(ctx);
  }
  if (!ctx->cap_stream) HIP_TRY(hipStreamCreateWithFlags(&ctx->cap_stream, hipStreamNonBlocking));
  hipStream_t cs = ctx->cap_stream;
  const magnus::IterCoef* base = reinterpret_cast<const magnus::IterCoef*>(ctx->table);
  HIP_TRY(hipStreamBeginCapture(cs, hipStreamCaptureModeRelaxed));
  int rc = MAGNUS_OK;
  double2* mids[2] = {ctx->vec(kS2), ctx->vec(kU)};
  const double2* src = y;
  for (int k = 0; k < G.nexp && rc == MAGNUS_OK; ++k) {
    // structure only: the coefficients come from the table
    ExpPlan T;
    T.scale = 1.0;
    T.lp = magnus::LejaPlan{G.m[k], G.s[k], 0.0};
    T.d.assign((size_t)G.m[k] + 1, std::complex<double>(1.0, 0.0));
    const TableRef tab{base + G.off[k], G.stride, ctx->gctr};
    double2* dst = (k == G.nexp - 1) ? y : mids[k & 1];
    const ExpOp op{h, 1.0, 1.0, S.commutator ? 1.0 : 0.0};
    rc = enqueue_exponential(ctx, op, T, src, dst, tol_e / (2.0 * G.s[k]), early, &tab, cs);
    src = dst;
  }
  if (rc == MAGNUS_OK && magnus::launch_step_advance(ctx->gctr, cs) != hipSuccess)
    rc = fail(MAGNUS_EHIP, "step counter launch during capture");
  hipGraph_t g = nullptr;
  const hipError_t e = hipStreamEndCapture(cs, &g);
  if (rc != MAGNUS_OK || e != hipSuccess) {
    if (g) (void)hipGraphDestroy(g);
    return rc != MAGNUS_OK ? rc : fail(MAGNUS_EHIP, "hipStreamEndCapture: %s", hipGetErrorString(e));
  }
  ctx->graph_g = g;
  HIP_TRY(hipGraphInstantiate(&ctx->graph_x, g, nullptr, nullptr, 0));
  if (!ctx->graph_done) HIP_TRY(hipEventCreateWithFlags(&ctx->graph_done, hipEventDisableTiming));
  return MAGNUS_OK;
}

// Replay steps [n0, n1): table chunks uploaded behind the previous replays,
// the counter set to the chunk's first step, one graph launch per step.
int graph_replay(magnus_ctx* ctx, const GraphPlan& G, double tau, int64_t n0, int64_t n1, double tol_e,
                 const magnus_leja_opts* o, Acc* acc, hipStream_t s) {
  int64_t per = std::max<int64_t>(1, graph_table_cap(ctx) / G.stride);
  if (ctx->graph_chunk > 0) per = std::min<int64_t>(per, ctx->graph_chunk);
  for (int64_t c0 = n0; c0 < n1; c0 += per) {
    const int64_t c1 = std::min(n1, c0 + per);
    int rc = graph_fill(G, tau, c0, c1, tol_e, o, acc, &ctx->graph_table);
    if (rc) return rc;
    HIP_TRY(hipMemcpyAsync(ctx->table, ctx->graph_table.data(), sizeof(magnus::IterCoef) * ctx->graph_table.size(),
                           hipMemcpyHostToDevice, s));
    HIP_TRY(magnus::launch_step_set(ctx->gctr, 0, s));
    for (int64_t n = c0; n < c1; ++n) HIP_TRY(hipGraphLaunch(ctx->graph_x, s));
  }
  HIP_TRY(hipEventRecord(ctx->graph_done, s));
  return MAGNUS_OK;
}

int check_batch(magnus_ctx* ctx, int32_t batch) {
  if (batch < 1) return fail(MAGNUS_EINVAL, "batch %d < 1", batch);
  if (batch > ctx->max_batch) return fail(MAGNUS_ENOMEM, "batch %d exceeds workspace max_batch %d", batch, ctx->max_batch);
  return MAGNUS_OK;
}

}  // namespace

// ---------------------------------------------------------------------------
// Scratch of the allocation-free Cf4 step (magnus_step_cf4_noalloc): the eight
// workspace vectors of one state of up to kNoAllocMaxDim entries, the
// per-workgroup norm partials of the iteration kernels, the outputs of the
// CSR structure scan and one control slot.  A file-scope device array, so the
// code object's loader places it on every device the library runs on, and it
// stays there until the process ends.  Host code never uses the array's name
// as an address: it asks each device for its copy's address once
// (hipGetSymbolAddress) and passes that pointer on.
// ---------------------------------------------------------------------------
namespace {
constexpr int64_t kNoAllocMaxDim = 1 << 17;
constexpr size_t kNaAlign = 256;
constexpr size_t na_round(size_t b) { return (b + kNaAlign - 1) / kNaAlign * kNaAlign; }
constexpr size_t kNaVecBytes = (size_t)kNumVec * (size_t)kNoAllocMaxDim * sizeof(double2);
constexpr int64_t kNaGrid = kNoAllocMaxDim / 8 + 2;  // as magnus_create: 8 rows per smallest row block
constexpr size_t kNaPartials = 4 * (size_t)kNaGrid + 64;  // two halves for the fused stop tests
constexpr int64_t kNaScanLen = 2 * (kNoAllocMaxDim / 4 + 2) + 3 * (kNoAllocMaxDim / 256 + 2);
constexpr size_t kNaPartialOff = kNaVecBytes;
constexpr size_t kNaScanOff = kNaPartialOff + na_round(kNaPartials * sizeof(double));
constexpr size_t kNaSlotOff = kNaScanOff + na_round((size_t)kNaScanLen * sizeof(double));
constexpr size_t kNoAllocBytes = kNaSlotOff + na_round(sizeof(Slot));  // 17.0 MiB
constexpr int kNaMaxDevices = 64;
}  // namespace

static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];

namespace {
std::mutex g_na_mu;
// One context per device whose workspace points into that device's scratch
// (set up on the first call on the device; never freed).
magnus_ctx g_na_ctx[kNaMaxDevices];

int noalloc_context(magnus_ctx** out) {
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= kNaMaxDevices) return fail(MAGNUS_EINVAL, "device %d beyond the %d the library serves", dev, kNaMaxDevices);
  std::lock_guard<std::mutex> g(g_na_mu);
  magnus_ctx& c = g_na_ctx[dev];
  if (!c.vecs) {
    void* ptr = nullptr;
    hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr)
      return fail(MAGNUS_EHIP, "address of the scratch array on device %d: %s", dev, hipGetErrorString(e));
    unsigned char* base = static_cast<unsigned char*>(ptr);
    c.device = dev;
    c.max_dim = kNoAllocMaxDim;
    c.max_batch = 1;
    c.max_grid = kNaGrid;
    c.partials = reinterpret_cast<double*>(base + kNaPartialOff);
    c.npartials = kNaPartials;
    c.scan = reinterpret_cast<double*>(base + kNaScanOff);
    c.scan_len = kNaScanLen;
    c.slots = reinterpret_cast<Slot*>(base + kNaSlotOff);
    c.nslots = 1;
    c.persist = 0;
    c.coding = 0;  // (its form would be allocated)
    if (const char* v = getenv("MAGNUS_CSR_VARIANT")) c.csr_variant = atoi(v);
    if (const char* v = getenv("MAGNUS_FUSE")) c.fuse = atoi(v);
    c.vecs = reinterpret_cast<double2*>(base);  // last: marks the device's context ready
  }
  *out = &c;
  return MAGNUS_OK;
}
}  // namespace

extern "C" {

const char* magnus_last_error(void) { return g_err.c_str(); }

int magnus_create(magnus_ctx** out, int64_t max_dim, int32_t max_batch, int32_t device) {
  if (!out) return fail(MAGNUS_EINVAL, "null output pointer");
  *out = nullptr;
  if (max_dim < 1 || max_batch < 1) return fail(MAGNUS_EINVAL, "max_dim and max_batch must be >= 1");
  if (max_dim > INT32_MAX / 2) return fail(MAGNUS_EINVAL, "max_dim too large");
  int ndev = 0;
  HIP_TRY(hipGetDeviceCount(&ndev));
  if (device < 0 || device >= ndev) return fail(MAGNUS_EINVAL, "device %d not in 0..%d", device, ndev - 1);
  HIP_TRY(hipSetDevice(device));
  magnus_ctx* c = new magnus_ctx();
  c->device = device;
  c->max_dim = max_dim;
  c->max_batch = max_batch;
  if (const char* v = getenv("MAGNUS_CSR_VARIANT")) c->csr_variant = atoi(v);
  // the smallest row block of any CSR iteration kernel is 8 rows; the dense ones have their own grid
  c->max_grid = std::max<int64_t>(max_dim / 8 + 2, magnus::dense2_grid((int)max_dim));
  c->scan_len = 2 * (max_dim / 4 + 2) + 3 * (max_dim / 256 + 2);
  c->nslots = std::max<int>(256, max_batch);
  if (const char* v = getenv("MAGNUS_PERSIST")) c->persist = atoi(v);
  if (const char* v = getenv("MAGNUS_FUSE")) c->fuse = atoi(v);
  if (const char* v = getenv("MAGNUS_GRAPH")) c->graph = atoi(v);
  if (const char* v = getenv("MAGNUS_GRAPH_STEPS")) c->graph_chunk = atoi(v);
  if (const char* v = getenv("MAGNUS_RAGGED_JOINT")) c->ragged_joint = atoi(v);
  if (const char* v = getenv("MAGNUS_DENSE_RPW")) {
    const int r = atoi(v);
    c->dense_rpw_env = (r == 1 || r == 2 || r == 4) ? r : 0;
  }
  if (const char* v = getenv("MAGNUS_ASSEMBLE_FUSED")) c->fuse_assembly = atoi(v);
  if (const char* v = getenv("MAGNUS_PERSIST_CACHE")) c->persist_cache = atoi(v);
  if (const char* v = getenv("MAGNUS_MFMA_TILE")) {
    const int t = atoi(v);
    c->mfma_tile_env = (t >= 0 && t < magnus::kMfmaTiles) ? t : -1;
  }
  const size_t nvec = (size_t)kNumVec * (size_t)max_dim * (size_t)max_batch;
  hipError_t e = hipMalloc(&c->vecs, sizeof(double2) * nvec);
  if (e == hipSuccess) e = hipMalloc(&c->slots, sizeof(Slot) * c->nslots);
  if (e == hipSuccess) e = hipMalloc(&c->table, sizeof(ColParam) * kTableCap);
  if (e == hipSuccess) e = hipMalloc(&c->arena, kArenaBytes);
  // the multi-state CSR kernel writes dim * B^2 / 128 doubles (B <= 32: at most 8 dim)
  c->npartials = 2 * (size_t)c->max_grid + 8 * (size_t)max_dim +
                 (size_t)max_dim * (size_t)std::max(1, max_batch) / 8 + (size_t)max_dim + 64;
  // the dot-product kernel's per-workgroup pairs, whatever the dimension
  c->npartials = std::max(c->npartials, (size_t)magnus::kDotPartials + 64);
  c->npartials = (c->npartials + 31) / 32 * 32;  // the dot products' complex result behind them is aligned
  const size_t with_dots = c->npartials + magnus::kDotPartials + 64;
  if (e == hipSuccess) e = hipMalloc(&c->partials, sizeof(double) * with_dots);
  c->dots = c->partials + c->npartials;
  if (e == hipSuccess && max_batch > 1) {
    // groups of dense states: at most a third of the K chunks' number of shares
    c->split_entries = std::min<long long>(magnus::kSplitEntries, (max_dim / 48 + 1) * max_dim * (long long)max_batch);
    if (hipMalloc(&c->split, sizeof(double2) * (size_t)c->split_entries) != hipSuccess) {  // (groups run unsplit then)
      c->split = nullptr;
      c->split_entries = 0;
      (void)hipGetLastError();
    }
  }
  if (e == hipSuccess) e = hipMalloc(&c->scan, sizeof(double) * (size_t)c->scan_len);
  if (e == hipSuccess) e = hipMalloc(&c->gctr, 256);
  if (const char* v = getenv("MAGNUS_CODED")) c->coding = atoi(v);
  if (e == hipSuccess) e = hipMemset(c->slots, 0, sizeof(Slot) * c->nslots);
  if (e == hipSuccess) e = hipMemset(c->vecs, 0, sizeof(double2) * nvec);
  if (e == hipSuccess) e = hipDeviceSynchronize();
  if (e != hipSuccess) {
    magnus_destroy(c);
    return fail(MAGNUS_EHIP, "workspace allocation: %s", hipGetErrorString(e));
  }
  (void)magnus::leja_points();  // build the planner tables once, up front
  *out = c;
  return MAGNUS_OK;
}

int magnus_reserve_dense(magnus_ctx* ctx, int64_t dim) {
  if (!ctx) return fail(MAGNUS_EINVAL, "null context");
  if (dim < 1 || dim > ctx->max_dim) return fail(MAGNUS_EINVAL, "dim %lld outside 1..max_dim", (long long)dim);
  if (ctx->assembled_dim >= dim) return MAGNUS_OK;
  HIP_TRY(hipSetDevice(ctx->device));
  if (ctx->assembled) {
    HIP_TRY(hipDeviceSynchronize());
    HIP_TRY(hipFree(ctx->assembled));
    ctx->assembled = nullptr;
    ctx->assembled_dim = 0;
  }
  HIP_TRY(hipMalloc(&ctx->assembled, sizeof(double2) * (size_t)dim * (size_t)dim));
  ctx->assembled_dim = dim;
  return MAGNUS_OK;
}

int magnus_dense_commutator(magnus_ctx* ctx, magnus_hamiltonian* h, magnus_stream stream) {
  if (!ctx || !h) return fail(MAGNUS_EINVAL, "null argument");
  int rc = check_ham(ctx, h, 0);
  if (rc) return rc;
  if (h->H1.format != MAGNUS_DENSE) return fail(MAGNUS_EINVAL, "magnus_dense_commutator needs dense terms");
  const int64_t dim = h->H1.dim;
  if ((rc = magnus_reserve_dense(ctx, dim))) return rc;
  HIP_TRY(hipSetDevice(ctx->device));
  hipStream_t s = (hipStream_t)stream;
  if (ctx->comm_dim < dim) {
    if (ctx->comm) {
      HIP_TRY(hipDeviceSynchronize());
      HIP_TRY(hipFree(ctx->comm));
      ctx->comm = nullptr;
      ctx->comm_dim = 0;
    }
    HIP_TRY(hipMalloc(&ctx->comm, sizeof(double2) * (size_t)dim * (size_t)dim));
    ctx->comm_dim = dim;
  }
  ctx->comm_h1 = ctx->comm_h2 = nullptr;
  ctx->m6_ready = false;
  const double2* H1 = reinterpret_cast<const double2*>(h->H1.val);
  const double2* H2 = reinterpret_cast<const double2*>(h->H2.val);
  HIP_TRY(magnus::launch_zgemm(H1, h->H1.ld, H2, h->H2.ld, ctx->assembled, (int)dim, s));
  HIP_TRY(magnus::launch_commutator_combine(ctx->assembled, (int)dim, 1.0, ctx->comm, s));
  magnus_term kt{};
  kt.format = MAGNUS_DENSE;
  kt.dim = dim;
  kt.ld = dim;
  kt.val = ctx->comm;
  double lo, hi;
  if ((rc = dense_scan(ctx, kt, s, &lo, &hi))) return rc;
  h->k_min = lo;
  h->k_max = hi;
  ctx->comm_h1 = h->H1.val;
  ctx->comm_h2 = h->H2.val;
  ctx->comm_n = dim;
  ctx->comm_ld = h->H1.ld;
  return MAGNUS_OK;
}

// out = i (A B - B A) of two CSR matrices into the storage (rp, ci, val) of
// rows + 1 and cap entries (grown as needed), with its Gershgorin enclosure.
int assemble_csr_commutator(magnus_ctx* ctx, const CsrDev& A, const CsrDev& Bm, int64_t dim, int*& rp_d, int*& ci_d,
                            double2*& val_d, int64_t& rows, int64_t& cap, int64_t& nnz_out, double* lo, double* hi,
                            hipStream_t s) {
  // count pass: per-row sizes in a work vector, the overflow flag in the scan buffer
  int* counts = reinterpret_cast<int*>(ctx->vec(kV));
  int* overflow = reinterpret_cast<int*>(ctx->scan);
  HIP_TRY(hipMemsetAsync(overflow, 0, sizeof(int), s));
  HIP_TRY(magnus::launch_csr_commutator(false, A, Bm, (int)dim, counts, nullptr, nullptr, nullptr, overflow, s));
  std::vector<int> cnt((size_t)dim);
  int ovf = 0;
  HIP_TRY(hipMemcpyAsync(cnt.data(), counts, sizeof(int) * cnt.size(), hipMemcpyDeviceToHost, s));
  HIP_TRY(hipMemcpyAsync(&ovf, overflow, sizeof(int), hipMemcpyDeviceToHost, s));
  HIP_TRY(hipStreamSynchronize(s));
  if (ovf)
    return fail(MAGNUS_ENOMEM, "a row of A B - B A lists more than %d products (use the matrix-free commutator)",
                magnus::kCommCap);
  std::vector<int> rp((size_t)dim + 1, 0);
  for (int64_t r = 0; r < dim; ++r) {
    if ((int64_t)rp[r] + cnt[r] > INT32_MAX) return fail(MAGNUS_ENOMEM, "the commutator has more than 2^31 entries");
    rp[r + 1] = rp[r] + cnt[r];
  }
  const int64_t nnz = rp[dim];
  if (rows < dim || cap < std::max<int64_t>(nnz, 1)) {
    HIP_TRY(hipStreamSynchronize(s));
    if (rp_d) HIP_TRY(hipFree(rp_d));
    if (ci_d) HIP_TRY(hipFree(ci_d));
    if (val_d) HIP_TRY(hipFree(val_d));
    rp_d = nullptr;
    ci_d = nullptr;
    val_d = nullptr;
    rows = cap = 0;
    HIP_TRY(hipMalloc(&rp_d, sizeof(int) * (size_t)(dim + 1)));
    HIP_TRY(hipMalloc(&ci_d, sizeof(int) * (size_t)std::max<int64_t>(nnz, 1)));
    HIP_TRY(hipMalloc(&val_d, sizeof(double2) * (size_t)std::max<int64_t>(nnz, 1)));
    rows = dim;
    cap = std::max<int64_t>(nnz, 1);
  }
  HIP_TRY(hipMemcpyAsync(rp_d, rp.data(), sizeof(int) * rp.size(), hipMemcpyHostToDevice, s));
  HIP_TRY(magnus::launch_csr_commutator(true, A, Bm, (int)dim, counts, rp_d, ci_d, val_d, overflow, s));
  nnz_out = nnz;
  magnus_term kt{};
  kt.format = MAGNUS_CSR;
  kt.dim = dim;
  kt.nnz = nnz;
  kt.row_ptr = rp_d;
  kt.col_idx = ci_d;
  kt.val = val_d;
  const magnus_term* const one[1] = {&kt};
  return csr_scan(ctx, one, 1, s, lo, hi);
}

int magnus_csr_commutator(magnus_ctx* ctx, magnus_hamiltonian* h, magnus_stream stream) {
  if (!ctx || !h) return fail(MAGNUS_EINVAL, "null argument");
  int rc = check_ham(ctx, h, 0);
  if (rc) return rc;
  if (h->H1.format != MAGNUS_CSR) return fail(MAGNUS_EINVAL, "magnus_csr_commutator needs CSR terms");
  hipStream_t s = (hipStream_t)stream;
  HIP_TRY(hipSetDevice(ctx->device));
  if ((rc = ensure_valid(ctx, h, s))) return rc;
  const int64_t dim = h->H1.dim;
  CsrDev A{h->H1.row_ptr, h->H1.col_idx, reinterpret_cast<const double2*>(h->H1.val)};
  CsrDev Bm{h->H2.row_ptr, h->H2.col_idx, reinterpret_cast<const double2*>(h->H2.val)};
  ctx->kc_key = std::make_tuple(nullptr, nullptr, nullptr, nullptr, (int64_t)0);
  double lo, hi;
  if ((rc = assemble_csr_commutator(ctx, A, Bm, dim, ctx->kc_rp, ctx->kc_ci, ctx->kc_val, ctx->kc_rows, ctx->kc_cap,
                                    ctx->kc_nnz, &lo, &hi, s)))
    return rc;
  h->k_min = lo;
  h->k_max = hi;
  if ((rc = probe_coding(ctx, h, true, &ctx->kc_codable, s))) return rc;
  ctx->kc_key = std::make_tuple((const void*)h->H1.row_ptr, h->H1.val, (const void*)h->H2.row_ptr, h->H2.val, dim);
  return MAGNUS_OK;
}

int magnus_csr_m6_prepare(magnus_ctx* ctx, magnus_hamiltonian* h, magnus_stream stream) {
  int rc = magnus_csr_commutator(ctx, h, stream);
  if (rc) return rc;
  hipStream_t s = (hipStream_t)stream;
  const int64_t dim = h->H1.dim;
  ctx->pm_key = std::make_tuple(nullptr, nullptr, nullptr, nullptr, (int64_t)0);
  const CsrDev K{ctx->kc_rp, ctx->kc_ci, ctx->kc_val};
  const CsrDev H[2] = {CsrDev{h->H1.row_ptr, h->H1.col_idx, reinterpret_cast<const double2*>(h->H1.val)},
                       CsrDev{h->H2.row_ptr, h->H2.col_idx, reinterpret_cast<const double2*>(h->H2.val)}};
  for (int a = 0; a < 2; ++a)  // P_a = -i[H_a, K] = i[K, H_a]
    if ((rc = assemble_csr_commutator(ctx, K, H[a], dim, ctx->pm_rp[a], ctx->pm_ci[a], ctx->pm_val[a],
                                      ctx->pm_rows[a], ctx->pm_cap[a], ctx->pm_nnz[a], &ctx->pm_lo[a],
                                      &ctx->pm_hi[a], s)))
      return rc;
  if (!m6_two_passes(ctx, h))  // P_1 and P_2 were assembled for their enclosures only
    for (int a = 0; a < 2; ++a) {
      {
        std::lock_guard<std::mutex> g(ctx->mu);
        ctx->validated.erase(std::make_tuple((const void*)ctx->pm_rp[a], (const void*)ctx->pm_ci[a],
                                             (const void*)ctx->pm_val[a], dim, ctx->pm_nnz[a]));
      }
      HIP_TRY(hipFree(ctx->pm_rp[a]));
      HIP_TRY(hipFree(ctx->pm_ci[a]));
      HIP_TRY(hipFree(ctx->pm_val[a]));
      ctx->pm_rp[a] = ctx->pm_ci[a] = nullptr;
      ctx->pm_val[a] = nullptr;
      ctx->pm_rows[a] = ctx->pm_cap[a] = 0;
    }
  if (ctx->pm_ws_dim < dim) {
    HIP_TRY(hipStreamSynchronize(s));
    if (ctx->pm_ws) HIP_TRY(hipFree(ctx->pm_ws));
    ctx->pm_ws = nullptr;
    ctx->pm_ws_dim = 0;
    HIP_TRY(hipMalloc(&ctx->pm_ws, magnus::kM6Vecs * sizeof(double2) * (size_t)dim));
    ctx->pm_ws_dim = dim;
  }
  ctx->pm_key = ctx->kc_key;
  return MAGNUS_OK;
}

int magnus_dense_m6_prepare(magnus_ctx* ctx, magnus_hamiltonian* h, magnus_stream stream) {
  int rc = magnus_dense_commutator(ctx, h, stream);
  if (rc) return rc;
  const int64_t dim = h->H1.dim;
  hipStream_t s = (hipStream_t)stream;
  if (ctx->m6_dim < dim) {
    if (ctx->m6) {
      HIP_TRY(hipDeviceSynchronize());
      HIP_TRY(hipFree(ctx->m6));
      ctx->m6 = nullptr;
      ctx->m6_dim = 0;
    }
    HIP_TRY(hipMalloc(&ctx->m6, 7 * sizeof(double2) * (size_t)dim * (size_t)dim));
    ctx->m6_dim = dim;
  }
  const size_t sz = (size_t)ctx->m6_dim * (size_t)ctx->m6_dim;
  double2* M = ctx->m6;
  double2* P1 = M;
  double2* P2 = M + sz;
  const double2* H1 = reinterpret_cast<const double2*>(h->H1.val);
  const double2* H2 = reinterpret_cast<const double2*>(h->H2.val);
  const long long ld = h->H1.ld;
  // (left, ld, right, ld, scale, out): out = scale i [left, right], the GEMM product in the assembly buffer
  struct Job {
    const double2* a;
    long long lda;
    const double2* b;
    long long ldb;
    double scale;
    double2* out;
  };
  const Job jobs[7] = {{H1, ld, ctx->comm, dim, -1.0, P1},           // P1 = -i[H1, K]
                       {H2, ld, ctx->comm, dim, -1.0, P2},           // P2 = -i[H2, K]
                       {H1, ld, P1, dim, 1.0, M + 2 * sz},           // U11 = i[H1, P1]
                       {H1, ld, P2, dim, 1.0, M + 3 * sz},           // U12 = i[H1, P2]
                       {H2, ld, P2, dim, 1.0, M + 4 * sz},           // U22 = i[H2, P2]
                       {ctx->comm, dim, P1, dim, -1.0, M + 5 * sz},  // R1 = -i[K, P1]
                       {ctx->comm, dim, P2, dim, -1.0, M + 6 * sz}}; // R2 = -i[K, P2]
  for (int j = 0; j < 7; ++j) {
    HIP_TRY(magnus::launch_zgemm(jobs[j].a, jobs[j].lda, jobs[j].b, jobs[j].ldb, ctx->assembled, (int)dim, s));
    HIP_TRY(magnus::launch_commutator_combine(ctx->assembled, (int)dim, jobs[j].scale, jobs[j].out, s));
    magnus_term t{};
    t.format = MAGNUS_DENSE;
    t.dim = dim;
    t.ld = dim;
    t.val = jobs[j].out;
    if ((rc = dense_scan(ctx, t, s, &ctx->m6_lo[j], &ctx->m6_hi[j]))) return rc;
  }
  ctx->m6_ready = true;
  return MAGNUS_OK;
}

}  // extern "C"

namespace {
// Dense terms: the GEMV iteration with 1, 2 and 4 rows per wave (two terms),
// and for batches the FP64-MFMA group iteration with each tile shape on the
// batch's states (one term, as a shared field assembles the exponent, when
// the context holds an assembly buffer; else two), 5 timed launches each.
int autotune_dense(magnus_ctx* ctx, const magnus_hamiltonian* h, int32_t batch, int32_t* variant, int32_t* group,
                   double* variant_us, double* group_us, hipStream_t s) {
  int rc = begin_call(ctx, s);
  if (rc) return rc;
  const int dim = (int)h->H1.dim;
  const size_t nvec = (size_t)ctx->max_dim * (size_t)ctx->max_batch;
  for (int k : {kA, kB, kS0, kY}) HIP_TRY(hipMemsetAsync(ctx->vec(k), 0, sizeof(double2) * nvec, s));
  const double2* D1 = reinterpret_cast<const double2*>(h->H1.val);
  const double2* D2 = reinterpret_cast<const double2*>(h->H2.val);
  hipEvent_t e0, e1;
  HIP_TRY(hipEventCreate(&e0));
  HIP_TRY(hipEventCreate(&e1));
  constexpr int kReps = 5;
  auto time_us = [&](auto f, double* us) -> hipError_t {
    hipError_t e = f();
    if (e == hipSuccess) e = hipEventRecord(e0, s);
    for (int r = 0; r < kReps && e == hipSuccess; ++r) e = f();
    if (e == hipSuccess) e = hipEventRecord(e1, s);
    if (e == hipSuccess) e = hipEventSynchronize(e1);
    float ms = 0.0f;
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
    *us = 1e3 * (double)ms / kReps;
    return e;
  };
  hipError_t err = hipSuccess;
  IterArgs a{};
  a.x1 = a.x2 = a.wcur = ctx->vec(kA);
  a.wout = ctx->vec(kB);
  a.pacc = ctx->vec(kS0);
  a.slot = ctx->slots;
  a.partials = ctx->partials;
  a.a1 = a.a2 = 1.0;
  a.first = 1;
  int best_rpw = 2;
  double best = INFINITY;
  const int rpws[3] = {1, 2, 4};
  for (int q = 0; q < 3 && err == hipSuccess; ++q) {
    double us = 0.0;
    err = time_us([&] { return magnus::launch_dense2_iter(D1, D2, dim, h->H1.ld, a, s, rpws[q]); }, &us);
    if (variant_us) variant_us[q] = us;
    if (us < best) {
      best = us;
      best_rpw = rpws[q];
    }
  }
  if (variant_us)
    for (int q = 3; q < kTuneVariants; ++q) variant_us[q] = NAN;
  int best_tile = 0;
  double best_t = INFINITY;
  if (err == hipSuccess && batch > 1) {
    std::vector<ColParam> table(batch);
    for (ColParam& c : table) c.a1 = c.a2 = 1.0;
    if ((rc = upload_table(ctx, table, s))) {
      (void)hipEventDestroy(e0);
      (void)hipEventDestroy(e1);
      return rc;
    }
    const bool one = ctx->assembled && ctx->assembled_dim >= dim;
    for (int t = 0; t < magnus::kMfmaTiles && err == hipSuccess; ++t) {
      MultiArgs m{};
      m.x = ctx->vec(kY);
      m.wout = ctx->vec(kA);
      m.pacc = ctx->vec(kB);
      m.slots = ctx->slots;
      m.partials = ctx->partials;
      m.prm = ctx->table;
      m.B = batch;
      m.first = 1;
      double us = 0.0;
      const int split = mfma_split(ctx, dim, m.B, t);
      err = time_us([&] { return magnus::launch_dense_mfma(one ? 1 : 2, D1, D2, h->H1.ld, dim, m, s, t, split, ctx->split); }, &us);
      if (group_us) group_us[t] = us;
      if (us < best_t) {
        best_t = us;
        best_tile = t;
      }
    }
  } else if (group_us) {
    for (int t = 0; t < magnus::kMfmaTiles; ++t) group_us[t] = NAN;
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (err != hipSuccess) return fail(MAGNUS_EHIP, "autotune: %s", hipGetErrorString(err));
  const auto key = std::make_pair(h->H1.val, h->H1.dim);
  ctx->tuned_dense_rpw[key] = best_rpw;
  if (batch > 1) ctx->tuned_mfma[key] = best_tile;
  if (variant) *variant = best_rpw;
  if (group) *group = batch > 1 ? best_tile : 0;
  return MAGNUS_OK;
}
}  // namespace

extern "C" {

int magnus_autotune(magnus_ctx* ctx, const magnus_hamiltonian* h, int32_t batch, int32_t* variant,
                    int32_t* group, double* variant_us, double* group_us, magnus_stream stream) {
  int rc = check_ham(ctx, h, 0);
  if (rc) return rc;
  if ((rc = check_batch(ctx, batch))) return rc;
  hipStream_t s = (hipStream_t)stream;
  if (h->H1.format == MAGNUS_DENSE) return autotune_dense(ctx, h, batch, variant, group, variant_us, group_us, s);
  if ((rc = begin_call(ctx, s))) return rc;
  if ((rc = ensure_valid(ctx, h, s))) return rc;
  const int dim = (int)h->H1.dim;
  const size_t nvec = (size_t)ctx->max_dim * (size_t)ctx->max_batch;
  for (int k : {kA, kB, kS0, kY})
    HIP_TRY(hipMemsetAsync(ctx->vec(k), 0, sizeof(double2) * nvec, s));
  CsrDev t1{h->H1.row_ptr, h->H1.col_idx, reinterpret_cast<const double2*>(h->H1.val)};
  CsrDev t2{h->H2.row_ptr, h->H2.col_idx, reinterpret_cast<const double2*>(h->H2.val)};
  hipEvent_t e0, e1;
  HIP_TRY(hipEventCreate(&e0));
  HIP_TRY(hipEventCreate(&e1));
  constexpr int kReps = 5;
  // time f (kReps launches after one untimed launch), in microseconds per launch
  auto time_us = [&](auto f, double* us) -> hipError_t {
    hipError_t e = f();
    if (e == hipSuccess) e = hipEventRecord(e0, s);
    for (int r = 0; r < kReps && e == hipSuccess; ++r) e = f();
    if (e == hipSuccess) e = hipEventRecord(e1, s);
    if (e == hipSuccess) e = hipEventSynchronize(e1);
    float ms = 0.0f;
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
    *us = 1e3 * (double)ms / kReps;
    return e;
  };
  hipError_t err = hipSuccess;
  // the single-state iteration: each row mapping on this matrix, with its stop
  // test (made by the iteration from the partial sums of the one before, or on
  // larger grids by the decide kernel after it), then the coded terms
  HIP_TRY(hipMemsetAsync(ctx->partials, 0, sizeof(double) * ctx->npartials, s));
  IterArgs a{};
  a.x1 = a.x2 = a.wcur = ctx->vec(kA);
  a.wout = ctx->vec(kB);
  a.pacc = ctx->vec(kS0);
  a.slot = ctx->slots;
  a.a1 = a.a2 = 1.0;
  a.check_stop = 1;
  a.iter = 3;
  auto stop_test = [&](int grid, int limit) {
    a.fused = ctx->fuse && grid <= limit;
    a.partials = ctx->partials;
    a.prev_partials = ctx->partials + 2 * (size_t)ctx->max_grid;
    a.prev_grid = grid;
  };
  double best = INFINITY;
  int best_code = 0;
  for (int code = 0; code <= kTuneVariants && err == hipSuccess; ++code) {  // (0: the first one again, to warm up)
    const int rpb = variant_rows(std::max(code, 1), dim);
    const int grid = magnus::csr2_grid(dim, rpb);
    double us = 0.0;
    stop_test(grid, magnus::csr2_fuse_grid(rpb));
    err = time_us(
        [&] {
          hipError_t e = magnus::launch_csr2_iter(magnus::kLeja, t1, t2, dim, a, rpb, s);
          if (e == hipSuccess && !a.fused) e = magnus::launch_leja_decide(a, grid, s);
          return e;
        },
        &us);
    if (code == 0) continue;
    if (variant_us) variant_us[code - 1] = us;
    if (us < best) {
      best = us;
      best_code = code;
    }
  }
  const auto key = std::make_pair((const void*)h->H1.row_ptr, h->H1.dim);
  const bool coded = coding_possible(ctx, h) && ctx->codable.count(pair_key(h));
  const magnus::CodeTerms T{2, {t1, t2}};
  ctx->uncoded_single.erase(key);
  if (err == hipSuccess && coded) {
    ctx->coded.rows = magnus::code_rows(dim);
    const int grid = magnus::code_grid(dim, ctx->coded.rows);
    stop_test(grid, magnus::kFuseMaxGrid);
    err = magnus::launch_code_build(T, dim, ctx->coded, nullptr, s);
    double us = 0.0;
    if (err == hipSuccess)
      err = time_us(
          [&] {
            hipError_t e = magnus::launch_coded_iter(magnus::kLeja, T, dim, ctx->coded, a, 0.0, s);
            if (e == hipSuccess && !a.fused) e = magnus::launch_leja_decide(a, grid, s);
            return e;
          },
          &us);
    if (err == hipSuccess && best < us) ctx->uncoded_single.insert(key);
  }
  // the multi-state iteration with its decisions: cost per state of each group
  // size up to the batch, then of pairs on the coded terms
  int best_group = 32;
  double best_per_state = INFINITY;
  std::vector<ColParam> table(32);
  for (ColParam& c : table) c.a1 = c.a2 = 1.0;
  if (err == hipSuccess && batch > 1) {
    if ((rc = upload_table(ctx, table, s))) {
      (void)hipEventDestroy(e0);
      (void)hipEventDestroy(e1);
      return rc;
    }
  }
  int gi = 0;
  for (int g : {2, 4, 8, 16, 32}) {
    double us = NAN;
    const int grid = magnus::csr2_multi_grid(dim, g);
    if (err == hipSuccess && g <= batch && (size_t)grid * g * 2 <= ctx->npartials) {
      MultiArgs m{};
      m.x = ctx->vec(kY);
      m.wout = ctx->vec(kA);
      m.pacc = ctx->vec(kB);
      m.slots = ctx->slots;
      m.partials = ctx->partials;
      m.prm = ctx->table;
      m.B = g;
      m.check_stop = 1;
      err = time_us(
          [&] {
            hipError_t e = magnus::launch_csr2_multi(magnus::kMultiLeja, t1, t2, dim, m, s);
            return e == hipSuccess ? magnus::launch_multi_decide(m, grid, s) : e;
          },
          &us);
      if (err == hipSuccess && us / g < best_per_state) {
        best_per_state = us / g;
        best_group = g;
      }
    }
    if (group_us) group_us[gi] = us;
    ++gi;
  }
  const int npairs = std::min(batch / 2, 16);
  if (batch > 1) ctx->uncoded_batch.erase(key);
  if (err == hipSuccess && coded && npairs > 0 && ctx->fuse) {
    ctx->coded.rows = batch_rows(h, batch);
    const int64_t blocks = (int64_t)magnus::code_grid(dim, ctx->coded.rows) * npairs;
    if (pair_partials_fit(ctx, blocks)) {
      magnus::PairArgs A{};
      A.np = 1;
      magnus::PairProblem& P = A.p[0];
      P.t1 = t1;
      P.t2 = t2;
      P.C = ctx->coded;
      P.dim = dim;
      P.npairs = npairs;
      P.x = ctx->vec(kY);
      P.wout = ctx->vec(kA);
      P.pacc = ctx->vec(kB);
      P.slots = ctx->slots;
      P.partials = ctx->partials + pair_partials_at(ctx);
      P.prev_partials = P.partials + 4 * (size_t)blocks;
      P.prm = P.prev = ctx->table;
      P.iter = 3;
      err = hipMemsetAsync(P.partials, 0, sizeof(double) * 8 * (size_t)blocks, s);
      if (err == hipSuccess) err = magnus::launch_code_build(T, dim, ctx->coded, nullptr, s);
      double us = 0.0;
      if (err == hipSuccess) err = time_us([&] { return magnus::launch_coded_pairs(false, A, s); }, &us);
      if (err == hipSuccess && best_per_state < us / (2 * npairs)) ctx->uncoded_batch.insert(key);
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (err != hipSuccess) return fail(MAGNUS_EHIP, "autotune: %s", hipGetErrorString(err));
  ctx->tuned_variant[key] = best_code;
  if (batch > 1) ctx->tuned_group[key] = best_group;
  if (variant) *variant = best_code;
  if (group) *group = batch > 1 ? best_group : 1;
  return MAGNUS_OK;
}

int magnus_destroy(magnus_ctx* ctx) {
  if (!ctx) return MAGNUS_OK;
  (void)hipSetDevice(ctx->device);
  if (ctx->vecs) (void)hipFree(ctx->vecs);
  if (ctx->slots) (void)hipFree(ctx->slots);
  if (ctx->table) (void)hipFree(ctx->table);
  if (ctx->arena) (void)hipFree(ctx->arena);
  if (ctx->assembled) (void)hipFree(ctx->assembled);
  if (ctx->comm) (void)hipFree(ctx->comm);
  if (ctx->m6) (void)hipFree(ctx->m6);
  if (ctx->kc_rp) (void)hipFree(ctx->kc_rp);
  if (ctx->kc_ci) (void)hipFree(ctx->kc_ci);
  if (ctx->kc_val) (void)hipFree(ctx->kc_val);
  for (int a = 0; a < 2; ++a) {
    if (ctx->pm_rp[a]) (void)hipFree(ctx->pm_rp[a]);
    if (ctx->pm_ci[a]) (void)hipFree(ctx->pm_ci[a]);
    if (ctx->pm_val[a]) (void)hipFree(ctx->pm_val[a]);
  }
  if (ctx->pm_ws) (void)hipFree(ctx->pm_ws);
  if (ctx->partials) (void)hipFree(ctx->partials);
  if (ctx->scan) (void)hipFree(ctx->scan);
  if (ctx->split) (void)hipFree(ctx->split);
  if (ctx->graph_x || ctx->graph_g) {
    if (ctx->graph_done) (void)hipEventSynchronize(ctx->graph_done);
    graph_release(ctx);
  }
  if (ctx->graph_done) (void)hipEventDestroy(ctx->graph_done);
  if (ctx->seen_at) {
    (void)hipEventSynchronize(ctx->seen_at);
    (void)hipEventDestroy(ctx->seen_at);
  }
  if (ctx->seen) (void)hipHostFree(ctx->seen);
  if (ctx->cap_stream) (void)hipStreamDestroy(ctx->cap_stream);
  if (ctx->gctr) (void)hipFree(ctx->gctr);
  release_coded(ctx);
  for (hipEvent_t e : ctx->pool) (void)hipEventDestroy(e);
  delete ctx;
  return MAGNUS_OK;
}

int magnus_check(magnus_ctx* ctx, magnus_stream stream) {
  if (!ctx) return fail(MAGNUS_EINVAL, "null context");
  hipStream_t s = (hipStream_t)stream;
  HIP_TRY(hipSetDevice(ctx->device));
  long long iters = 0;
  int status = 0;
  int rc = read_slots(ctx, s, &iters, &status);
  if (rc) return rc;
  status |= ctx->sticky_status;
  if (status & 1) return fail(MAGNUS_ENAN, "non-finite vector norm met on the device");
  return MAGNUS_OK;
}

int magnus_spectral_bounds(magnus_ctx* ctx, magnus_hamiltonian* h, magnus_stream stream) {
  if (!ctx || !h) return fail(MAGNUS_EINVAL, "null argument");
  hipStream_t s = (hipStream_t)stream;
  HIP_TRY(hipSetDevice(ctx->device));
  const int64_t dim = h->H1.dim;
  if (dim < 1 || dim > ctx->max_dim) return fail(dim < 1 ? MAGNUS_EINVAL : MAGNUS_ENOMEM, "dim %lld", (long long)dim);
  // the enclosures are not yet known: validate the rest of the terms only
  auto check = [&](magnus_term& t, const char* name) {
    const double l0 = t.lam_min, u0 = t.lam_max;
    t.lam_min = 0.0;
    t.lam_max = 0.0;
    const int rc = check_term(t, dim, name);
    t.lam_min = l0;
    t.lam_max = u0;
    return rc;
  };
  if (int rc = check(h->H1, "H1")) return rc;
  double lo[2], hi[2];
  auto set = [&](magnus_term& t, int k) {
    t.lam_min = lo[k];
    t.lam_max = hi[k];
  };
  if (h->H1.format == MAGNUS_CSR && h->H2.format == MAGNUS_CSR && !check(h->H2, "H2")) {  // both with one wait
    const magnus_term* const terms[2] = {&h->H1, &h->H2};
    int valid = 0;
    bool fits = false;
    const int rc = csr_scan(ctx, terms, 2, s, lo, hi, &valid, h, &fits);
    if (valid > 0) set(h->H1, 0);
    note_codable(ctx, h, fits);
    if (rc) return rc;
    set(h->H2, 1);
  } else {
    for (magnus_term* t : {&h->H1, &h->H2}) {
      int rc = t == &h->H2 ? check(h->H2, "H2") : MAGNUS_OK;
      if (rc) return rc;
      const magnus_term* const one[1] = {t};
      rc = (t->format == MAGNUS_CSR) ? csr_scan(ctx, one, 1, s, lo, hi) : dense_scan(ctx, *t, s, lo, hi);
      if (rc) return rc;
      set(*t, 0);
    }
  }
  const double n1 = std::fmax(std::fabs(h->H1.lam_min), std::fabs(h->H1.lam_max));
  const double n2 = std::fmax(std::fabs(h->H2.lam_min), std::fabs(h->H2.lam_max));
  h->k_min = -2.0 * n1 * n2;
  h->k_max = 2.0 * n1 * n2;
  return MAGNUS_OK;
}

namespace {

// y = H x for one term (the iteration kernels with the other term empty or absent).
int apply_term(magnus_ctx* ctx, const magnus_term& t, const double2* x, double2* y, hipStream_t s) {
  const int dim = (int)t.dim;
  IterArgs a{};
  a.x1 = a.x2 = a.wcur = x;
  a.wout = y;
  a.pacc = ctx->vec(kS1);
  a.slot = ctx->slots;
  a.partials = ctx->partials;
  a.a1 = 1.0;
  a.first = 1;
  if (t.format == MAGNUS_DENSE) {
    HIP_TRY(magnus::launch_dense2_iter(reinterpret_cast<const double2*>(t.val), nullptr, dim, t.ld, a, s));
    return MAGNUS_OK;
  }
  CsrDev t1{t.row_ptr, t.col_idx, reinterpret_cast<const double2*>(t.val)};
  CsrDev none{reinterpret_cast<const int*>(ctx->vec(kV)), nullptr, nullptr};  // all rows empty
  HIP_TRY(magnus::launch_csr2_iter(magnus::kLeja, t1, none, dim, a, variant_rows(0, dim), s));
  return MAGNUS_OK;
}

// Re(x^H y) on the host (one device dot product and a wait).
int dot_re(magnus_ctx* ctx, const double2* x, const double2* y, int64_t n, double* out, hipStream_t s) {
  double2* dev_out = reinterpret_cast<double2*>(ctx->dots + magnus::kDotPartials);
  HIP_TRY(magnus::launch_cdot(x, 1, y, 1, n, ctx->dots, dev_out, s));
  double2 h;
  HIP_TRY(hipMemcpyAsync(&h, dev_out, sizeof(double2), hipMemcpyDeviceToHost, s));
  HIP_TRY(hipStreamSynchronize(s));
  *out = h.x;
  return MAGNUS_OK;
}

// Lanczos on one Hermitian term from a fixed pseudo-random start: extreme Ritz
// values after `steps` steps and their change over the last steps.
int lanczos_term(magnus_ctx* ctx, const magnus_term& t, int steps, double* lo, double* hi, double* drift,
                 hipStream_t s) {
  const int64_t n = t.dim;
  double2* P = ctx->vec(kA);  // previous basis vector
  double2* C = ctx->vec(kB);  // current basis vector
  double2* W = ctx->vec(kS0);
  HIP_TRY(hipMemsetAsync(ctx->vec(kV), 0, sizeof(int) * (size_t)(n + 1), s));
  HIP_TRY(hipMemsetAsync(P, 0, sizeof(double2) * (size_t)n, s));
  {
    // start vector: splitmix64 stream mapped to [-1, 1)^2, normalised on the host
    std::vector<double2> v0((size_t)n);
    uint64_t z = 0x9E3779B97F4A7C15ull;
    double nrm = 0.0;
    auto next = [&z]() {
      z += 0x9E3779B97F4A7C15ull;
      uint64_t r = z;
      r = (r ^ (r >> 30)) * 0xBF58476D1CE4E5B9ull;
      r = (r ^ (r >> 27)) * 0x94D049BB133111EBull;
      r ^= r >> 31;
      return (double)(r >> 11) * (2.0 / 9007199254740992.0) - 1.0;
    };
    for (auto& e : v0) {
      e.x = next();
      e.y = next();
      nrm += e.x * e.x + e.y * e.y;
    }
    const double inv = 1.0 / std::sqrt(nrm);
    for (auto& e : v0) {
      e.x *= inv;
      e.y *= inv;
    }
    HIP_TRY(hipMemcpyAsync(C, v0.data(), sizeof(double2) * v0.size(), hipMemcpyHostToDevice, s));
    HIP_TRY(hipStreamSynchronize(s));
  }
  std::vector<double> al, be;
  double beta_prev = 0.0, lo_prev = 0.0, hi_prev = 0.0;
  *drift = 0.0;
  const int k = (int)std::min<int64_t>(steps, n);
  for (int j = 0; j < k; ++j) {
    int rc = apply_term(ctx, t, C, W, s);
    if (rc) return rc;
    double alpha, beta2;
    if ((rc = dot_re(ctx, C, W, n, &alpha, s))) return rc;
    HIP_TRY(magnus::launch_lanczos_orth(W, C, P, alpha, beta_prev, n, s));
    if ((rc = dot_re(ctx, W, W, n, &beta2, s))) return rc;
    al.push_back(alpha);
    const double beta = std::sqrt(std::max(beta2, 0.0));
    if (!std::isfinite(alpha) || !std::isfinite(beta)) return fail(MAGNUS_ENAN, "Lanczos met a non-finite value");
    if (j + 1 == k || beta <= 1e-13 * (std::fabs(alpha) + 1.0)) break;  // done, or an invariant subspace
    be.push_back(beta);
    HIP_TRY(magnus::launch_scale(W, 1.0 / beta, P, n, s));  // P becomes the next vector
    std::swap(P, C);
    beta_prev = beta;
    if (j + 1 == k - 10) magnus::tridiag_extremes(al, be, &lo_prev, &hi_prev);
  }
  be.resize(al.size() - 1);
  magnus::tridiag_extremes(al, be, lo, hi);
  if ((int)al.size() > 10) *drift = std::max(std::fabs(*lo - lo_prev), std::fabs(*hi - hi_prev));
  return MAGNUS_OK;
}

}  // namespace

int magnus_spectral_bounds_lanczos(magnus_ctx* ctx, magnus_hamiltonian* h, int32_t steps, double margin,
                                   magnus_stream stream) {
  int rc = magnus_spectral_bounds(ctx, h, stream);  // validates; the Gershgorin enclosures cap the estimate
  if (rc) return rc;
  if (steps < 2 || !(margin >= 0.0)) return fail(MAGNUS_EINVAL, "steps %d < 2 or margin %g < 0", steps, margin);
  hipStream_t s = (hipStream_t)stream;
  for (magnus_term* t : {&h->H1, &h->H2}) {
    double lo, hi, drift;
    if ((rc = lanczos_term(ctx, *t, steps, &lo, &hi, &drift, s))) return rc;
    const double d = std::max(margin * (hi - lo), 3.0 * drift);
    t->lam_min = std::max(t->lam_min, lo - d);
    t->lam_max = std::min(t->lam_max, hi + d);
    if (t->lam_min > t->lam_max) t->lam_min = t->lam_max = 0.5 * (lo + hi);
  }
  const double n1 = std::fmax(std::fabs(h->H1.lam_min), std::fabs(h->H1.lam_max));
  const double n2 = std::fmax(std::fabs(h->H2.lam_min), std::fabs(h->H2.lam_max));
  h->k_min = -2.0 * n1 * n2;
  h->k_max = 2.0 * n1 * n2;
  return MAGNUS_OK;
}

int expmv_leja(magnus_ctx* ctx, const magnus_hamiltonian* h, double a, double b, double kappa, double tau,
               const void* v, void* w, int32_t batch, const magnus_leja_opts* opts, magnus_stats* stats,
               magnus_stream stream) {
  int rc = check_ham(ctx, h, kappa != 0.0);
  if (rc) return rc;
  if ((rc = check_opts(opts)) || (rc = check_batch(ctx, batch))) return rc;
  if (!v || !w) return fail(MAGNUS_EINVAL, "null state pointer");
  if (!is_fin(a) || !is_fin(b) || !is_fin(kappa) || !is_fin(tau))
    return fail(MAGNUS_EDOMAIN, "non-finite coefficient or step");
  if (kappa != 0.0 && h->H1.format != MAGNUS_CSR && !dense_comm_ready(ctx, h))
    return fail(MAGNUS_EINVAL, "dense commutator exponents need magnus_dense_commutator for this pair of terms");
  hipStream_t s = (hipStream_t)stream;
  if ((rc = begin_call(ctx, s))) return rc;
  if ((rc = ensure_valid(ctx, h, s))) return rc;
  const int64_t dim = h->H1.dim;
  const double tol_e = per_exp_tol(opts, 1);
  if (tau != 0.0)
    if ((rc = begin_coded(ctx, h, kappa != 0.0 && csr_comm_ready(ctx, h), kappa == 0.0 ? 1 : batch,
                          kappa == 0.0 ? batch : 0, s)))
      return rc;
  Acc acc;
  acc.products_per_iter = kappa != 0.0 ? 4 : 2;
  const double2* vin = reinterpret_cast<const double2*>(v);
  double2* wout = reinterpret_cast<double2*>(w);
  for (int32_t c = 0; c < batch;) {
    const int g = (multi_ok(h, kappa) && tau != 0.0) ? group_for(ctx, h, batch - c) : 1;
    if (g > 1) {
      std::vector<double> av(g, a), bv(g, b);
      rc = multi_expmv_group(ctx, h, g, av.data(), bv.data(), tau, vin + c * dim, wout + c * dim, tol_e, opts, &acc, s);
    } else {
      rc = run_exponential(ctx, ExpOp{h, a, b, kappa}, tau, vin + c * dim, wout + c * dim, tol_e, opts, &acc, s);
    }
    if (rc) return rc;
    c += g;
  }
  return end_call(ctx, acc, tol_e, stats, s);
}

// One step of small states in one launch, when that is faster than a launch
// per iteration: rows that the kernel holds in registers (chains, us per
// iteration, a launch each / in one launch: n = 6 4.4 / 0.9, n = 10 4.6 / 2.4;
// rows read from memory 5.2 and more), and iterations that fit the launch's
// arguments.  *done: whether it was launched.
static int small_step(magnus_ctx* ctx, const magnus_hamiltonian* h, const magnus::Scheme& S, double tau,
                      const double* f, const double2* in, double2* out, int batch, double tol_e,
                      const magnus_leja_opts* o, Acc* acc, bool* done, hipStream_t s) {
  *done = false;
  const int64_t dim = h->H1.dim;
  if (batch > ctx->nslots || !small_ok(ctx, h, batch) || ctx->csr_variant ||
      S.nexp > magnus::kPersistStepExps || !rows_in_registers(ctx, h))
    return MAGNUS_OK;
  magnus::PersistStep a{};
  std::vector<ColParam> table;
  Acc one;
  for (int k = 0; k < S.nexp; ++k) {
    if (int rc = persist_exponential(h, S.rho[k], scheme_b(S, k, f), tau, tol_e, o, &a.plan.exps[k], &table, &one))
      return rc;
    if (table.size() > (size_t)magnus::kPersistStepRecords) return MAGNUS_OK;
  }
  std::copy(table.begin(), table.end(), a.plan.table);
  a.problem.t1 = csr_dev(h->H1);
  a.problem.t2 = csr_dev(h->H2);
  a.problem.dim = (int)dim;
  a.in = in;
  a.out = out;
  a.slots = ctx->slots;
  a.nexp = S.nexp;
  a.early = o->early_termination;
  if (int rc = flush_fused_check(ctx, s)) return rc;
  HIP_TRY(timed(ctx, MAGNUS_KERNEL_PERSIST, s, [&] { return magnus::launch_persist_step(a, batch, s); }));
  acc->exponentials += one.exponentials * batch;
  acc->substeps += one.substeps * batch;
  acc->planned += one.planned * batch;
  acc->max_m = std::max(acc->max_m, one.max_m);
  acc->max_s = std::max(acc->max_s, one.max_s);
  acc->max_bound = std::max(acc->max_bound, one.max_bound);
  *done = true;
  return MAGNUS_OK;
}

static int step_common(int method, magnus_ctx* ctx, const magnus_hamiltonian* h, double tau, double f1,
                       double f2, const void* psi_in, void* psi_out, int32_t batch,
                       const magnus_leja_opts* opts, magnus_stats* stats, magnus_stream stream) {
  int rc = check_ham(ctx, h, method == MAGNUS_M4);
  if (rc) return rc;
  if ((rc = check_opts(opts)) || (rc = check_batch(ctx, batch))) return rc;
  if (!psi_in || !psi_out) return fail(MAGNUS_EINVAL, "null state pointer");
  if (!is_fin(tau) || !is_fin(f1) || !is_fin(f2)) return fail(MAGNUS_EDOMAIN, "non-finite step or field value");
  if (method == MAGNUS_M4 && h->H1.format != MAGNUS_CSR && !dense_comm_ready(ctx, h))
    return fail(MAGNUS_EINVAL, "M4 on dense terms needs magnus_dense_commutator for this pair of terms");
  hipStream_t s = (hipStream_t)stream;
  if ((rc = begin_call(ctx, s))) return rc;
  if ((rc = ensure_valid(ctx, h, s))) return rc;
  const int64_t dim = h->H1.dim;
  magnus::Scheme S;
  magnus::method_scheme(method, &S);
  const double fv[2] = {f1, f2};
  const double tol_e = per_exp_tol(opts, S.nexp);
  Acc acc;
  acc.products_per_iter = method == MAGNUS_M4 ? 4 : 2;
  const double2* in = reinterpret_cast<const double2*>(psi_in);
  double2* out = reinterpret_cast<double2*>(psi_out);
  if (tau != 0.0 && !S.commutator) {
    bool done = false;
    if ((rc = small_step(ctx, h, S, tau, fv, in, out, batch, tol_e, opts, &acc, &done, s))) return rc;
    if (done) return end_call(ctx, acc, tol_e, stats, s);
  }
  if (tau != 0.0)
    if ((rc = begin_coded(ctx, h, S.commutator && csr_comm_ready(ctx, h), S.commutator ? batch : S.nexp,
                          S.commutator ? 0 : batch, s)))
      return rc;
  for (int32_t c = 0; c < batch;) {
    const int g = (!S.commutator && multi_ok(h, 0.0)) ? group_for(ctx, h, batch - c) : 1;
    if (g > 1) {
      if ((rc = pack_group(ctx, h, in + c * dim, ctx->vec(kY), g, s))) return rc;
      rc = multi_cf_steps(ctx, h, S, g, tau, 0, 1, [&](int, int64_t, int j) { return fv[j]; }, tol_e, opts, &acc, s);
      if (rc) return rc;
      rc = unpack_group(ctx, h, ctx->vec(kY), out + c * dim, g, s);
    } else {
      rc = S.commutator ? m4_state(ctx, h, tau, f1, f2, in + c * dim, out + c * dim, tol_e, opts, &acc, s)
                        : cf_state(ctx, h, S, tau, fv, in + c * dim, out + c * dim, tol_e, opts, &acc, s);
    }
    if (rc) return rc;
    c += g;
  }
  return end_call(ctx, acc, tol_e, stats, s);
}

int magnus_step_cf4(magnus_ctx* ctx, const magnus_hamiltonian* h, double tau, double f1, double f2,
                    const void* psi_in, void* psi_out, int32_t batch, const magnus_leja_opts* opts,
                    magnus_stats* stats, magnus_stream stream) {
  return step_common(MAGNUS_CF4, ctx, h, tau, f1, f2, psi_in, psi_out, batch, opts, stats, stream);
}

int magnus_step_m4(magnus_ctx* ctx, const magnus_hamiltonian* h, double tau, double f1, double f2,
                   const void* psi_in, void* psi_out, int32_t batch, const magnus_leja_opts* opts,
                   magnus_stats* stats, magnus_stream stream) {
  return step_common(MAGNUS_M4, ctx, h, tau, f1, f2, psi_in, psi_out, batch, opts, stats, stream);
}

int magnus_step_cf4_noalloc(const magnus_hamiltonian* h, double tau, double f1, double f2, const void* psi_in,
                            void* psi_out, const magnus_leja_opts* opts, magnus_stats* stats, magnus_stream stream) {
  if (!h) return fail(MAGNUS_EINVAL, "null hamiltonian");
  if (h->H1.dim > kNoAllocMaxDim)
    return fail(MAGNUS_ENOMEM, "dim %lld exceeds the %lld entries the allocation-free scratch holds",
                (long long)h->H1.dim, (long long)kNoAllocMaxDim);
  magnus_ctx* ctx = nullptr;
  int rc = noalloc_context(&ctx);
  if (rc) return rc;
  return step_common(MAGNUS_CF4, ctx, h, tau, f1, f2, psi_in, psi_out, 1, opts, stats, stream);
}

int propagate(magnus_ctx* ctx, const magnus_hamiltonian* h, int32_t method, double tau, int64_t nsteps,
              const double* f_nodes, int32_t batch_f, void* psi, int32_t batch, void* checkpoints,
              int32_t every_k, const magnus_leja_opts* opts, magnus_stats* stats, magnus_stream stream) {
  magnus::Scheme S;
  if (!magnus::method_scheme(method, &S)) return fail(MAGNUS_EINVAL, "unknown method %d", method);
  int rc = check_ham(ctx, h, S.commutator);
  if (rc) return rc;
  if ((rc = check_opts(opts)) || (rc = check_batch(ctx, batch))) return rc;
  if (!psi) return fail(MAGNUS_EINVAL, "null state pointer");
  if (nsteps < 0) return fail(MAGNUS_EINVAL, "nsteps %lld < 0", (long long)nsteps);
  if (nsteps > 0 && !f_nodes) return fail(MAGNUS_EINVAL, "null f_nodes");
  if (batch_f != 1 && batch_f != batch) return fail(MAGNUS_EINVAL, "batch_f %d must be 1 or batch", batch_f);
  if (checkpoints && every_k < 1) return fail(MAGNUS_EINVAL, "every_k %d < 1", every_k);
  if (!is_fin(tau)) return fail(MAGNUS_EDOMAIN, "non-finite step");
  for (int64_t k = 0; k < S.q * nsteps * (int64_t)batch_f; ++k)
    if (!is_fin(f_nodes[k])) return fail(MAGNUS_EDOMAIN, "non-finite field value at node %lld", (long long)k);
  if (method == MAGNUS_M4 && h->H1.format != MAGNUS_CSR && !dense_comm_ready(ctx, h))
    return fail(MAGNUS_EINVAL, "M4 on dense terms needs magnus_dense_commutator for this pair of terms");
  if (S.sixth && !(h->H1.format == MAGNUS_DENSE ? dense_m6_ready(ctx, h) : csr_m6_ready(ctx, h)))
    return fail(MAGNUS_EINVAL, "M6 needs terms prepared by magnus_dense_m6_prepare or magnus_csr_m6_prepare");
  hipStream_t s = (hipStream_t)stream;
  if ((rc = begin_call(ctx, s))) return rc;
  if ((rc = ensure_valid(ctx, h, s))) return rc;
  const int64_t dim = h->H1.dim;
  const int64_t exps = S.nexp * nsteps;
  const double tol_e = per_exp_tol(opts, exps);
  Acc acc;
  acc.products_per_iter = method == MAGNUS_M4 ? 4 : 2;
  double2* st = reinterpret_cast<double2*>(psi);
  double2* ck = reinterpret_cast<double2*>(checkpoints);
  const int64_t nck = checkpoints ? (nsteps + every_k - 1) / every_k + 1 : 0;
  const size_t stride = (size_t)dim * (size_t)batch;
  if (ck) HIP_TRY(hipMemcpyAsync(ck, st, sizeof(double2) * stride, hipMemcpyDeviceToDevice, s));
  auto fval = [&](int c, int64_t n, int j) {
    return f_nodes[((batch_f == 1 ? 0 : (int64_t)c) * nsteps + n) * S.q + j];
  };
  const bool grouped = !S.commutator && multi_ok(h, 0.0) && batch > 1;
  const bool small = !S.commutator && small_ok(ctx, h, batch);
  std::vector<SmallState> sst;
  if (small)
    for (int32_t c = 0; c < batch; ++c)
      sst.push_back(SmallState{0, st + c * dim, f_nodes + (batch_f == 1 ? 0 : (int64_t)c) * nsteps * S.q});
  // checkpoint steps: multiples of every_k and the last step
  auto next_stop = [&](int64_t n) {
    if (!ck) return nsteps;
    const int64_t k = ((n / every_k) + 1) * every_k;
    return std::min(k, nsteps);
  };
  if (!small && tau != 0.0)
    if ((rc = begin_coded(ctx, h, S.commutator && csr_comm_ready(ctx, h),
                          exps * (S.commutator ? batch : 1), grouped ? batch : 0, s,
                          S.sixth ? CodeUse::kM6 : CodeUse::kSingle)))
      return rc;
  // one state on the grid path with every stop test fused: one step captured,
  // replayed once per step
  GraphPlan G;
  const bool use_graph = batch == 1 && !small && tau != 0.0 && nsteps >= 2 && graph_eligible(ctx, h, S);
  if (use_graph) {
    if ((rc = graph_plan(ctx, h, S, tau, nsteps, [&](int64_t k, int j) { return fval(0, k, j); }, tol_e, opts, &G)))
      return rc;
    if ((rc = flush_fused_check(ctx, s))) return rc;
    if ((rc = graph_capture(ctx, h, S, G, st, tol_e, opts->early_termination))) return rc;
  }
  int64_t n = 0;
  while (n < nsteps) {
    const int64_t stop = next_stop(n);
    if (small) {
      rc = persist_steps(ctx, {h}, sst, S, tau, n, stop, tol_e, opts, &acc, s);
      if (rc) return rc;
    }
    for (int32_t c = small ? batch : 0; c < batch;) {
      const int g = grouped ? group_for(ctx, h, batch - c) : 1;
      if (g > 1) {
        if ((rc = pack_group(ctx, h, st + c * dim, ctx->vec(kY), g, s))) return rc;
        rc = multi_cf_steps(ctx, h, S, g, tau, n, stop,
                            [&](int cc, int64_t k, int j) { return fval(c + cc, k, j); }, tol_e, opts, &acc, s);
        if (rc) return rc;
        if ((rc = unpack_group(ctx, h, ctx->vec(kY), st + c * dim, g, s))) return rc;
      } else if (use_graph) {
        if ((rc = graph_replay(ctx, G, tau, n, stop, tol_e, opts, &acc, s))) return rc;
      } else {
        for (int64_t k = n; k < stop; ++k) {
          double2* y = st + c * dim;
          double fv[3];
          for (int j = 0; j < S.q; ++j) fv[j] = fval(c, k, j);
          rc = S.sixth        ? m6_state(ctx, h, tau, fv, y, y, tol_e, opts, &acc, s)
               : S.commutator ? m4_state(ctx, h, tau, fv[0], fv[1], y, y, tol_e, opts, &acc, s)
                              : cf_state(ctx, h, S, tau, fv, y, y, tol_e, opts, &acc, s);
          if (rc) return rc;
        }
      }
      c += g;
    }
    n = stop;
    if (ck) {
      const int64_t slot = n % every_k == 0 ? n / every_k : nck - 1;
      HIP_TRY(hipMemcpyAsync(ck + slot * stride, st, sizeof(double2) * stride, hipMemcpyDeviceToDevice, s));
    }
  }
  return end_call(ctx, acc, tol_e, stats, s);
}

int magnus_timing(magnus_ctx* ctx, int32_t enable) {
  if (!ctx) return fail(MAGNUS_EINVAL, "null context");
  if (enable < 0) return fail(MAGNUS_EINVAL, "timing stride %d", enable);
  HIP_TRY(hipSetDevice(ctx->device));
  if (enable) {
    HIP_TRY(hipDeviceSynchronize());  // pooled events may still be pending
    ctx->records.clear();
    ctx->pool_used = 0;
    for (auto& k : ctx->timing_seq) k = 0;
  }
  ctx->timing = enable;
  return MAGNUS_OK;
}

int magnus_timing_read(magnus_ctx* ctx, int32_t kind, double* total_ms, int64_t* launches) {
  if (!ctx || !total_ms || !launches) return fail(MAGNUS_EINVAL, "null argument");
  if (kind < MAGNUS_KERNEL_CSR_LEJA || kind > MAGNUS_KERNEL_CSR_LEJA3) return fail(MAGNUS_EINVAL, "kernel class %d", kind);
  HIP_TRY(hipSetDevice(ctx->device));
  double t = 0.0;
  int64_t n = 0;
  for (auto& r : ctx->records) {
    if (std::get<0>(r) != kind) continue;
    HIP_TRY(hipEventSynchronize(std::get<2>(r)));
    float ms = 0.0f;
    HIP_TRY(hipEventElapsedTime(&ms, std::get<1>(r), std::get<2>(r)));
    t += ms;
    ++n;
  }
  *total_ms = t;
  *launches = n;
  return MAGNUS_OK;
}

int magnus_propagate_ragged(magnus_ctx* ctx, const magnus_problem* probs, int32_t nprob, int32_t method,
                            double tau, int64_t nsteps, const magnus_leja_opts* opts, magnus_stats* stats,
                            magnus_stream stream) {
  if (!ctx) return fail(MAGNUS_EINVAL, "null context");
  if (!probs || nprob < 1) return fail(MAGNUS_EINVAL, "no problems");
  magnus::Scheme S;
  if (!magnus::method_scheme(method, &S)) return fail(MAGNUS_EINVAL, "unknown method %d", method);
  int rc = check_opts(opts);
  if (rc) return rc;
  if (nsteps < 0 || !is_fin(tau)) return fail(MAGNUS_EINVAL, "bad nsteps or tau");
  hipStream_t s = (hipStream_t)stream;
  if ((rc = begin_call(ctx, s))) return rc;
  for (int32_t i = 0; i < nprob; ++i) {
    const magnus_problem& P = probs[i];
    if ((rc = check_ham(ctx, &P.h, method == MAGNUS_M4))) return rc;
    if (!P.psi || P.batch < 1 || (P.batch_f != 1 && P.batch_f != P.batch) || (nsteps > 0 && !P.f_nodes))
      return fail(MAGNUS_EINVAL, "problem %d: bad state, batch or field", i);
    for (int64_t k = 0; k < S.q * nsteps * (int64_t)P.batch_f; ++k)
      if (!is_fin(P.f_nodes[k])) return fail(MAGNUS_EDOMAIN, "problem %d: non-finite field value", i);
    if ((rc = ensure_valid(ctx, &P.h, s))) return rc;
  }
  const double tol_e = per_exp_tol(opts, S.nexp * nsteps);
  Acc acc;
  // small problems (product-of-exponentials methods): every state in one persistent launch
  std::vector<const magnus_hamiltonian*> hs;
  std::vector<SmallState> sst;
  std::vector<int> big;
  // every CSR problem of at most kSmallDim rows joins the persistent launches:
  // the alternative here is a batched propagation per problem with a host
  // wait after it, which costs more than the single-call crossover assumes
  for (int32_t i = 0; i < nprob; ++i) {
    const magnus_problem& P = probs[i];
    if (!S.commutator && small_ok(ctx, &P.h, std::max<int64_t>(32, P.batch))) {
      const int pi = (int)hs.size();
      hs.push_back(&P.h);
      double2* psi = reinterpret_cast<double2*>(P.psi);
      for (int32_t c = 0; c < P.batch; ++c)
        sst.push_back(
            SmallState{pi, psi + c * P.h.H1.dim, P.f_nodes + (P.batch_f == 1 ? 0 : (int64_t)c) * nsteps * S.q});
    } else {
      big.push_back(i);
    }
  }
  // the large problems together when they have the same batch and fit the
  // workspace at once: each split into groups of JB states (the group size
  // tuned for the largest of them, else the largest that divides the batch),
  // one launch per Leja iteration for all groups, their control slots after
  // the small states' (no reset, no host wait between problems)
  bool joint = ctx->ragged_joint && !S.commutator && big.size() >= 2;
  int JB = 0;
  if (joint) {
    const int batch = probs[big[0]].batch;
    int largest = big[0];
    for (int i : big)
      if (probs[i].h.H1.dim > probs[largest].h.H1.dim) largest = i;
    JB = group_for(ctx, &probs[largest].h, batch);
    while (JB > 1 && batch % JB != 0) JB /= 2;
    size_t vtot = 0, ptot = 0, groups = 0;
    for (int i : big) {
      const magnus_problem& P = probs[i];
      joint = joint && P.h.H1.format == MAGNUS_CSR && P.batch == batch;
      vtot += (size_t)P.h.H1.dim * batch;
      if (JB >= 2) ptot += (size_t)magnus::ragged_grid((int)P.h.H1.dim, JB) * JB * 2 * (batch / JB);
      groups += JB >= 2 ? (size_t)(batch / JB) : 0;
    }
    joint = joint && JB >= 2 && JB <= ctx->max_batch && groups <= (size_t)magnus::kMaxRagged &&
            vtot <= (size_t)ctx->max_dim * (size_t)ctx->max_batch && ptot <= ctx->npartials &&
            sst.size() + groups * (size_t)JB <= (size_t)ctx->nslots;
  }
  // on coded terms the problems run as pairs of states
  std::vector<RagProblem> coded;
  bool report = false;
  if (ctx->ragged_joint && !S.commutator && !big.empty() && nsteps > 0 && tau != 0.0)
    if ((rc = code_ragged(ctx, probs, big, S, nsteps, (int)sst.size(), &coded, s))) return rc;
  if (!coded.empty()) {
    if ((rc = ragged_joint_steps(ctx, coded, S, tau, nsteps, tol_e, opts, &acc, s))) return rc;
    // batched propagations otherwise, each with a host wait that reports a
    // non-finite norm; here the small states are planned and launched before it
    if (!joint && (rc = copy_slots(ctx, s))) return rc;
    report = !joint;
    big.clear();
  } else if (joint && nsteps > 0) {
    std::vector<RagProblem> R;
    size_t voff = 0, poff = 0;
    int slot0 = (int)sst.size();
    for (int i : big) {
      const magnus_problem& P = probs[i];
      for (int c0 = 0; c0 < P.batch; c0 += JB) {
        R.push_back(RagProblem{&P, {}, c0, JB, voff, slot0, poff});
        voff += (size_t)P.h.H1.dim * JB;
        poff += (size_t)magnus::ragged_grid((int)P.h.H1.dim, JB) * JB * 2;
        slot0 += JB;
      }
    }
    if ((rc = ragged_joint_steps(ctx, R, S, tau, nsteps, tol_e, opts, &acc, s))) return rc;
    big.clear();
  }
  // the large problems first: each is one batched propagation (which resets the control slots)
  for (int i : big) {
    const magnus_problem& P = probs[i];
    if (P.batch > ctx->max_batch) return fail(MAGNUS_ENOMEM, "problem %d: batch %d exceeds max_batch", i, P.batch);
    magnus_leja_opts o = *opts;
    o.tol = tol_e;
    o.tol_mode = 0;
    magnus_stats ps{};
    // with stats, so a non-finite norm in this problem surfaces here (the slots are reset afterwards)
    rc = propagate(ctx, &P.h, method, tau, nsteps, P.f_nodes, P.batch_f, P.psi, P.batch, nullptr, 1, &o, &ps,
                   stream);
    if (rc) return rc;
    acc.exponentials += ps.exponentials;
    acc.substeps += ps.substeps;
    acc.planned += ps.planned_iters;
    acc.max_m = std::max(acc.max_m, ps.max_degree_used);
    acc.max_s = std::max(acc.max_s, ps.max_substeps_used);
    acc.max_bound = std::max(acc.max_bound, ps.max_err_bound);
    acc.extra_iters += ps.iters;  // counted by the nested call
  }
  if (!sst.empty() && nsteps > 0) {
    if (!big.empty()) HIP_TRY(magnus::launch_slot_reset(ctx->slots, ctx->nslots, s));
    // one launch per group of at most nslots states (one control slot each); the
    // slots keep counting, so groups after the first are folded into extra_iters
    for (size_t g0 = 0; g0 < sst.size(); g0 += (size_t)ctx->nslots) {
      const size_t g1 = std::min(sst.size(), g0 + (size_t)ctx->nslots);
      if (g0 > 0) {
        long long it = 0;
        int st = 0;
        if ((rc = read_slots(ctx, s, &it, &st))) return rc;  // the previous group's counters and status
        acc.extra_iters += it;
        ctx->sticky_status |= st;
        HIP_TRY(magnus::launch_slot_reset(ctx->slots, ctx->nslots, s));
      }
      std::vector<SmallState> part(sst.begin() + (long)g0, sst.begin() + (long)g1);
      if ((rc = persist_steps(ctx, hs, part, S, tau, 0, nsteps, tol_e, opts, &acc, s))) return rc;
    }
  }
  if (report && (rc = await_slots(ctx))) return rc;
  return end_call(ctx, acc, tol_e, stats, s);
}

int64_t magnus_adjoint_workspace_bytes(int64_t dim, int64_t nsteps, int32_t every_k) {
  if (dim < 1 || nsteps < 1 || every_k < 1) return -1;
  const int64_t k = std::min<int64_t>(every_k, nsteps);
  const int64_t nck = (nsteps + k - 1) / k + 1;
  const int64_t vecs = nck + (k + 1) + k + 2 + 4;
  return (vecs * dim + 2 * nsteps + 1) * (int64_t)sizeof(double2);
}

int magnus_propagate_adjoint(magnus_ctx* ctx, const magnus_hamiltonian* h, double tau, int64_t nsteps,
                             const double* f_nodes, const double* df_nodes, int32_t nparams, const void* psi0,
                             const void* psi_target, int32_t every_k, void* workspace, int64_t workspace_bytes,
                             double* loss, double* grad, const magnus_leja_opts* opts, magnus_stats* stats,
                             magnus_stream stream) {
  int rc = check_ham(ctx, h, 0);
  if (rc) return rc;
  if ((rc = check_opts(opts))) return rc;
  if (ctx->max_batch < 2) return fail(MAGNUS_ENOMEM, "the adjoint needs a context with max_batch >= 2");
  if (nsteps < 1 || nparams < 0 || every_k < 1) return fail(MAGNUS_EINVAL, "nsteps, nparams or every_k out of range");
  if (!f_nodes || (nparams > 0 && !df_nodes) || !psi0 || !psi_target || !workspace || !loss || (nparams > 0 && !grad))
    return fail(MAGNUS_EINVAL, "null argument");
  if (!is_fin(tau)) return fail(MAGNUS_EDOMAIN, "non-finite step");
  for (int64_t i = 0; i < 2 * nsteps; ++i)
    if (!is_fin(f_nodes[i])) return fail(MAGNUS_EDOMAIN, "non-finite field value");
  for (int64_t i = 0; i < 2 * nsteps * (int64_t)nparams; ++i)
    if (!is_fin(df_nodes[i])) return fail(MAGNUS_EDOMAIN, "non-finite field derivative");
  const int64_t need = magnus_adjoint_workspace_bytes(h->H1.dim, nsteps, every_k);
  if (workspace_bytes < need)
    return fail(MAGNUS_ENOMEM, "workspace of %lld bytes, need %lld", (long long)workspace_bytes, (long long)need);
  hipStream_t s = (hipStream_t)stream;
  if ((rc = begin_call(ctx, s))) return rc;
  if ((rc = ensure_valid(ctx, h, s))) return rc;

  if (tau != 0.0)
    if ((rc = begin_coded(ctx, h, false, 6 * nsteps, 0, s, CodeUse::kGradient))) return rc;
  if (ctx->coded_h == h && (!ctx->fuse || !pair_partials_fit(ctx, 2LL * magnus::code_grid((int)h->H1.dim, ctx->coded.rows))))
    ctx->coded_h = nullptr;
  const int64_t dim = h->H1.dim;
  const int64_t k = std::min<int64_t>(every_k, nsteps);
  const int64_t nck = (nsteps + k - 1) / k + 1;
  const int64_t nseg = (nsteps + k - 1) / k;
  double2* base = reinterpret_cast<double2*>(workspace);
  double2* ck = base;                       // nck states
  double2* seg_psi = ck + nck * dim;        // k + 1 states
  double2* seg_phi = seg_psi + (k + 1) * dim;  // k states
  double2* lam = seg_phi + k * dim;
  double2* mu = lam + dim;
  double2* X2 = mu + dim;                   // interleaved pair
  double2* Y2 = X2 + 2 * dim;
  double2* g = Y2 + 2 * dim;                // 2 nsteps + 1 complex
  const double tol_e = per_exp_tol(opts, 2 * nsteps);
  Acc acc;
  auto beta_of = [&](int64_t n) { return magnus::kAlpha2 * f_nodes[2 * n] + magnus::kAlpha1 * f_nodes[2 * n + 1]; };
  auto gamma_of = [&](int64_t n) { return magnus::kAlpha1 * f_nodes[2 * n] + magnus::kAlpha2 * f_nodes[2 * n + 1]; };
  const double2* tgt = reinterpret_cast<const double2*>(psi_target);

  // psi_{n+1} = E_b E_a psi_n through the half-step state phi_n
  auto step_to = [&](int64_t n, const double2* p0, double2* ph, double2* p1) {
    const int rc1 = run_exponential(ctx, ExpOp{h, 0.5, beta_of(n), 0.0}, tau, p0, ph, tol_e, opts, &acc, s);
    return rc1 ? rc1 : run_exponential(ctx, ExpOp{h, 0.5, gamma_of(n), 0.0}, tau, ph, p1, tol_e, opts, &acc, s);
  };
  // forward sweep with checkpoints (state kept in mu); the last segment's states
  // go where the backward sweep, which starts with it, looks for them
  const int64_t tail = (nseg - 1) * k;
  HIP_TRY(hipMemcpyAsync(ck, psi0, sizeof(double2) * dim, hipMemcpyDeviceToDevice, s));
  HIP_TRY(hipMemcpyAsync(nseg > 1 ? mu : seg_psi, psi0, sizeof(double2) * dim, hipMemcpyDeviceToDevice, s));
  for (int64_t n = 0; n < nsteps; ++n) {
    if (n >= tail) {
      double2* p0 = seg_psi + (n - tail) * dim;
      if ((rc = step_to(n, p0, seg_phi + (n - tail) * dim, p0 + dim))) return rc;
      continue;
    }
    if ((rc = step_to(n, mu, ctx->vec(kS2), mu))) return rc;
    if ((n + 1) % k == 0) {
      HIP_TRY(hipMemcpyAsync(ck + (n + 1) / k * dim, mu, sizeof(double2) * dim, hipMemcpyDeviceToDevice, s));
      if (n + 1 == tail) HIP_TRY(hipMemcpyAsync(seg_psi, mu, sizeof(double2) * dim, hipMemcpyDeviceToDevice, s));
    }
  }
  HIP_TRY(magnus::launch_cdot(tgt, 1, seg_psi + (nsteps - tail) * dim, 1, dim, ctx->dots, g + 2 * nsteps, s));
  HIP_TRY(hipMemcpyAsync(lam, tgt, sizeof(double2) * dim, hipMemcpyDeviceToDevice, s));

  // The block (Frechet) exponentials of a step, of phi_n with gamma_n and of
  // psi_n with beta_n, do not depend on lambda: on coded terms they run together,
  // as two pairs (each work buffer two vectors of the context, back to back).
  bool pairs = ctx->coded_h == h;
  const double half[4] = {0.5, 0.5, 0.5, 0.5};
  for (int64_t seg = nseg - 1; seg >= 0; --seg) {
    const int64_t n0 = seg * k, n1 = std::min(n0 + k, nsteps);
    if (seg < nseg - 1) {  // recompute psi_n and the half-step states phi_n of the segment
      HIP_TRY(hipMemcpyAsync(seg_psi, ck + seg * dim, sizeof(double2) * dim, hipMemcpyDeviceToDevice, s));
      for (int64_t n = n0; n < n1; ++n) {
        double2* p0 = seg_psi + (n - n0) * dim;
        if ((rc = step_to(n, p0, seg_phi + (n - n0) * dim, p0 + dim))) return rc;
      }
    }
    // the segment's block exponentials, planned and uploaded together
    std::vector<ColParam> table;
    std::vector<MultiExp> ea(n1 - n0), eb(n1 - n0);
    auto plan_segment = [&](Acc* a) {
      table.clear();
      for (int64_t n = n0; n < n1; ++n) {
        const double ga = gamma_of(n), be = beta_of(n), both[4] = {ga, ga, be, be};
        int rc1 = plan_multi(h, half, both, pairs ? 4 : 2, tau, tol_e, opts, 1, &table, &ea[n - n0], a);
        if (!rc1 && !pairs) rc1 = plan_multi(h, half, both + 2, 2, tau, tol_e, opts, 1, &table, &eb[n - n0], a);
        if (rc1) return rc1;
      }
      return (int)MAGNUS_OK;
    };
    Acc planned = acc;
    if ((rc = plan_segment(&planned))) return rc;
    if (pairs && table.size() > kTableCap) {
      // two pairs share the larger degree: one after the other the segment may still fit
      pairs = false;
      planned = acc;
      if ((rc = plan_segment(&planned))) return rc;
    }
    acc = planned;
    if ((rc = upload_table(ctx, table, s))) return rc;
    for (int64_t n = n1 - 1; n >= n0; --n) {
      const double2 *psi = seg_psi + (n - n0) * dim, *phi = seg_phi + (n - n0) * dim;
      const double2 *la = Y2, *lb = Y2;  // L_a phi_n, L_b psi_n (every second element)
      if (pairs) {
        la = ctx->vec(kS2);
        lb = la + 2 * dim;
        MultiExp E = ea[n - n0];
        E.src = X2;
        E.dst = ctx->vec(kS2);
        const PairWork W{h, ctx->coded, 2, ctx->vec(kA), ctx->vec(kS0), ctx->vec(kV), X2, 0, 0};
        HIP_TRY(magnus::launch_frechet_pairs_init(phi, psi, X2, (int)dim, s));
        if ((rc = launch_pairs_exp(ctx, {W}, {E}, tol_e, opts->early_termination, true, s))) return rc;
      } else {
        MultiExp A = ea[n - n0];
        A.src = X2;
        A.dst = Y2;
        HIP_TRY(magnus::launch_frechet_init(phi, X2, (int)dim, s));
        if ((rc = launch_multi(ctx, h, A, tol_e, opts->early_termination, s))) return rc;
      }
      // g_a(n) = lambda_{n+1}^H L_a phi_n
      HIP_TRY(magnus::launch_cdot(lam, 1, la, 2, dim, ctx->dots, g + 2 * n, s));
      // mu_n = E_a^H lambda_{n+1}
      rc = run_exponential(ctx, ExpOp{h, 0.5, gamma_of(n), 0.0}, -tau, lam, mu, tol_e, opts, &acc, s);
      if (rc) return rc;
      if (!pairs) {
        MultiExp Bx = eb[n - n0];
        Bx.src = X2;
        Bx.dst = Y2;
        HIP_TRY(magnus::launch_frechet_init(psi, X2, (int)dim, s));
        if ((rc = launch_multi(ctx, h, Bx, tol_e, opts->early_termination, s))) return rc;
      }
      // g_b(n) = mu_n^H L_b psi_n
      HIP_TRY(magnus::launch_cdot(mu, 1, lb, 2, dim, ctx->dots, g + 2 * n + 1, s));
      // lambda_n = E_b^H mu_n
      rc = run_exponential(ctx, ExpOp{h, 0.5, beta_of(n), 0.0}, -tau, mu, lam, tol_e, opts, &acc, s);
      if (rc) return rc;
    }
  }
  std::vector<double2> hg(2 * nsteps + 1);
  HIP_TRY(hipMemcpyAsync(hg.data(), g, sizeof(double2) * hg.size(), hipMemcpyDeviceToHost, s));
  HIP_TRY(hipStreamSynchronize(s));
  for (const double2& v : hg)
    if (!is_fin(v.x) || !is_fin(v.y)) ctx->sticky_status |= 1;
  const std::complex<double> z(hg[2 * nsteps].x, hg[2 * nsteps].y);
  *loss = 1.0 - std::norm(z);
  for (int32_t p = 0; p < nparams; ++p) {
    std::complex<double> dz = 0.0;
    for (int64_t n = 0; n < nsteps; ++n) {
      const double d1 = df_nodes[(2 * n) * nparams + p], d2v = df_nodes[(2 * n + 1) * nparams + p];
      const double dbeta = magnus::kAlpha2 * d1 + magnus::kAlpha1 * d2v;
      const double dgamma = magnus::kAlpha1 * d1 + magnus::kAlpha2 * d2v;
      dz += dgamma * std::complex<double>(hg[2 * n].x, hg[2 * n].y) +
            dbeta * std::complex<double>(hg[2 * n + 1].x, hg[2 * n + 1].y);
    }
    grad[p] = -2.0 * std::real(std::conj(z) * dz);
  }
  return end_call(ctx, acc, tol_e, stats, s);
}

int magnus_method_nodes(int32_t method) {
  magnus::Scheme S;
  if (!magnus::method_scheme(method, &S)) return fail(MAGNUS_EINVAL, "unknown method %d", method);
  return S.q;
}

int magnus_quadrature_nodes(int32_t method, double t0, double tau, int64_t nsteps, double* t_out) {
  magnus::Scheme S;
  if (!magnus::method_scheme(method, &S)) return fail(MAGNUS_EINVAL, "unknown method %d", method);
  if (nsteps < 0 || (nsteps > 0 && !t_out)) return fail(MAGNUS_EINVAL, "bad output");
  for (int64_t n = 0; n < nsteps; ++n) {
    const double tn = t0 + (double)n * tau;
    for (int j = 0; j < S.q; ++j) t_out[S.q * n + j] = tn + S.c[j] * tau;
  }
  return MAGNUS_OK;
}

int magnus_leja_points(int32_t m, double* xi) {
  if (m < 0 || m >= magnus::kNumPoints || !xi) return fail(MAGNUS_EINVAL, "m %d outside 0..%d", m, magnus::kNumPoints - 1);
  const auto& p = magnus::leja_points();
  for (int k = 0; k <= m; ++k) xi[k] = p[k];
  return MAGNUS_OK;
}

int magnus_divided_differences(double theta, int32_t m, double* d) {
  if (m < 0 || m >= magnus::kNumPoints || !d) return fail(MAGNUS_EINVAL, "m %d outside 0..%d", m, magnus::kNumPoints - 1);
  if (!is_fin(theta) || std::fabs(theta) > magnus::kThetaCap)
    return fail(MAGNUS_EDOMAIN, "|theta| %g above %g", theta, magnus::kThetaCap);
  std::vector<std::complex<double>> v(m + 1);
  magnus::divided_differences(theta, m, v.data());
  for (int k = 0; k <= m; ++k) { d[2 * k] = v[k].real(); d[2 * k + 1] = v[k].imag(); }
  return MAGNUS_OK;
}

double magnus_leja_error(double theta, int32_t m) {
  if (!is_fin(theta) || std::fabs(theta) > magnus::kThetaCap) return INFINITY;
  return magnus::leja_error(theta, m);
}

int magnus_leja_plan(double theta, double tol, int32_t max_degree, int32_t max_substeps, int32_t* m, int32_t* s,
                     double* bound) {
  if (!m || !s || !bound) return fail(MAGNUS_EINVAL, "null output");
  if (!(tol > 0.0) || !is_fin(theta)) return fail(MAGNUS_EDOMAIN, "bad theta or tol");
  magnus::LejaPlan p;
  if (!magnus::plan_degree(theta, tol, max_degree, max_substeps, &p))
    return fail(MAGNUS_ENOCONV, "caps cannot reach tol %g at theta %g", tol, theta);
  *m = p.m;
  *s = p.s;
  *bound = p.bound;
  return MAGNUS_OK;
}

}  // extern "C"

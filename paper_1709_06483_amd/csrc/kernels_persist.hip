// Whole propagations inside one workgroup, for states of small dimension.
//
// At a few thousand rows a Leja iteration moves well under a megabyte, so
// the cost of separate kernel launches (and of a grid-wide reduction for
// the stop test) dominates.  Here one workgroup carries one state through
// every exponential of the call: each Leja iteration is its threads over the
// rows (two-term CSR product gathering from LDS, shift, Newton accumulation,
// norm partials), one workgroup barrier, a fixed-order sum of the partials that
// every thread does and the stop verdict, all without leaving the kernel.
// The states of a call (or several problems of a ragged batch) are separate
// workgroups of one launch.
//
// Up to 1,024 rows the matrix lies in registers, since reading it again in
// every iteration took most of the time.  Chains, us per iteration, the matrix
// re-read (term 1 from LDS) / in registers: n = 6 2.1 / 0.9, n = 8 2.9 / 1.1,
// n = 9 3.3 / 1.5, n = 10 5.2 / 2.4.  What bounds it then is the number of
// instructions a SIMD issues in turn (n = 10: 363 vector, 79 scalar and 50 LDS
// instructions per wave and iteration, counted, of two waves) and below n = 9 the
// latency of their chain.  Two rows to each of 512 threads: the part of an
// iteration that every wave repeats (the sums, two square roots, the verdict) is
// then done by 8 waves; 1,024 threads with a row each took 3.2 us at n = 10.
#include "device_common.h"

#include <cstddef>

namespace magnus {
namespace {

using namespace dev;

constexpr int kPT = 1024;  // threads per workgroup
static_assert(kPT == kPersistStepDim, "rows in registers");

// What the host wrote before the launch and the whole workgroup reads alike, by scalar loads.
template <class T>
using Scalar = const __attribute__((address_space(4))) T;
template <class T>
__device__ __forceinline__ Scalar<T>* scalar(const T* p) {
  return (Scalar<T>*)(unsigned long long)p;
}
__device__ __forceinline__ PersistProblem persist_problem(const PersistArgs& a, int b) {
  Scalar<PersistProblem>* p = scalar(a.probs) + scalar(a.state_prob)[b];
  return PersistProblem{CsrDev{p->t1.rp, p->t1.ci, p->t1.val}, CsrDev{p->t2.rp, p->t2.ci, p->t2.val}, p->dim};
}

// sum_k val[k] X[col[k]] over one row, the vector X resident in LDS.
__device__ __forceinline__ d2 row_product(int k0, int k1, const int* __restrict__ col, const d2* __restrict__ val,
                                          const d2* X) {
  d2 s = {0.0, 0.0};
#pragma unroll 4
  for (int k = k0; k < k1; ++k) s += cmul(val[k], X[col[k]]);
  return s;
}

// Threads of a workgroup for dimensions up to 1,024, each with one or two rows.
constexpr int kRowThreads = 512;

// The parameters of one exponential's iterations, as a wave holds them: lane
// 6 k + f field f of iteration 10 c + k + 1 of chunk c.  Vector loads, issued
// an exponential ahead for its first two chunks: scalar loads share their
// counter with LDS, so the next LDS access would wait for them.
constexpr int kParamFields = 6, kParamChunk = 10;
struct IterParam {
  double a1, a2, sigma, dre, dim, dabs;
};
static_assert(sizeof(IterParam) == 8 * kParamFields && offsetof(ColParam, dabs) == 8 * (kParamFields - 1),
              "the first fields of ColParam");
__device__ __forceinline__ double lane_value(double v, int lane) {
  union U {
    double d;
    int u[2];
  } a{v};
  for (int k = 0; k < 2; ++k) a.u[k] = __builtin_amdgcn_readlane(a.u[k], lane);
  return a.d;
}
// Lanes 60 .. 62 hold d_0 and |d_0|.  (Records past the exponential's last are
// not used: the last is read instead.)
constexpr int kParamD0 = kParamFields * kParamChunk;
static_assert(offsetof(ColParam, d0re) == 8 * kParamFields && offsetof(ColParam, d0abs) == 8 * (kParamFields + 2),
              "then d_0 and |d_0|");
__device__ __forceinline__ double param_chunk(const ColParam* table, int m, int c) {
  const int lane = threadIdx.x & 63, k = min(kParamChunk * c + lane / kParamFields, m - 1);
  const double* p = lane < kParamD0 ? reinterpret_cast<const double*>(table + k) + lane % kParamFields
                                    : reinterpret_cast<const double*>(table) + min(kParamFields + lane - kParamD0, 8);
  return *p;
}
__device__ __forceinline__ IterParam iter_param(double chunk, int k) {
  const int l = kParamFields * k;
  return IterParam{lane_value(chunk, l),     lane_value(chunk, l + 1), lane_value(chunk, l + 2),
                   lane_value(chunk, l + 3), lane_value(chunk, l + 4), lane_value(chunk, l + 5)};
}

// An exponential's header, likewise: lanes 0 .. 2.
struct ExpHead {
  int m, s;
  const ColParam* table;
  double tol_sub;
};
__device__ __forceinline__ double head_words(const PersistExp* e) {
  return reinterpret_cast<const double*>(e)[min((int)(threadIdx.x & 63), 2)];
}
__device__ __forceinline__ ExpHead exp_head(const ColParam* table, double words) {
  union U {
    double d;
    long long l;
    int i[2];
  } ms, off;
  ms.d = lane_value(words, 0);
  off.d = lane_value(words, 1);
  return ExpHead{ms.i[0], ms.i[1], table + off.l, lane_value(words, 2)};
}
static_assert(sizeof(PersistExp) == 24 && offsetof(PersistExp, table_off) == 8 && offsetof(PersistExp, tol_sub) == 16,
              "three words");

// A value that every lane holds, in scalar registers.
__device__ __forceinline__ double uniform(double v) { return lane_value(v, 0); }

// The exponentials of one state.
struct PersistSchedule {
  const PersistExp* exps;
  const ColParam* table;
  int nexp, early;
};

struct PersistControl {
  long long iters = 0;
  int status = 0, stopped = 0, iters_sub = 0;
  double vnorm = 0.0, prev = 0.0, est = 0.0;
};

// The exponentials of one state, thread t owning rows t + k blockDim, k < R.
// products(X, w, a1, a2, y) gives its rows of (a1 H1 + a2 H2) X, w its own
// elements; the Newton accumulator and the rows' w_i stay in registers, the
// basis vectors in two LDS buffers (iteration i gathers from one and writes the
// other).  Returns with the state in `cur` and the control state of the stop
// test, the same in every thread, in `c`.
template <int R, class F>
__device__ __forceinline__ void persist_rows(const PersistSchedule& a, int dim, d2* X, d2* Y, double (*red)[2][16],
                                             d2 (&cur)[R], PersistControl& c, F products) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int nt = R == 1 ? 0 : kRowThreads;
  const PersistExp* exps = a.exps;
  int rpar = 0;
  double words = head_words(exps);
  ExpHead next = exp_head(a.table, words);
  double next0 = param_chunk(next.table, next.m, 0), next1 = param_chunk(next.table, next.m, 1);
  words = head_words(exps + min(1, a.nexp - 1));
  for (int e = 0; e < a.nexp; ++e) {
    const ExpHead E = next;
    const double chunk0 = next0, chunk1 = next1;
    const double d0re = lane_value(chunk0, kParamD0), d0im = lane_value(chunk0, kParamD0 + 1),
                 d0abs = lane_value(chunk0, kParamD0 + 2);
    next = exp_head(a.table, words);  // (past the last: the last again)
    next0 = param_chunk(next.table, next.m, 0);
    next1 = param_chunk(next.table, next.m, 1);
    words = head_words(exps + min(e + 2, a.nexp - 1));
    for (int sub = 0; sub < E.s; ++sub) {
      d2 w[R], P[R];
#pragma unroll
      for (int k = 0; k < R; ++k) {
        w[k] = cur[k];
        P[k] = d2{0.0, 0.0};
        if (tid + k * nt < dim) X[tid + k * nt] = cur[k];
      }
      __syncthreads();
      double chunk = chunk0;
      int at = 0;  // of iteration i in its chunk
      for (int i = 1; i <= E.m; ++i) {
        if (at == kParamChunk) {
          if (i == kParamChunk + 1) {
            chunk = chunk1;
          } else {
            chunk = param_chunk(E.table, E.m, (i - 1) / kParamChunk);
            __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0), here and not in every iteration
          }
          at = 0;
        }
        const IterParam prm = iter_param(chunk, at++);
        const bool first = (i == 1);
        const d2 dd = {prm.dre, prm.dim};
        double pw = 0.0, pv = 0.0;
        d2 y[R];
        products(X, w, prm.a1, prm.a2, y);
#pragma unroll
        for (int k = 0; k < R; ++k)
          if (tid + k * nt < dim) {
            const d2 wn = y[k] - rmul(prm.sigma, w[k]);
            if (first) {
              P[k] = cmul(d2{d0re, d0im}, w[k]) + cmul(dd, wn);
              pv += nrm2(w[k]);
            } else {
              P[k] += cmul(dd, wn);
            }
            Y[tid + k * nt] = wn;
            w[k] = wn;
            pw += nrm2(wn);
          }
        pw = lanes_sum(pw);
        if (first) pv = lanes_sum(pv);
        if (lane == 0) {
          red[rpar][0][wv] = pw;
          red[rpar][1][wv] = pv;
        }
        __syncthreads();  // publishes w_i and the partial sums
        // (the entries of waves past the workgroup's stay zero)
        const double tw = row16_sum(red[rpar][0][lane & 15]);
        const double tv = first ? row16_sum(red[rpar][1][lane & 15]) : 0.0;
        rpar ^= 1;
        d2* t = X;
        X = Y;
        Y = t;
        // the early-termination test (same rule as the grid path's decide kernel)
        const double wnrm = sqrt(tw);
        const double vn = first ? sqrt(tv) : c.vnorm;
        const double pt = first ? d0abs * vn : c.prev;
        const double term = prm.dabs * wnrm;
        const int bad = __builtin_amdgcn_readfirstlane(!isfinite(tw) || !isfinite(vn) ? 1 : 0);
        c.est = uniform(term + pt);
        c.status |= bad;
        c.vnorm = uniform(vn);
        c.prev = uniform(term);
        c.iters_sub = first ? 1 : c.iters_sub + 1;
        c.stopped = __builtin_amdgcn_readfirstlane(bad || (a.early && c.est <= E.tol_sub * vn) ? 1 : 0);
        ++c.iters;
        if (c.stopped && i < E.m) break;  // uniform: the remaining terms are below tolerance
      }
#pragma unroll
      for (int k = 0; k < R; ++k) cur[k] = P[k];
    }
  }
}

// A row's entries of both terms in registers, in groups of four of one term
// (first those of term 1): the values, all real or all imaginary in a term, and
// the columns as byte offsets into an LDS vector, two to a register; the
// vector's element kPT is zero and stands for no entry.  The diagonal, real,
// is kept apart.
constexpr int kRegGroups = 6;
struct RowRegs {
  double val[4 * kRegGroups];
  unsigned at[2 * kRegGroups];
  double diag[2];
  int parts[2];   // which parts the term's values have: bit 0 real, bit 1 imaginary
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t entry_buffer(const void* p, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
}

// The first g1 groups of term 1 and g2 of term 2 (uniform).  Loads past the
// row's end are out of the buffer: zeros, without an access.
__device__ __forceinline__ void load_regs(RowRegs& R, const PersistProblem& pb, int row, const int (&start)[2],
                                          const int (&len)[2], int g1, int g2) {
  constexpr int kPast = 1 << 26;
  typedef unsigned u4 __attribute__((ext_vector_type(4)));
  const int nnz[2] = {*scalar(pb.t1.rp + pb.dim), *scalar(pb.t2.rp + pb.dim)};
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    R.diag[t] = 0.0;
    R.parts[t] = 0;
  }
#pragma unroll
  for (int g = 0; g < kRegGroups; ++g) {
    const bool second = g >= g1;  // uniform
    const CsrDev& T = second ? pb.t2 : pb.t1;
    const int k0 = 4 * (second ? g - g1 : g), n = second ? len[1] : len[0], s = second ? start[1] : start[0];
    const int entries = g < g1 + g2 ? (second ? nnz[1] : nnz[0]) : 0;
    const __amdgpu_buffer_rsrc_t col_buf = entry_buffer(T.ci, entries * 4), val_buf = entry_buffer(T.val, entries * 16);
    int col[4];
    u4 v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int e = k0 + j < n ? s + k0 + j : kPast;
      col[j] = __builtin_amdgcn_raw_buffer_load_b32(col_buf, e * 4, 0, 0);
      v[j] = __builtin_amdgcn_raw_buffer_load_b128(val_buf, e * 16, 0, 0);
    }
    unsigned at[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const bool has = k0 + j < n && g < g1 + g2;
      d2 h = __builtin_bit_cast(d2, v[j]);
      const bool on_diag = has && col[j] == row;
      R.diag[0] += on_diag && !second ? h.x : 0.0;
      R.diag[1] += on_diag && second ? h.x : 0.0;
      const int parts = on_diag ? (h.y != 0.0 ? 3 : 0) : (h.x != 0.0 ? 1 : 0) | (h.y != 0.0 ? 2 : 0);
      h = on_diag ? d2{0.0, 0.0} : h;
      R.parts[0] |= second ? 0 : parts;
      R.parts[1] |= second ? parts : 0;
      R.val[4 * g + j] = h.x != 0.0 ? h.x : h.y;
      at[j] = 16u * (unsigned)(has && !on_diag ? col[j] : kPT);
      asm volatile("" : "+v"(R.val[4 * g + j]));  // formed here: else the loaded pairs are kept, and spill
    }
    R.at[2 * g] = at[0] | at[1] << 16;
    R.at[2 * g + 1] = at[2] | at[3] << 16;
    asm volatile("" : "+v"(R.at[2 * g]), "+v"(R.at[2 * g + 1]), "+v"(R.diag[0]), "+v"(R.diag[1]), "+v"(R.parts[0]),
                 "+v"(R.parts[1]));
  }
}

// The thread's rows of (a1 H1 + a2 H2) X off the diagonal; a group's gathers of
// all rows go out together (with one row those of the next group before its
// products).
template <int R>
__device__ __forceinline__ void reg_products(const RowRegs (&regs)[R], int g1, int g2, const d2* X, double a1, double a2,
                                             d2 (&y)[R]) {
  const char* x = reinterpret_cast<const char*>(X);
  d2 s[R];
  auto add_term = [&](int t) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      y[r] += rmul(t == 0 ? a1 : a2, regs[r].parts[t] == 2 ? d2{-s[r].y, s[r].x} : s[r]);
      s[r] = d2{0.0, 0.0};
    }
  };
  constexpr int kDeep = R == 1 ? 2 : 1;  // groups in flight (two rows' values leave registers for one)
  d2 v[kDeep][R][4];
  auto load = [&](int g) {
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int j = 0; j < 4; j += 2) {
        unsigned at = regs[r].at[2 * g + j / 2];
        asm volatile("" : "+v"(at));  // unpacked here: kept unpacked the offsets would spill
        v[g % kDeep][r][j] = *reinterpret_cast<const d2*>(x + (at & 0xffffu));
        v[g % kDeep][r][j + 1] = *reinterpret_cast<const d2*>(x + (at >> 16));
      }
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int r = 0; r < R; ++r) y[r] = s[r] = d2{0.0, 0.0};
  const int groups = g1 + g2;
  if (groups == 0) return;
  if (kDeep == 2) load(0);
#pragma unroll
  for (int g = 0; g < kRegGroups; ++g) {
    if (kDeep == 1) load(g);
    else if (g + 1 < kRegGroups && g + 1 < groups) load(g + 1 < kRegGroups ? g + 1 : g);
    if (g == g1) {  // the first group of term 2
      asm volatile("");  // (a branch, not selects in every group)
      add_term(0);
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int j = 0; j < 4; ++j) s[r] += rmul(regs[r].val[4 * g + j], v[g % kDeep][r][j]);
    __builtin_amdgcn_sched_barrier(0);
    if (g + 1 >= groups) break;
  }
  add_term(g2 > 0 ? 1 : 0);
}

// Groups of four entries of the wave's longest row.
__device__ __forceinline__ int wave_groups(int len) {
  int g = 0;
  while (__any(len > 4 * g)) ++g;
  return __builtin_amdgcn_readfirstlane(g);
}

__device__ __forceinline__ void persist_record(Slot* S, const PersistControl& c) {
  S->stopped = c.stopped;
  S->iters_sub = c.iters_sub;
  S->status |= c.status;
  S->iters_total += c.iters;
  S->vnorm = c.vnorm;
  S->prev_term = c.prev;
  S->last_est = c.est;
}

template <int R>
__device__ __forceinline__ void persist_finish(double2* state, Slot* S, int dim, const d2 (&cur)[R],
                                               const PersistControl& c) {
  const int tid = threadIdx.x;
#pragma unroll
  for (int k = 0; k < R; ++k)
    if (tid + k * kRowThreads < dim) reinterpret_cast<d2*>(state)[tid + k * kRowThreads] = cur[k];
  if (tid == 0) persist_record(S, c);
}

// Term 1 into LDS (the host checked that its entries fit; a barrier follows).
__device__ __forceinline__ void cache_term1(const PersistProblem& pb, d2* val, int* col) {
  const int n = min(pb.t1.rp[pb.dim], kPersistCache);
  for (int k = threadIdx.x; k < n; k += (int)blockDim.x) {
    val[k] = reinterpret_cast<const d2*>(pb.t1.val)[k];
    col[k] = pb.t1.ci[k];
  }
}

// Dimensions up to 1,024: R rows per thread.  Rows whose entries take at most
// kRegGroups groups of four (those of one wave's longest rows counted), the
// off-diagonal ones of a row and term all real or all imaginary, are read into
// registers once, so that an iteration touches only LDS, where it gathers w; if
// one row of the state does not fit, all are read from memory in every
// iteration, with CACHE term 1 from a copy in LDS (one workgroup per CU then;
// complex values, us per iteration with / without: 400 rows of 14 + 8 entries
// 3.5 / 4.4, 512 rows of 10 + 20 4.5 / 5.7 on the grid).
template <int R, bool CACHE>
__device__ __forceinline__ void persist_state(const PersistProblem& pb, const PersistSchedule& plan, const double2* in,
                                              double2* out, Slot* slot) {
  __shared__ d2 X[2][kPT + 1];
  __shared__ double red[2][2][16];
  __shared__ d2 cval[CACHE ? kPersistCache : 1];
  __shared__ int ccol[CACHE ? kPersistCache : 1];
  const int tid = threadIdx.x;
  const int dim = pb.dim;
  d2 cur[R];
  int start[R][2], len[R][2];
  int longest[2] = {0, 0};
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int row = tid + k * kRowThreads;
    cur[k] = d2{0.0, 0.0};
    start[k][0] = start[k][1] = len[k][0] = len[k][1] = 0;
    if (row < dim) {
      cur[k] = reinterpret_cast<const d2*>(in)[row];
      start[k][0] = pb.t1.rp[row];
      len[k][0] = pb.t1.rp[row + 1] - start[k][0];
      start[k][1] = pb.t2.rp[row];
      len[k][1] = pb.t2.rp[row + 1] - start[k][1];
    }
    for (int t = 0; t < 2; ++t) longest[t] = max(longest[t], min(len[k][t], 4 * kRegGroups + 4));
  }
  if (tid < 2) X[tid][kPT] = d2{0.0, 0.0};
  if (tid < 64) red[tid >> 5][tid >> 4 & 1][tid & 15] = 0.0;
  PersistControl c;
  const int g1 = wave_groups(longest[0]), g2 = wave_groups(longest[1]);
  bool fits = !__syncthreads_or(g1 + g2 > kRegGroups);
  RowRegs regs[R];
  if (fits) {
    int mixed = 0;
#pragma unroll
    for (int k = 0; k < R; ++k) {
      load_regs(regs[k], pb, tid + k * kRowThreads, start[k], len[k], g1, g2);
      mixed |= regs[k].parts[0] == 3 || regs[k].parts[1] == 3;
    }
    fits = !__syncthreads_or(mixed);
  }
  if (fits) {
    persist_rows<R>(plan, dim, X[0], X[1], red, cur, c, [&](const d2* x, const d2 (&w)[R], double a1, double a2, d2 (&y)[R]) {
      reg_products<R>(regs, g1, g2, x, a1, a2, y);
#pragma unroll
      for (int k = 0; k < R; ++k) y[k] += rmul(a1 * regs[k].diag[0] + a2 * regs[k].diag[1], w[k]);
    });
  } else {
    if constexpr (CACHE) cache_term1(pb, cval, ccol);
    persist_rows<R>(plan, dim, X[0], X[1], red, cur, c, [&](const d2* x, const d2 (&)[R], double a1, double a2, d2 (&y)[R]) {
#pragma unroll
      for (int k = 0; k < R; ++k) {
        const int s1 = start[k][0], s2 = start[k][1];
        d2 y1;
        if constexpr (CACHE) y1 = row_product(s1, s1 + len[k][0], ccol, cval, x);
        else y1 = row_product(s1, s1 + len[k][0], pb.t1.ci, reinterpret_cast<const d2*>(pb.t1.val), x);
        y[k] = rmul(a1, y1) + rmul(a2, row_product(s2, s2 + len[k][1], pb.t2.ci, reinterpret_cast<const d2*>(pb.t2.val), x));
      }
    });
  }
  persist_finish<R>(out, slot, dim, cur, c);
}

template <int R, bool CACHE>
__global__ __launch_bounds__(kRowThreads) void persist_rows_kernel(PersistArgs a) {
  const int b = blockIdx.x;
  const PersistProblem pb = persist_problem(a, b);
  const PersistSchedule plan{a.exps + (long long)b * a.nexp, a.table, a.nexp, a.early};
  persist_state<R, CACHE>(pb, plan, a.state[b], a.state[b], &a.slots[b]);
}

// Rows that are not expected to fit (513 to 1,024 of them): read from memory in
// every iteration by a thread each (773 rows of 38 entries 9.4 us per iteration,
// 11 with two rows to each of 512 threads), with
// CACHE term 1 from a copy in LDS, one workgroup per CU then (16 entries a row:
// 5.2 us, 6.5 without).
template <bool CACHE>
__global__ __launch_bounds__(kPT) void persist_csr_kernel(PersistArgs a) {
  __shared__ d2 X[2][kPT + 1];
  __shared__ double red[2][2][16];
  __shared__ d2 cval[CACHE ? kPersistCache : 1];
  __shared__ int ccol[CACHE ? kPersistCache : 1];
  const int b = blockIdx.x;
  const int tid = threadIdx.x;
  const PersistProblem pb = persist_problem(a, b);
  const PersistSchedule plan{a.exps + (long long)b * a.nexp, a.table, a.nexp, a.early};
  const int dim = pb.dim;
  const d2* v1 = reinterpret_cast<const d2*>(pb.t1.val);
  const d2* v2 = reinterpret_cast<const d2*>(pb.t2.val);
  d2 cur[1] = {d2{0.0, 0.0}};
  int s1 = 0, e1 = 0, s2 = 0, e2 = 0;
  if (tid < dim) {
    cur[0] = reinterpret_cast<const d2*>(a.state[b])[tid];
    s1 = pb.t1.rp[tid];
    e1 = pb.t1.rp[tid + 1];
    s2 = pb.t2.rp[tid];
    e2 = pb.t2.rp[tid + 1];
  }
  if (tid < 64) red[tid >> 5][tid >> 4 & 1][tid & 15] = 0.0;
  if constexpr (CACHE) cache_term1(pb, cval, ccol);
  __syncthreads();
  PersistControl c;
  persist_rows<1>(plan, dim, X[0], X[1], red, cur, c, [&](const d2* x, const d2 (&)[1], double a1, double a2, d2 (&y)[1]) {
    d2 y1;
    if constexpr (CACHE) y1 = row_product(s1, e1, ccol, cval, x);
    else y1 = row_product(s1, e1, pb.t1.ci, v1, x);
    y[0] = rmul(a1, y1) + rmul(a2, row_product(s2, e2, pb.t2.ci, v2, x));
  });
  if (tid < dim) reinterpret_cast<d2*>(a.state[b])[tid] = cur[0];
  if (tid == 0) persist_record(&a.slots[b], c);
}

// One step, the same for every state, its parameters in the launch's own
// arguments: no copy to the device before it.
template <int R>
__global__ __launch_bounds__(kRowThreads) void persist_step_kernel(PersistStep a) {
  __shared__ PersistInline plan;
  // (the argument block by its address: indexing the argument itself would copy it to scratch)
  const auto* args = reinterpret_cast<const PersistStep*>((unsigned long long)__builtin_amdgcn_kernarg_segment_ptr());
  const int words = sizeof(PersistInline) / 8;
  for (int k = threadIdx.x; k < words; k += (int)blockDim.x)
    reinterpret_cast<double*>(&plan)[k] = reinterpret_cast<const double*>(&args->plan)[k];
  __syncthreads();
  const PersistSchedule schedule{plan.exps, plan.table, a.nexp, a.early};
  const long long at = (long long)blockIdx.x * a.problem.dim;
  persist_state<R, false>(a.problem, schedule, a.in + at, a.out + at, &a.slots[blockIdx.x]);
}

// Larger dimensions, up to CAP: thread t owns rows t, t + kPT, ... (at most
// CAP / kPT of them); the Newton accumulator and the vector each substep starts
// from stay in its registers, the basis vectors in two LDS buffers, so the only
// global traffic of an iteration is the CSR data itself.
template <int CAP>
__global__ __launch_bounds__(kPT) void persist_propagate_kernel(PersistArgs a) {
  constexpr int R = CAP / kPT;
  __shared__ d2 X[2][CAP];
  __shared__ double red[2][2][kPT / 64];
  const int b = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const PersistProblem pb = persist_problem(a, b);
  const int dim = pb.dim;
  const d2* v1 = reinterpret_cast<const d2*>(pb.t1.val);
  const d2* v2 = reinterpret_cast<const d2*>(pb.t2.val);
  d2* state = reinterpret_cast<d2*>(a.state[b]);
  const PersistExp* exps = a.exps + (long long)b * a.nexp;

  d2 cur[R];
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int r = tid + k * kPT;
    cur[k] = r < dim ? state[r] : d2{0.0, 0.0};
  }
  // control state of the stop test, identical in every thread
  Slot* S = &a.slots[b];
  long long iters = 0;
  int status = 0, stopped = 0, iters_sub = 0;
  double vnorm = 0.0, prev = 0.0, est = 0.0;
  int par = 0, rpar = 0;

  for (int e = 0; e < a.nexp; ++e) {
    const PersistExp E = exps[e];
    for (int sub = 0; sub < E.s; ++sub) {
#pragma unroll
      for (int k = 0; k < R; ++k)
        if (tid + k * kPT < dim) X[par][tid + k * kPT] = cur[k];
      __syncthreads();
      d2 P[R];
#pragma unroll
      for (int k = 0; k < R; ++k) P[k] = d2{0.0, 0.0};
      for (int i = 1; i <= E.m; ++i) {
        const ColParam prm = a.table[E.table_off + (i - 1)];
        const bool first = (i == 1);
        const d2 dd = {prm.dre, prm.dim};
        double pw = 0.0, pv = 0.0;
#pragma unroll
        for (int k = 0; k < R; ++k) {
          const int r = tid + k * kPT;
          if (r >= dim) continue;
          // (row bounds re-read, from cache, in every iteration: the kernel stays free of spills)
          const d2 y1 = row_product(pb.t1.rp[r], pb.t1.rp[r + 1], pb.t1.ci, v1, X[par]);
          const d2 y2 = row_product(pb.t2.rp[r], pb.t2.rp[r + 1], pb.t2.ci, v2, X[par]);
          const d2 xr = X[par][r];
          const d2 wn = rmul(prm.a1, y1) + rmul(prm.a2, y2) - rmul(prm.sigma, xr);
          if (first) {
            P[k] = cmul(d2{prm.d0re, prm.d0im}, xr) + cmul(dd, wn);
            pv += nrm2(xr);
          } else {
            P[k] += cmul(dd, wn);
          }
          X[par ^ 1][r] = wn;
          pw += nrm2(wn);
        }
        pw = wave_sum(pw);
        pv = wave_sum(pv);
        if (lane == 0) { red[rpar][0][wv] = pw; red[rpar][1][wv] = pv; }
        __syncthreads();  // publishes w_i and the partial sums
        double tw = 0.0, tv = 0.0;
        for (int w = 0; w < kPT / 64; ++w) { tw += red[rpar][0][w]; tv += red[rpar][1][w]; }
        rpar ^= 1;
        par ^= 1;
        // the early-termination test (same rule as the grid path's decide kernel)
        const double wnrm = sqrt(tw);
        const double vn = first ? sqrt(tv) : vnorm;
        const double pt = first ? prm.d0abs * vn : prev;
        const double term = prm.dabs * wnrm;
        const bool bad = !isfinite(tw) || !isfinite(vn);
        est = term + pt;
        status |= bad ? 1 : 0;
        vnorm = vn;
        prev = term;
        iters_sub = first ? 1 : iters_sub + 1;
        stopped = (bad || (a.early && est <= E.tol_sub * vn)) ? 1 : 0;
        ++iters;
        if (stopped && i < E.m) break;  // uniform: the remaining terms are below tolerance
      }
#pragma unroll
      for (int k = 0; k < R; ++k) cur[k] = P[k];
    }
  }
#pragma unroll
  for (int k = 0; k < R; ++k)
    if (tid + k * kPT < dim) state[tid + k * kPT] = cur[k];
  if (tid == 0) {
    S->stopped = stopped;
    S->iters_sub = iters_sub;
    S->status |= status;
    S->iters_total += iters;
    S->vnorm = vnorm;
    S->prev_term = prev;
    S->last_est = est;
  }
}

}  // namespace

hipError_t launch_persist_propagate(const PersistArgs& a, int nstates, int max_dim, hipStream_t s) {
  const int threads = (max_dim + 63) / 64 * 64;
  if (max_dim <= 0) return hipSuccess;
  if (max_dim <= kRowThreads && a.cache1 && !a.in_regs) persist_rows_kernel<1, true><<<nstates, threads, 0, s>>>(a);
  else if (max_dim <= kRowThreads) persist_rows_kernel<1, false><<<nstates, threads, 0, s>>>(a);
  else if (max_dim <= kPT && a.in_regs) persist_rows_kernel<2, false><<<nstates, kRowThreads, 0, s>>>(a);
  else if (max_dim <= kPT && a.cache1) persist_csr_kernel<true><<<nstates, kPT, 0, s>>>(a);
  else if (max_dim <= kPT) persist_csr_kernel<false><<<nstates, kPT, 0, s>>>(a);
  else if (max_dim <= kPersistMaxDim) persist_propagate_kernel<kPersistMaxDim><<<nstates, kPT, 0, s>>>(a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_persist_step(const PersistStep& a, int nstates, hipStream_t s) {
  const int dim = a.problem.dim, threads = (dim + 63) / 64 * 64;
  if (dim <= 0 || nstates <= 0) return hipSuccess;
  if (dim <= kRowThreads) persist_step_kernel<1><<<nstates, threads, 0, s>>>(a);
  else if (dim <= kPersistStepDim) persist_step_kernel<2><<<nstates, kRowThreads, 0, s>>>(a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace magnus

// Device helpers shared by the HIP kernels of libmagnus (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.h"

namespace magnus {
namespace dev {

using d2 = double __attribute__((ext_vector_type(2)));

constexpr int kThreads = 256;

__device__ __forceinline__ d2 cmul(d2 a, d2 b) { return d2{a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x}; }
__device__ __forceinline__ d2 rmul(double s, d2 a) { return d2{s * a.x, s * a.y}; }
// Contractions spelled out, for results that two kernels form alike bit for bit.
__device__ __forceinline__ d2 fma_r(double s, d2 a, d2 c) {
  return d2{__builtin_fma(s, a.x, c.x), __builtin_fma(s, a.y, c.y)};
}
__device__ __forceinline__ d2 fma_c(d2 a, d2 b, d2 c) {
  return d2{__builtin_fma(-a.y, b.y, __builtin_fma(a.x, b.x, c.x)), __builtin_fma(a.y, b.x, __builtin_fma(a.x, b.y, c.y))};
}
__device__ __forceinline__ d2 tod2(double2 v) { return d2{v.x, v.y}; }
__device__ __forceinline__ double2 fromd2(d2 v) { return make_double2(v.x, v.y); }
__device__ __forceinline__ double nrm2(d2 v) { return v.x * v.x + v.y * v.y; }

// Workgroups are dispatched round-robin over the 8 XCDs; give each XCD a
// contiguous range of row blocks so rows that share gathered vector entries
// share that XCD's L2.
__device__ __forceinline__ int xcd_remap(int b, int nb) {
  const int q = nb >> 3, rem = nb & 7, x = b & 7, k = b >> 3;
  return x * q + min(x, rem) + k;
}

__device__ __forceinline__ int load_stopped(const Slot* s) {
  return __hip_atomic_load(&s->stopped, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  return v;
}

// Rotations of a value by N lanes within each row of 16 lanes.
template <int N>
__device__ __forceinline__ double row_rotated(double v) {
  union U {
    double d;
    unsigned u[2];
  } a{v}, b;
  for (int k = 0; k < 2; ++k) b.u[k] = __builtin_amdgcn_mov_dpp(a.u[k], 0x120 + N, 0xf, 0xf, true);
  return b.d;
}

// Sum over each row of 16 lanes, in all of them, without LDS traffic.
__device__ __forceinline__ double row16_sum(double v) {
  v += row_rotated<8>(v);
  v += row_rotated<4>(v);
  v += row_rotated<2>(v);
  return v + row_rotated<1>(v);
}

// Sum over the wave's 64 lanes, in every lane: rows of 16, then swaps of rows
// and of halves.
__device__ __forceinline__ double lanes_sum(double v) {
  union U {
    double d;
    unsigned u[2];
  } a{row16_sum(v)}, x, y;
  for (int k = 0; k < 2; ++k) {
    const auto r = __builtin_amdgcn_permlane16_swap(a.u[k], a.u[k], false, false);
    x.u[k] = r[0];
    y.u[k] = r[1];
  }
  a.d = x.d + y.d;
  for (int k = 0; k < 2; ++k) {
    const auto r = __builtin_amdgcn_permlane32_swap(a.u[k], a.u[k], false, false);
    x.u[k] = r[0];
    y.u[k] = r[1];
  }
  return x.d + y.d;
}

// Cross-lane exchange through a wave-private LDS slice: wait for this wave's
// LDS traffic and keep the compiler from moving memory operations across.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
  __builtin_amdgcn_wave_barrier();
}

// Early-termination verdict of one Leja substep from the reduced norms of the
// iteration just finished (Section 3; our reading: stop once
// |d_i| |w_i| + |d_{i-1}| |w_{i-1}| <= tol |v|).
__device__ __forceinline__ void leja_verdict(Slot* S, bool first, bool early, double tol, double dabs,
                                             double d0abs, double wsq, double vsq) {
  const double wn = sqrt(wsq);
  const double vn = first ? sqrt(vsq) : S->vnorm;
  const double prev = first ? d0abs * vn : S->prev_term;
  const double term = dabs * wn;
  const double est = term + prev;
  const bool bad = !isfinite(wsq) || !isfinite(vn);
  if (bad) S->status |= 1;
  S->vnorm = vn;
  S->prev_term = term;
  S->last_est = est;
  S->iters_sub = first ? 1 : S->iters_sub + 1;
  S->stopped = (bad || (early && est <= tol * vn)) ? 1 : 0;
  S->iters_total += 1;
}

// The launch's arguments with the coefficients of the current step read from
// its table column when it runs from a replayed graph (uniform scalar loads).
__device__ __forceinline__ IterArgs resolve_args(const IterArgs& in) {
  IterArgs a = in;
  if (!in.coef) return a;
  const IterCoef* c = in.coef + (long long)(*in.step) * in.coef_stride;
  if (!in.unit_a) {
    a.a1 = c->a1;
    a.a2 = c->a2;
  }
  a.kap = c->kap;
  a.sigma = c->sigma;
  a.d = make_double2(c->dre, c->dim);
  a.d0 = make_double2(c->d0re, c->d0im);
  a.dabs = c->dabs;
  a.d0abs = c->d0abs;
  a.prev_dabs = c->prev_dabs;
  a.tol = c->tol;
  a.skip = !c->active;
  return a;
}

// Whether an iteration launch must return at once because its substep has
// stopped.  Without a.fused the verdict of the previous iteration is in the
// slot (written by the decide kernel launched after it).  With a.fused, every
// workgroup reduces the previous iteration's partials itself in one fixed
// order (each thread a fixed subset in order, then the waves in order), so
// every workgroup reaches the same verdict; workgroup 0 records it in the
// slot and counts the iteration.  Called by every thread of the workgroup;
// the result is uniform over it.  Slot fields written here are never read by
// the same launch: term[] is double-buffered by iteration parity, vnorm is
// written on the second iteration only, when every workgroup computes it.
// lds: kFuseLds doubles of the caller's LDS, free to reuse once this returns.
//
// Two halves, so that a kernel can put loads of its own between them: the
// test's inputs all lie in memory that the previous launch wrote, each load is
// a round trip of about a microsecond, and none depends on another, so
// stop_loads issues them together (reading the slot after the sums instead
// cost two more round trips in every iteration).
constexpr int kFuseLds = 40;
constexpr int kStopLoads = 4;  // partial sums per thread: kFuseMaxGrid over at least 256 threads
template <int N = kStopLoads>
struct StopLoads {
  double w[N], v[N];
  double vnorm, term;
  int stopped;
};
template <int N>
__device__ __forceinline__ void stop_loads(const IterArgs& a, StopLoads<N>& s) {
  s.stopped = a.check_stop ? load_stopped(a.slot) : 0;
  if (!a.fused || !a.check_stop) return;
  const int n = a.prev_grid, nt = blockDim.x, tid = threadIdx.x;
#pragma unroll
  for (int u = 0; u < N; ++u) s.w[u] = a.prev_partials[min(u * nt + tid, n - 1)];
  s.vnorm = s.term = 0.0;
  if (a.iter == 2) {  // the previous iteration was the substep's first
#pragma unroll
    for (int u = 0; u < N; ++u) s.v[u] = a.prev_partials[n + min(u * nt + tid, n - 1)];
  } else {
    s.vnorm = a.slot->vnorm;
    s.term = a.slot->term[a.iter & 1];  // iteration iter-2's term
  }
}

template <int N>
__device__ __forceinline__ bool stop_verdict(const IterArgs& a, const StopLoads<N>& s, double* lds) {
  if (!a.fused) return a.skip || s.stopped;
  Slot* S = a.slot;
  const int tid = threadIdx.x;
  if (!a.check_stop) {  // a substep's first iteration: it always runs
    if (blockIdx.x == 0 && tid == 0) {
      S->stopped = 0;
      S->iters_sub = 1;
      S->iters_total += 1;
    }
    return false;
  }
  double* fz_w = lds;       // per-wave sums (at most 16 waves)
  double* fz_v = lds + 16;
  if (tid == 0) lds[32] = s.stopped ? 1.0 : 0.0;  // one thread's reading for all: workgroup 0 may be writing it
  const int n = a.prev_grid, nt = blockDim.x;
  const bool vfirst = a.iter == 2;
  double sw = 0.0, sv = 0.0;
#pragma unroll
  for (int u = 0; u < N; ++u)
    if (u * nt + tid < n) {
      sw += s.w[u];
      if (vfirst) sv += s.v[u];
    }
  sw = wave_sum(sw);
  if (vfirst) sv = wave_sum(sv);
  const int lane = tid & 63, wv = tid >> 6, nw = nt >> 6;
  if (lane == 0) {
    fz_w[wv] = sw;
    fz_v[wv] = sv;
  }
  __syncthreads();
  // past this step's degree (uniform: scalar loads), or stopped by an earlier verdict of this substep
  if (a.skip || lds[32] != 0.0) return true;
  double tw = 0.0, tv = 0.0;
  for (int w = 0; w < nw; ++w) {
    tw += fz_w[w];
    tv += fz_v[w];
  }
  __syncthreads();  // every wave has read the sums: the caller may reuse lds
  const double vn = vfirst ? sqrt(tv) : s.vnorm;
  const double prev = vfirst ? a.d0abs * vn : s.term;
  const double term = a.prev_dabs * sqrt(tw);
  const double est = term + prev;
  const bool bad = !isfinite(tw) || !isfinite(vn);
  const bool stop = bad || (a.early && est <= a.tol * vn);
  if (blockIdx.x == 0 && tid == 0) {
    if (bad) S->status |= 1;
    if (vfirst) S->vnorm = vn;
    S->term[(a.iter - 1) & 1] = term;
    S->last_est = est;
    if (stop) {
      S->stopped = 1;
    } else {
      S->iters_sub = a.iter;
      S->iters_total += 1;
    }
  }
  return stop;
}

__device__ __forceinline__ bool iteration_stopped(const IterArgs& a, double* lds) {
  StopLoads<> s;
  stop_loads(a, s);
  return stop_verdict(a, s, lds);
}

// Leja update for one row; y = (scale-folded) H_hat w at that row.
__device__ __forceinline__ void leja_row(const IterArgs& a, int r, d2 y, double& pw, double& pv) {
  const d2 w_old = tod2(a.wcur[r]);
  const d2 wn = y - rmul(a.sigma, w_old);
  d2 p;
  if (a.first) {
    p = cmul(tod2(a.d0), w_old) + cmul(tod2(a.d), wn);
    pv += nrm2(w_old);
  } else {
    p = tod2(a.pacc[r]) + cmul(tod2(a.d), wn);
  }
  a.wout[r] = fromd2(wn);
  a.pacc[r] = fromd2(p);
  pw += nrm2(wn);
}

// |w_i|^2 of the workgroup at partials[blockIdx.x]; on a substep's first
// iteration also |v|^2 at partials[gridDim.x + blockIdx.x].
__device__ __forceinline__ void store_partials(const IterArgs& a, double bw, double bv) {
  a.partials[blockIdx.x] = bw;
  if (a.first) a.partials[gridDim.x + blockIdx.x] = bv;
}

// Block sums of the norm partials, one pair per workgroup (plain stores: the
// reduction across workgroups happens in leja_decide_kernel, after this
// kernel has finished, so no device-scope atomics or fences are needed).
__device__ __forceinline__ void block_partials(const IterArgs& a, double pw, double pv) {
  __shared__ double red[2][kThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  pw = wave_sum(pw);
  pv = wave_sum(pv);
  if (lane == 0) { red[0][wv] = pw; red[1][wv] = pv; }
  __syncthreads();
  if (tid == 0) {
    double bw = 0.0, bv = 0.0;
    for (int w = 0; w < kThreads / 64; ++w) { bw += red[0][w]; bv += red[1][w]; }
    store_partials(a, bw, bv);
  }
}

}  // namespace dev
}  // namespace magnus

// HIP kernels of libmagnus for gfx950 (CDNA4, wave64).
//
// The hot loop is one Leja iteration (Section 3, the Newton-form recurrence
// w <- A w - xi_{i-1} w, p <- p + d_i w), fused into a single pass over the
// Hamiltonian: the matrix-vector product of both terms of H(t) = H1 + f H2
// (Section 4), the shift, the accumulation into p, and the partial sums of
// |w_i|^2 (and |v|^2 on the first iteration) for the error control.  A
// one-workgroup kernel that follows reduces the partials in a fixed order and
// writes the early-termination verdict for the next iteration to read, so the
// host never waits.
#include "device_common.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace magnus {
namespace {

using namespace dev;

// One workgroup: reduce the partials of the iteration just finished in a
// fixed order, then the early-termination test of Section 3 (our reading:
// stop once |d_i w_i| + |d_{i-1} w_{i-1}| <= tol |v|).  Every thread issues
// all of its loads before summing, so the kernel costs about one memory
// round trip.  The kernel sits between every two iterations, so its own
// dispatch and completion matter on small grids: four waves dispatch and
// finish sooner than sixteen (measured, Cf4 on chains: n = 13 6,531 -> 7,548
// steps/s, n = 16 3,579 -> 3,829, n = 20 unchanged).
constexpr int kDecideThreads = 256;
constexpr int kDecidePer = 16;
// sum of p[0..n) over the workgroup's threads (each thread's loads all issued first)
__device__ __forceinline__ double decide_sum(const double* p, int n, int tid) {
  double s = 0.0;
  for (int k0 = 0; k0 < n; k0 += kDecideThreads * kDecidePer) {
    double v[kDecidePer];
#pragma unroll
    for (int u = 0; u < kDecidePer; ++u) {
      const int k = k0 + u * kDecideThreads + tid;
      v[u] = k < n ? p[k] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < kDecidePer; ++u) s += v[u];
  }
  return s;
}

__global__ __launch_bounds__(kDecideThreads) void leja_decide_kernel(IterArgs a, int grid) {
  __shared__ double red[2][kDecideThreads / 64];
  if (a.check_stop && load_stopped(a.slot)) return;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  // |v|^2 partials exist (and matter) only on a substep's first iteration
  double sw = decide_sum(a.partials, grid, tid);
  double sv = a.first ? decide_sum(a.partials + grid, grid, tid) : 0.0;
  sw = wave_sum(sw);
  sv = wave_sum(sv);
  if (lane == 0) { red[0][wv] = sw; red[1][wv] = sv; }
  __syncthreads();
  if (tid == 0) {
    double tw = 0.0, tv = 0.0;
    for (int w = 0; w < kDecideThreads / 64; ++w) { tw += red[0][w]; tv += red[1][w]; }
    leja_verdict(a.slot, a.first, a.early, a.tol, a.dabs, a.d0abs, tw, tv);
  }
}

// After the last iteration of a call whose stop tests were fused into the
// iteration kernels: no later launch reduces that iteration's partials, so
// this one checks them for non-finite norms (unless the substep had stopped
// before it, leaving stale partials).
__global__ __launch_bounds__(kDecideThreads) void leja_final_check_kernel(IterArgs a) {
  __shared__ double red[2][kDecideThreads / 64];
  if (load_stopped(a.slot)) return;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  double sw = decide_sum(a.prev_partials, a.prev_grid, tid);
  double sv = a.iter == 2 ? decide_sum(a.prev_partials + a.prev_grid, a.prev_grid, tid) : 0.0;
  sw = wave_sum(sw);
  sv = wave_sum(sv);
  if (lane == 0) { red[0][wv] = sw; red[1][wv] = sv; }
  __syncthreads();
  if (tid == 0) {
    double tw = 0.0, tv = 0.0;
    for (int w = 0; w < kDecideThreads / 64; ++w) { tw += red[0][w]; tv += red[1][w]; }
    if (!isfinite(tw) || !isfinite(tv)) a.slot->status |= 1;
  }
}

// ---------------------------------------------------------------------------
// Two-term CSR iteration.  A workgroup owns ROWS consecutive rows; all of its
// threads stream the rows' nonzeros of both terms (coalesced, non-temporal,
// so the gathered vectors keep the caches), multiply by the gathered vector
// entries and stage the products in LDS; then LPR threads per row sum the
// row's products in a fixed order.  Any nonzero distribution is handled by
// processing the workgroup's nonzeros in chunks of CAP.
// ---------------------------------------------------------------------------
template <int ROWS, int MODE>
__global__ __launch_bounds__(kThreads) void csr2_iter_kernel(CsrDev t1, CsrDev t2, int dim, IterArgs a_in) {
  const IterArgs a = resolve_args(a_in);
  constexpr int LPR = kThreads / ROWS;
  constexpr int CAP = ROWS * 32;
  constexpr int U = 4;
  __shared__ d2 prod[CAP];
  __shared__ int rps[2][ROWS + 1];
  static_assert(2 * CAP >= kFuseLds, "stop-test scratch");
  if (iteration_stopped(a, reinterpret_cast<double*>(prod))) return;

  const int tid = threadIdx.x;
  const int L = xcd_remap(blockIdx.x, gridDim.x);
  const int row0 = L * ROWS;
  const int nrows = min(ROWS, dim - row0);
  for (int i = tid; i <= nrows; i += kThreads) {
    rps[0][i] = t1.rp[row0 + i];
    rps[1][i] = t2.rp[row0 + i];
  }
  __syncthreads();
  const int base1 = rps[0][0], n1 = rps[0][nrows] - base1;
  const int base2 = rps[1][0], n2 = rps[1][nrows] - base2;
  const int total = n1 + n2;
  const int rr = tid / LPR, q = tid % LPR;
  int s1 = 0, e1 = 0, s2 = 0, e2 = 0;
  if (rr < nrows) {
    s1 = rps[0][rr] - base1;
    e1 = rps[0][rr + 1] - base1;
    s2 = n1 + rps[1][rr] - base2;
    e2 = n1 + rps[1][rr + 1] - base2;
  }
  const d2* x1 = reinterpret_cast<const d2*>(a.x1);
  const d2* x2 = reinterpret_cast<const d2*>(a.x2);
  const d2* v1 = reinterpret_cast<const d2*>(t1.val);
  const d2* v2 = reinterpret_cast<const d2*>(t2.val);
  d2 acc1 = {0.0, 0.0}, acc2 = {0.0, 0.0};

  for (int c0 = 0; c0 < total; c0 += CAP) {
    const int cn = min(CAP, total - c0);
    for (int kb = 0; kb < cn; kb += kThreads * U) {
      int col[U];
      d2 val[U];
      bool in1[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = kb + u * kThreads + tid;
        const int g = c0 + k;
        in1[u] = g < n1;
        col[u] = 0;
        val[u] = d2{0.0, 0.0};
        if (k < cn) {
          if (in1[u]) {
            col[u] = __builtin_nontemporal_load(t1.ci + base1 + g);
            val[u] = __builtin_nontemporal_load(v1 + base1 + g);
          } else {
            col[u] = __builtin_nontemporal_load(t2.ci + base2 + (g - n1));
            val[u] = __builtin_nontemporal_load(v2 + base2 + (g - n1));
          }
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = kb + u * kThreads + tid;
        if (k < cn) {
          const d2 x = in1[u] ? x1[col[u]] : x2[col[u]];
          prod[k] = cmul(val[u], x);
        }
      }
    }
    __syncthreads();
    if (rr < nrows) {
      const int hi = c0 + cn;
      for (int k = max(s1, c0) + q; k < min(e1, hi); k += LPR) acc1 += prod[k - c0];
      for (int k = max(s2, c0) + q; k < min(e2, hi); k += LPR) acc2 += prod[k - c0];
    }
    __syncthreads();
  }
#pragma unroll
  for (int off = LPR / 2; off > 0; off >>= 1) {
    acc1.x += __shfl_xor(acc1.x, off, 64);
    acc1.y += __shfl_xor(acc1.y, off, 64);
    acc2.x += __shfl_xor(acc2.x, off, 64);
    acc2.y += __shfl_xor(acc2.y, off, 64);
  }
  const bool owner = (q == 0) && (rr < nrows);
  const int r = row0 + rr;
  if constexpr (MODE == kSplit) {
    if (owner) {
      a.wout[r] = fromd2(acc1);
      a.pacc[r] = fromd2(acc2);
    }
    return;
  } else {
    double pw = 0.0, pv = 0.0;
    if (owner) {
      d2 y;
      if constexpr (MODE == kLeja) {
        y = rmul(a.a1, acc1) + rmul(a.a2, acc2);
      } else {
        const d2 Ur = x2[r], Vr = x1[r];
        const d2 dl = acc1 - acc2;
        y = rmul(a.a1, Ur) + rmul(a.a2, Vr) + d2{-a.kap * dl.y, a.kap * dl.x};
      }
      leja_row(a, r, y, pw, pv);
    }
    block_partials(a, pw, pv);
  }
}

// ---------------------------------------------------------------------------
// Two-term CSR iteration, row-per-lane variant.  The workgroup first copies
// its rows' column indices and values (both terms) into LDS with coalesced,
// non-temporal loads; then lane l of every wave owns row row0 + l and wave q
// walks the row's entries k = q, q + 4, ... .  Neighbouring lanes therefore
// gather x at the same position of neighbouring rows, which for structured
// Hamiltonians (neighbouring basis states couple to neighbouring states) turns
// most gathers into contiguous 1 KiB loads.  The four partial sums per row are
// combined in LDS in a fixed order and wave 0 applies the Leja update to 64
// consecutive rows with coalesced stores.
// ---------------------------------------------------------------------------
template <int ROWS, int MODE>
__global__ __launch_bounds__(kThreads) void csr2_rowlane_kernel(CsrDev t1, CsrDev t2, int dim, IterArgs a_in) {
  const IterArgs a = resolve_args(a_in);
  constexpr int NW = kThreads / ROWS;  // entry groups per row
  constexpr int CAP = ROWS * 32;
  constexpr int U = CAP / kThreads;
  __shared__ d2 sval[CAP];
  __shared__ int scol[CAP];
  __shared__ int rps[2][ROWS + 1];
  __shared__ d2 part[2][NW][ROWS];
  __shared__ double wred[2][kThreads / 64];
  static_assert(2 * CAP >= kFuseLds, "stop-test scratch");
  if (iteration_stopped(a, reinterpret_cast<double*>(sval))) return;

  const int tid = threadIdx.x;
  const int lane = tid % ROWS, wv = tid / ROWS;  // row within the block, entry group
  const int L = xcd_remap(blockIdx.x, gridDim.x);
  const int row0 = L * ROWS;
  const int nrows = min(ROWS, dim - row0);
  for (int i = tid; i <= nrows; i += kThreads) {
    rps[0][i] = t1.rp[row0 + i];
    rps[1][i] = t2.rp[row0 + i];
  }
  __syncthreads();
  const int base1 = rps[0][0], n1 = rps[0][nrows] - base1;
  const int base2 = rps[1][0], n2 = rps[1][nrows] - base2;
  const int total = n1 + n2;
  // this lane's row segments in the concatenated (term 1, term 2) sequence
  int s1 = 0, e1 = 0, s2 = 0, e2 = 0;
  if (lane < nrows) {
    s1 = rps[0][lane] - base1;
    e1 = rps[0][lane + 1] - base1;
    s2 = n1 + rps[1][lane] - base2;
    e2 = n1 + rps[1][lane + 1] - base2;
  }
  const d2* x1 = reinterpret_cast<const d2*>(a.x1);
  const d2* x2 = reinterpret_cast<const d2*>(a.x2);
  const d2* v1 = reinterpret_cast<const d2*>(t1.val);
  const d2* v2 = reinterpret_cast<const d2*>(t2.val);
  d2 acc1 = {0.0, 0.0}, acc2 = {0.0, 0.0};

  for (int c0 = 0; c0 < total; c0 += CAP) {
    const int cn = min(CAP, total - c0);
    int col[U];
    d2 val[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = u * kThreads + tid;
      const int g = c0 + k;
      col[u] = 0;
      val[u] = d2{0.0, 0.0};
      if (k < cn) {
        if (g < n1) {
          col[u] = __builtin_nontemporal_load(t1.ci + base1 + g);
          val[u] = __builtin_nontemporal_load(v1 + base1 + g);
        } else {
          col[u] = __builtin_nontemporal_load(t2.ci + base2 + (g - n1));
          val[u] = __builtin_nontemporal_load(v2 + base2 + (g - n1));
        }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = u * kThreads + tid;
      if (k < cn) {
        scol[k] = col[u];
        sval[k] = val[u];
      }
    }
    __syncthreads();
    const int hi = c0 + cn;
    {
      const int lo = max(s1, c0) + wv, end = min(e1, hi);
#pragma unroll 4
      for (int k = lo; k < end; k += NW) acc1 += cmul(sval[k - c0], x1[scol[k - c0]]);
    }
    {
      const int lo = max(s2, c0) + wv, end = min(e2, hi);
#pragma unroll 4
      for (int k = lo; k < end; k += NW) acc2 += cmul(sval[k - c0], x2[scol[k - c0]]);
    }
    __syncthreads();
  }
  part[0][wv][lane] = acc1;
  part[1][wv][lane] = acc2;
  __syncthreads();
  // threads 0..ROWS-1 finish one row each (lane == tid there)
  const bool owner = tid < ROWS && lane < nrows;
  const int r = row0 + lane;
  d2 r1 = {0.0, 0.0}, r2 = {0.0, 0.0};
  if (tid < ROWS) {
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      r1 += part[0][w][lane];
      r2 += part[1][w][lane];
    }
  }
  if constexpr (MODE == kSplit) {
    if (owner) {
      a.wout[r] = fromd2(r1);
      a.pacc[r] = fromd2(r2);
    }
  } else {
    double pw = 0.0, pv = 0.0;
    if (owner) {
      d2 y;
      if constexpr (MODE == kLeja) {
        y = rmul(a.a1, r1) + rmul(a.a2, r2);
      } else {
        const d2 Ur = x2[r], Vr = x1[r];
        const d2 dl = r1 - r2;
        y = rmul(a.a1, Ur) + rmul(a.a2, Vr) + d2{-a.kap * dl.y, a.kap * dl.x};
      }
      leja_row(a, r, y, pw, pv);
    }
    pw = wave_sum(pw);
    pv = wave_sum(pv);
    if ((tid & 63) == 0) { wred[0][tid >> 6] = pw; wred[1][tid >> 6] = pv; }
    __syncthreads();
    if (tid == 0) {
      double bw = 0.0, bv = 0.0;
      for (int k = 0; k < kThreads / 64; ++k) { bw += wred[0][k]; bv += wred[1][k]; }
      store_partials(a, bw, bv);
    }
  }
}

// ---------------------------------------------------------------------------
// Two-term CSR iteration, wave-tile variant.  Every wave owns RPW consecutive
// rows and works through them on its own: it stages its rows' column indices
// and values (both terms) in a private LDS slice with coalesced non-temporal
// loads, gathers x with lanes laid out row-fastest (lane = g * RPW + r, so
// neighbouring lanes gather the same entry position of neighbouring rows),
// sums each row's G = 64 / RPW groups with shuffles in a fixed order and
// applies the Leja update to its RPW rows.  No block-wide barrier separates
// the phases, so the waves of a CU overlap freely; the only barrier combines
// the four waves' norm partials at the end.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this wave's LDS accesses are done
  __builtin_amdgcn_wave_barrier();
}

// Seven waves per SIMD (at most 72 VGPRs): enough independent tiles in flight
// per CU to cover the memory latency of each tile's load -> gather chain.  The
// commutator pass holds two more own-row vectors and gets six (no spills).
// keep_entries: tiles whose entries start within the first keep_entries of the
// two terms together are read with normal loads, so that they stay in the
// memory-side cache (MALL) until the next pass over the matrix; the rest are
// read non-temporally.
template <int RPW, int MODE>
__global__ __launch_bounds__(kThreads, MODE == kLejaComm ? 6 : 7) void csr2_wave_kernel(CsrDev t1, CsrDev t2, int dim, IterArgs a_in,
                                                                                      int keep_entries) {
  const IterArgs a = resolve_args(a_in);
  constexpr int NWAVE = kThreads / 64;
  constexpr int G = 64 / RPW;      // entry groups per row
  constexpr int CAPW = RPW * 32;   // entries staged per chunk
  constexpr int U = CAPW / 64;     // entries per lane per chunk
  static_assert(RPW + 1 <= 32, "row pointers are loaded by half-waves");
  __shared__ d2 sval[NWAVE][CAPW];
  __shared__ int scol[NWAVE][CAPW];
  __shared__ int srp[NWAVE][2][RPW + 1];
  __shared__ double wred[2][NWAVE];
  // The stop flag is the same for every wave of the launch; it is tested only
  // once the row pointers and own-row operands are in flight, so its latency
  // overlaps theirs (the fused test reduces the partials first).
  const bool stopped = iteration_stopped(a, reinterpret_cast<double*>(&sval[0][0]));

  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int L = xcd_remap(blockIdx.x, gridDim.x);
  const int row0 = (L * NWAVE + wv) * RPW;
  const int nrows = max(0, min(RPW, dim - row0));
  const int r = lane % RPW, g = lane / RPW;
  const bool owner = (lane < RPW) && (r < nrows);
  const int row = row0 + r;
  double pw = 0.0, pv = 0.0;

  int rpa = 0, rpb = 0;
  d2 w_old = {0.0, 0.0}, p_old = {0.0, 0.0}, own1 = {0.0, 0.0}, own2 = {0.0, 0.0};
  if (nrows > 0) {
    if (lane <= nrows) rpa = t1.rp[row0 + lane];
    if (lane >= 32 && lane - 32 <= nrows) rpb = t2.rp[row0 + lane - 32];
    // own-row operands of the update, fetched early
    if (owner) {
      if constexpr (MODE != kSplit) {
        w_old = tod2(a.wcur[row]);
        if (!a.first) p_old = tod2(a.pacc[row]);
      }
      if constexpr (MODE == kLejaComm) {
        own1 = tod2(a.x1[row]);
        own2 = tod2(a.x2[row]);
      }
    }
  }
  if (stopped) return;  // uniform over the workgroup

  if (nrows > 0) {
    if (lane <= nrows) srp[wv][0][lane] = rpa;
    if (lane >= 32 && lane - 32 <= nrows) srp[wv][1][lane - 32] = rpb;
    wave_lds_sync();
    const int base1 = srp[wv][0][0], n1 = srp[wv][0][nrows] - base1;
    const int base2 = srp[wv][1][0], n2 = srp[wv][1][nrows] - base2;
    const int total = n1 + n2;
    int s1 = 0, e1 = 0, s2 = 0, e2 = 0;
    if (r < nrows) {
      s1 = srp[wv][0][r] - base1;
      e1 = srp[wv][0][r + 1] - base1;
      s2 = n1 + srp[wv][1][r] - base2;
      e2 = n1 + srp[wv][1][r + 1] - base2;
    }
    const d2* x1 = reinterpret_cast<const d2*>(a.x1);
    const d2* x2 = reinterpret_cast<const d2*>(a.x2);
    const d2* v1 = reinterpret_cast<const d2*>(t1.val);
    const d2* v2 = reinterpret_cast<const d2*>(t2.val);
    d2 acc1 = {0.0, 0.0}, acc2 = {0.0, 0.0};
    const bool keep = (long long)base1 + base2 < keep_entries;  // uniform over the wave (no int overflow)
    for (int c0 = 0; c0 < total; c0 += CAPW) {
      const int cn = min(CAPW, total - c0);
      int col[U];
      d2 val[U];
      auto load_chunk = [&](auto streaming) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int k = u * 64 + lane;
          const int gk = c0 + k;
          col[u] = 0;
          val[u] = d2{0.0, 0.0};
          auto ld = [&](const auto* p) {
            if constexpr (decltype(streaming)::value) return __builtin_nontemporal_load(p);
            else return *p;
          };
          if (k < cn) {
            if (gk < n1) {
              col[u] = ld(t1.ci + base1 + gk);
              val[u] = ld(v1 + base1 + gk);
            } else {
              col[u] = ld(t2.ci + base2 + (gk - n1));
              val[u] = ld(v2 + base2 + (gk - n1));
            }
          }
        }
      };
      if (keep) load_chunk(std::false_type{});
      else load_chunk(std::true_type{});
      wave_lds_sync();  // the previous chunk's LDS reads are done
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = u * 64 + lane;
        if (k < cn) {
          scol[wv][k] = col[u];
          sval[wv][k] = val[u];
        }
      }
      wave_lds_sync();
      const int hi = c0 + cn;
      {
        const int lo = max(s1, c0) + g, end = min(e1, hi);
#pragma unroll 4
        for (int k = lo; k < end; k += G) acc1 += cmul(sval[wv][k - c0], x1[scol[wv][k - c0]]);
      }
      {
        const int lo = max(s2, c0) + g, end = min(e2, hi);
#pragma unroll 4
        for (int k = lo; k < end; k += G) acc2 += cmul(sval[wv][k - c0], x2[scol[wv][k - c0]]);
      }
    }
#pragma unroll
    for (int off = 32; off >= RPW; off >>= 1) {
      acc1.x += __shfl_xor(acc1.x, off, 64);
      acc1.y += __shfl_xor(acc1.y, off, 64);
      acc2.x += __shfl_xor(acc2.x, off, 64);
      acc2.y += __shfl_xor(acc2.y, off, 64);
    }
    if (owner) {
      if constexpr (MODE == kSplit) {
        a.wout[row] = fromd2(acc1);
        a.pacc[row] = fromd2(acc2);
      } else {
        d2 y;
        if constexpr (MODE == kLeja) {
          y = rmul(a.a1, acc1) + rmul(a.a2, acc2);
        } else {
          // own2 = U_r (term-2 gather vector), own1 = V_r (term-1 gather vector)
          const d2 dl = acc1 - acc2;
          y = rmul(a.a1, own2) + rmul(a.a2, own1) + d2{-a.kap * dl.y, a.kap * dl.x};
        }
        const d2 wn = y - rmul(a.sigma, w_old);
        d2 p;
        if (a.first) {
          p = cmul(tod2(a.d0), w_old) + cmul(tod2(a.d), wn);
          pv = nrm2(w_old);
        } else {
          p = p_old + cmul(tod2(a.d), wn);
        }
        a.wout[row] = fromd2(wn);
        a.pacc[row] = fromd2(p);
        pw = nrm2(wn);
      }
    }
  }
  if constexpr (MODE != kSplit) {
    pw = wave_sum(pw);
    pv = wave_sum(pv);
    if (lane == 0) { wred[0][wv] = pw; wred[1][wv] = pv; }
    __syncthreads();
    if (tid == 0) {
      double bw = 0.0, bv = 0.0;
      for (int k = 0; k < NWAVE; ++k) { bw += wred[0][k]; bv += wred[1][k]; }
      store_partials(a, bw, bv);
    }
  }
}

// ---------------------------------------------------------------------------
// CSR iteration on two terms, or with NT = 3 also on the assembled commutator
// (mode kLeja), eight lanes per row without staging.  A lane takes every eighth
// entry of the row's terms (one list, term 1's first), U of them at a time.
// Up to about 2^15 rows an iteration is bound by its chain of dependent loads:
// the stop test's inputs, the row's bounds and its own elements go out first,
// then the U entries, then (once the verdict is known) the U gathers; beyond
// that by the gathers that leave the L2.  Against staging a block's entries in
// LDS with a row to a lane, us per iteration: chains, n = 13 6.3, now 5.2,
// n = 14 6.8, now 5.9; 50,021 rows of 24 random entries 17.2, now 15.7; with the
// commutator assembled, n = 12 8.1 (a wave to 8 rows), now 5.3, n = 16 24.6, now
// 16.7.  U = 4 leaves rows of 24 entries a second chain of loads (16.1), U = 6
// takes registers (15.7, and 6.7 / 6.5 at 5,000 rows of 38).
// ---------------------------------------------------------------------------
constexpr int kRowLanes = 8;

// Sum over the 8 lanes of a row, in all of them: quads, then the quads' mirror images.
__device__ __forceinline__ double lanes8_sum(double v) {
  auto moved = [](double x, auto ctrl) {
    union U {
      double d;
      unsigned u[2];
    } a{x}, b;
    for (int j = 0; j < 2; ++j) b.u[j] = __builtin_amdgcn_mov_dpp(a.u[j], decltype(ctrl)::value, 0xf, 0xf, true);
    return b.d;
  };
  v += moved(v, std::integral_constant<int, 0xB1>{});   // quad_perm 1, 0, 3, 2
  v += moved(v, std::integral_constant<int, 0x4E>{});   // quad_perm 2, 3, 0, 1
  return v + moved(v, std::integral_constant<int, 0x141>{});  // row_half_mirror
}

// STOP: the previous iteration's partial sums per thread.
template <int MODE, int NT, int TH, int STOP>
__global__ __launch_bounds__(TH, 5) void csr_rows_kernel(CsrDev t1, CsrDev t2, CsrDev t3, int dim, IterArgs a_in,
                                                         double a3_arg) {
  const IterArgs a = resolve_args(a_in);
  const double a3 = a_in.coef ? a.kap : a3_arg;
  constexpr int U = 5;
  __shared__ double fz[kFuseLds];
  __shared__ double red[2][TH / 64];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, q = tid % kRowLanes;
  const int L = xcd_remap(blockIdx.x, gridDim.x);
  const int r = L * (TH / kRowLanes) + tid / kRowLanes, row = min(r, dim - 1);
  const d2* x1 = reinterpret_cast<const d2*>(a.x1);
  const d2* x2 = reinterpret_cast<const d2*>(a.x2);
  const d2* v1 = reinterpret_cast<const d2*>(t1.val);
  const d2* v2 = reinterpret_cast<const d2*>(t2.val);
  const d2* v3 = reinterpret_cast<const d2*>(t3.val);
  StopLoads<STOP> stop;
  stop_loads(a, stop);
  const int s1 = t1.rp[row], s2 = t2.rp[row];
  const int s3 = NT == 3 ? t3.rp[row] : 0, e3 = NT == 3 ? t3.rp[row + 1] : 0;
  const int n1 = r < dim ? t1.rp[row + 1] - s1 : 0, n2 = r < dim ? n1 + t2.rp[row + 1] - s2 : 0;
  const int n = r < dim ? n2 + e3 - s3 : 0;  // (n1, n2, n: where the terms end in the row's list)
  d2 w_old, p_old = {0.0, 0.0}, u_old = {0.0, 0.0}, v_old = {0.0, 0.0};
  if (MODE != kSplit) {
    w_old = tod2(a.wcur[row]);
    if (!a.first) p_old = tod2(a.pacc[row]);
    if (MODE == kLejaComm) {
      u_old = x2[row];
      v_old = x1[row];
    }
  }
  int col[U];
  d2 val[U];
  auto load = [&](int k0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = k0 + kRowLanes * u;
      col[u] = 0;
      val[u] = d2{0.0, 0.0};
      if (k < n) {
        const bool in1 = k < n1, in2 = NT == 2 || k < n2;
        col[u] = (in1 ? t1.ci + s1 : in2 ? t2.ci + (s2 - n1) : t3.ci + (s3 - n2))[k];
        val[u] = (in1 ? v1 + s1 : in2 ? v2 + (s2 - n1) : v3 + (s3 - n2))[k];
      }
    }
  };
  load(q);
  __builtin_amdgcn_sched_barrier(0);
  if (stop_verdict(a, stop, fz)) return;
  d2 acc1 = {0.0, 0.0}, acc2 = {0.0, 0.0};
  for (int k0 = q;;) {
    d2 g[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      g[u] = d2{0.0, 0.0};
      if (k0 + kRowLanes * u < n) g[u] = (k0 + kRowLanes * u < n1 ? x1 : x2)[col[u]];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const d2 y = cmul(val[u], g[u]);
      const bool in1 = k0 + kRowLanes * u < n1;
      if constexpr (NT == 3) {
        acc1 += rmul(in1 ? a.a1 : k0 + kRowLanes * u < n2 ? a.a2 : a3, y);
      } else {
        acc1 += in1 ? y : d2{0.0, 0.0};
        acc2 += in1 ? d2{0.0, 0.0} : y;
      }
    }
    k0 += kRowLanes * U;
    if (!__any(k0 < n)) break;
    load(k0);
  }
  acc1 = d2{lanes8_sum(acc1.x), lanes8_sum(acc1.y)};
  if (NT == 2) acc2 = d2{lanes8_sum(acc2.x), lanes8_sum(acc2.y)};
  const bool owner = q == 0 && r < dim;
  if constexpr (MODE == kSplit) {
    if (owner) {
      a.wout[r] = fromd2(acc1);
      a.pacc[r] = fromd2(acc2);
    }
  } else {
    double pw = 0.0, pv = 0.0;
    if (owner) {
      d2 y;
      if constexpr (NT == 3) {
        y = acc1;
      } else if constexpr (MODE == kLeja) {
        y = rmul(a.a1, acc1) + rmul(a.a2, acc2);
      } else {
        const d2 dl = acc1 - acc2;
        y = rmul(a.a1, u_old) + rmul(a.a2, v_old) + d2{-a.kap * dl.y, a.kap * dl.x};
      }
      const d2 wn = y - rmul(a.sigma, w_old);
      d2 p;
      if (a.first) {
        p = cmul(tod2(a.d0), w_old) + cmul(tod2(a.d), wn);
        pv = nrm2(w_old);
      } else {
        p = p_old + cmul(tod2(a.d), wn);
      }
      a.wout[r] = fromd2(wn);
      a.pacc[r] = fromd2(p);
      pw = nrm2(wn);
    }
    pw = lanes_sum(pw);
    pv = lanes_sum(pv);
    if (lane == 0) {
      red[0][wv] = pw;
      red[1][wv] = pv;
    }
    __syncthreads();
    if (tid == 0) {
      double bw = 0.0, bv = 0.0;
      for (int k = 0; k < TH / 64; ++k) {
        bw += red[0][k];
        bv += red[1][k];
      }
      store_partials(a, bw, bv);
    }
  }
}

// ---------------------------------------------------------------------------
// Dense iterations (row-major matrices), bound by the matrix bytes.  A
// workgroup owns the rows [dim b / grid, dim (b+1) / grid) and its four waves
// split the columns: lane l of wave q sums columns j = 64 q + l + 256 m, so
// every matrix load is a coalesced 1 KiB transaction per wave, and a small
// matrix still has its rows spread over every CU with few loads in each wave's
// chain (rows split over waves instead: N = 1001 one term 10.0 us, now 6.2;
// first M4 iteration with its assembly 26.6, now 14.8).  A wave works on RPW
// rows at a time and loads x_j once for them (and both terms); a group's loads
// (UNR column steps) are issued together.  Workgroups go round the XCDs in the
// order of their rows, so that each reads its share of the rows kept in the
// MALL and of those that stream (rows in a contiguous range per XCD: N = 8192
// 160.6 us, now 153 = 7.0 TB/s from HBM and MALL together).
// ---------------------------------------------------------------------------
constexpr int kDenseMaxRows = 256;  // rows of a workgroup: one thread each for the update

// The rows of a workgroup's products: row by row group the loads of F::load
// and products of F::use over this wave's columns, the lanes' sums to
// part[row][wave].  The first group's loads are issued before the stop test,
// whose own loads they do not depend on; false if the substep has stopped.
template <int RPW, int UNR, class F>
__device__ __forceinline__ bool dense_rows(const IterArgs& a, int dim, int row0, int rows, F& f, d2 (*part)[kThreads / 64],
                                           double* fz) {
  constexpr int kStep = kThreads * UNR;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  StopLoads<> stop;
  stop_loads(a, stop);
  f.load(row0, tid);
  __builtin_amdgcn_sched_barrier(0);
  if (stop_verdict(a, stop, fz)) return false;
  int r = 0, j = tid;  // the group in flight
  for (;;) {
    f.use(row0 + r, j);
    j += kStep;
    if (j - tid >= dim) {
      f.sums(part, r, lane, wv);
      r += RPW;
      j = tid;
      if (r >= rows) break;
    }
    __builtin_amdgcn_sched_barrier(0);
    f.load(row0 + r, j);
    __builtin_amdgcn_sched_barrier(0);
  }
  __syncthreads();
  return true;
}

__device__ __forceinline__ void dense_update(const IterArgs& a, int row0, int rows, d2 (*part)[kThreads / 64]) {
  const int tid = threadIdx.x;
  double pw = 0.0, pv = 0.0;
  if (tid < rows) {
    d2 y = part[tid][0];
#pragma unroll
    for (int k = 1; k < kThreads / 64; ++k) y += part[tid][k];
    leja_row(a, row0 + tid, y, pw, pv);
  }
  block_partials(a, pw, pv);
}

__device__ __forceinline__ int dense_row0(int b, int dim) { return (int)((long long)dim * b / gridDim.x); }

// Rows below keep_rows are read with normal loads so that they stay in the
// memory-side cache (MALL) from one iteration to the next (the matrix is read
// again by every iteration); the rest stream through non-temporally.
template <int RPW, int UNR, int NT, bool STREAM>
struct DenseProduct {
  const d2 *x, *A1, *A2;
  int dim, last;  // last: the workgroup's last row
  long long ld_row;
  double a1, a2;
  d2 xj[UNR], h1[UNR][RPW], h2[UNR][NT == 2 ? RPW : 1], acc1[RPW], acc2[RPW];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int r = 0; r < RPW; ++r) acc1[r] = acc2[r] = d2{0.0, 0.0};
  }
  // columns past the end read the last one and are not used
  __device__ __forceinline__ void load(int row, int j0) {
    auto ld = [](const d2* p) {
      if constexpr (STREAM) return __builtin_nontemporal_load(p);
      else return *p;
    };
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int j = min(j0 + kThreads * u, dim - 1);
      xj[u] = x[j];
#pragma unroll
      for (int r = 0; r < RPW; ++r) {
        if (r > 0 && row + r > last) break;
        const long long off = (row + r) * ld_row;
        h1[u][r] = ld(A1 + off + j);
        if constexpr (NT == 2) h2[u][r] = ld(A2 + off + j);
      }
    }
  }
  __device__ __forceinline__ void use(int, int j0) {
#pragma unroll
    for (int u = 0; u < UNR; ++u)
      if (j0 + kThreads * u < dim)
#pragma unroll
        for (int r = 0; r < RPW; ++r) {
          acc1[r] = fma_c(h1[u][r], xj[u], acc1[r]);
          if constexpr (NT == 2) acc2[r] = fma_c(h2[u][r], xj[u], acc2[r]);
        }
  }
  __device__ __forceinline__ void sums(d2 (*part)[kThreads / 64], int r0, int lane, int wv) {
#pragma unroll
    for (int r = 0; r < RPW; ++r) {
      d2 y = rmul(a1, acc1[r]);
      if constexpr (NT == 2) y += rmul(a2, acc2[r]);
      y = d2{lanes_sum(y.x), lanes_sum(y.y)};
      if (lane == 0 && r0 + r < kDenseMaxRows) part[r0 + r][wv] = y;
    }
    clear();
  }
};

template <int RPW, int UNR, int NT>
__global__ __launch_bounds__(kThreads) void dense2_iter_kernel(const double2* H1, const double2* H2, int dim,
                                                              long long ld, IterArgs a, int keep_rows) {
  __shared__ double fz[kFuseLds];
  __shared__ d2 part[kDenseMaxRows][kThreads / 64];
  const int row0 = dense_row0(blockIdx.x, dim), rows = dense_row0(blockIdx.x + 1, dim) - row0;
  auto products = [&](auto streaming) {
    DenseProduct<RPW, UNR, NT, decltype(streaming)::value> f;
    f.x = reinterpret_cast<const d2*>(a.x1);
    f.A1 = reinterpret_cast<const d2*>(H1);
    f.A2 = reinterpret_cast<const d2*>(H2);
    f.dim = dim;
    f.last = row0 + rows - 1;
    f.ld_row = ld;
    f.a1 = a.a1;
    f.a2 = a.a2;
    f.clear();
    return dense_rows<RPW, UNR>(a, dim, row0, rows, f, part, fz);
  };
  if (!(row0 < keep_rows ? products(std::false_type{}) : products(std::true_type{}))) return;
  dense_update(a, row0, rows, part);
}

// The first iteration of an exponential on dense terms fused with the
// assembly of its exponent: while it streams H1 and H2 (and K) it stores
// Hs = ca H1 + cb H2 (+ ck K) into the assembly buffer (row stride dim, all
// stores non-temporal: dim 8192 Cf4 382 steps/s, against 367 with the rows
// that the next iterations keep in the MALL stored normally and 354 with all
// stores normal) and multiplies Hs x.  Hs is
// formed by the same expression as dense_assemble_kernel, and every lane
// sums the same columns in the same order as the one-term iteration, so the
// result is bitwise that of assembling first and iterating on the assembled
// matrix; the separate assembly pass and one full read of the assembled
// matrix disappear.
template <int RPW, int UNR, bool WITH_K>
struct DenseAssembleProduct : DenseProduct<RPW, UNR, 1, true> {
  using Base = DenseProduct<RPW, UNR, 1, true>;
  DenseAssembly D;
  d2 b[UNR][RPW], k[UNR][WITH_K ? RPW : 1];
  __device__ __forceinline__ void load(int row, int j0) {
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int j = min(j0 + kThreads * u, this->dim - 1);
      this->xj[u] = this->x[j];
#pragma unroll
      for (int r = 0; r < RPW; ++r) {
        const long long row_r = min(row + r, this->last);
        this->h1[u][r] = __builtin_nontemporal_load(reinterpret_cast<const d2*>(D.H1) + row_r * D.ld + j);
        b[u][r] = __builtin_nontemporal_load(reinterpret_cast<const d2*>(D.H2) + row_r * D.ld + j);
        if constexpr (WITH_K)
          k[u][r] = __builtin_nontemporal_load(reinterpret_cast<const d2*>(D.K) + row_r * this->dim + j);
      }
    }
  }
  __device__ __forceinline__ void use(int row, int j0) {
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int j = j0 + kThreads * u;
      if (j < this->dim)
#pragma unroll
        for (int r = 0; r < RPW; ++r) {
          d2 h = fma_r(D.ca, this->h1[u][r], rmul(D.cb, b[u][r]));
          if constexpr (WITH_K) h = fma_r(D.ck, k[u][r], h);
          this->h1[u][r] = h;
          if (row + r <= this->last)
            __builtin_nontemporal_store(h, reinterpret_cast<d2*>(D.out) + (long long)(row + r) * this->dim + j);
        }
    }
    Base::use(row, j0);
  }
};

template <int RPW, int UNR, bool WITH_K>
__global__ __launch_bounds__(kThreads) void dense_assemble_iter_kernel(DenseAssembly D, int dim, IterArgs a) {
  __shared__ double fz[kFuseLds];
  __shared__ d2 part[kDenseMaxRows][kThreads / 64];
  const int row0 = dense_row0(blockIdx.x, dim), rows = dense_row0(blockIdx.x + 1, dim) - row0;
  DenseAssembleProduct<RPW, UNR, WITH_K> f;
  f.x = reinterpret_cast<const d2*>(a.x1);
  f.dim = dim;
  f.last = row0 + rows - 1;
  f.a1 = a.a1;
  f.D = D;
  f.clear();
  if (!dense_rows<RPW, UNR>(a, dim, row0, rows, f, part, fz)) return;
  dense_update(a, row0, rows, part);
}

// ---------------------------------------------------------------------------
// Gershgorin discs + structure check (CSR), one thread per row.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void csr_gershgorin_kernel(CsrDev t, int dim, long long nnz,
                                                                double* out) {
  __shared__ double smin[kThreads], smax[kThreads];
  __shared__ int sbad[kThreads];
  const int tid = threadIdx.x;
  const int r = blockIdx.x * kThreads + tid;
  double lo = INFINITY, hi = -INFINITY;
  int bad = 0;
  if (r < dim) {
    const long long rs = t.rp[r], re = t.rp[r + 1];
    if (r == 0 && rs != 0) bad = 1;
    if (r == dim - 1 && re != nnz) bad = 1;
    if (rs < 0 || re < rs || re > nnz) bad = 1;
    double diag = 0.0, rad = 0.0;
    if (!bad) {
      for (long long j = rs; j < re; ++j) {
        const int c = t.ci[j];
        const double2 v = t.val[j];
        if (c < 0 || c >= dim) { bad = 1; break; }
        if (c == r) { diag += v.x; rad += fabs(v.y); }
        else rad += sqrt(v.x * v.x + v.y * v.y);
      }
    }
    lo = diag - rad;
    hi = diag + rad;
  }
  smin[tid] = lo; smax[tid] = hi; sbad[tid] = bad;
  __syncthreads();
  for (int s = kThreads / 2; s > 0; s >>= 1) {
    if (tid < s) {
      smin[tid] = fmin(smin[tid], smin[tid + s]);
      smax[tid] = fmax(smax[tid], smax[tid + s]);
      sbad[tid] |= sbad[tid + s];
    }
    __syncthreads();
  }
  if (tid == 0) {
    out[3 * blockIdx.x] = smin[0];
    out[3 * blockIdx.x + 1] = smax[0];
    out[3 * blockIdx.x + 2] = (double)sbad[0];
  }
}

// Gershgorin discs of a dense row-major term, one wave per row.
__global__ __launch_bounds__(kThreads) void dense_gershgorin_kernel(const double2* H, int dim, long long ld,
                                                                  double* out) {
  __shared__ double smin[kThreads / 64], smax[kThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int r = blockIdx.x * (kThreads / 64) + wv;
  double lo = INFINITY, hi = -INFINITY;
  if (r < dim) {
    double rad = 0.0, diag = 0.0;
    for (int j = lane; j < dim; j += 64) {
      const double2 v = H[(long long)r * ld + j];
      if (j == r) { diag += v.x; rad += fabs(v.y); }
      else rad += sqrt(v.x * v.x + v.y * v.y);
    }
    rad = wave_sum(rad);
    diag = wave_sum(diag);
    lo = diag - rad;
    hi = diag + rad;
  }
  if (lane == 0) { smin[wv] = lo; smax[wv] = hi; }
  __syncthreads();
  if (tid == 0) {
    double a = INFINITY, b = -INFINITY;
    for (int w = 0; w < kThreads / 64; ++w) { a = fmin(a, smin[w]); b = fmax(b, smax[w]); }
    out[2 * blockIdx.x] = a;
    out[2 * blockIdx.x + 1] = b;
  }
}

__global__ void copy_kernel(const double2* __restrict__ src, double2* __restrict__ dst, long long n) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = src[i];
}

__global__ void step_set_kernel(int* ctr, int value) { *ctr = value; }
__global__ void step_advance_kernel(int* ctr) { *ctr += 1; }

__global__ void slot_reset_kernel(Slot* s, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    s[i].counter = 0u;
    s[i].stopped = 0;
    s[i].iters_sub = 0;
    s[i].status = 0;
    s[i].iters_total = 0;
    s[i].vnorm = 0.0;
    s[i].prev_term = 0.0;
    s[i].last_est = 0.0;
    s[i].term[0] = 0.0;
    s[i].term[1] = 0.0;
  }
}

}  // namespace

int csr_keep_entries(int dim) {
  // the MALL's 256 MiB less a margin and the vectors an iteration touches
  // (about 80 bytes per row), in 20-byte CSR entries
  const long long keep = std::max(0LL, (240LL << 20) - 80LL * dim) / 20;
  return (int)std::min<long long>(keep, 1LL << 30);
}

int csr2_fuse_grid(int rows_per_block) { return rows_per_block > kRowsDirect ? 2048 : kFuseMaxGrid; }

int csr2_grid(int dim, int rows_per_block) {
  if (rows_per_block == kStreamTile) return csr2_stream_grid(dim);
  int rows = rows_per_block < 0 ? -rows_per_block : rows_per_block;
  if (rows_per_block > kRowsDirect) rows = rows_per_block - kRowsDirect;
  else if (rows_per_block > kWaveTile) rows = (rows_per_block - kWaveTile) * (kThreads / 64);
  return (dim + rows - 1) / rows;
}

namespace {
template <int MODE, int NT>
hipError_t launch_rows(const CsrDev& t1, const CsrDev& t2, const CsrDev& t3, int dim, const IterArgs& a, double a3,
                       int rows_per_block, hipStream_t s) {
  const int grid = csr2_grid(dim, rows_per_block);
  if constexpr (NT == 3)
    if (rows_per_block == kRowsDirect + 64 && grid <= 2048) {
      csr_rows_kernel<MODE, NT, 512, 4><<<grid, 512, 0, s>>>(t1, t2, t3, dim, a, a3);
      return hipGetLastError();
    }
  if (rows_per_block == kRowsDirect + 32 && grid <= 1024)
    csr_rows_kernel<MODE, NT, 256, 4><<<grid, 256, 0, s>>>(t1, t2, t3, dim, a, a3);
  else if (rows_per_block == kRowsDirect + 32 && grid <= 2048)
    csr_rows_kernel<MODE, NT, 256, 8><<<grid, 256, 0, s>>>(t1, t2, t3, dim, a, a3);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}
}  // namespace

// Streamed tiles where the two terms are streamed (and past the direct kernel's
// largest grid), else eight lanes per row: chains of 10, 14 and 16 sites 5.3, 6.3
// and 16.7 us per iteration, against 7.5, 9.5 and 24.6 with a wave to 8 rows.
int csr3_rows(int dim, int rows_per_block) {
  if (rows_per_block == kStreamTile || dim > 131072) return kStreamTile;
  return dim > 65536 ? kRowsDirect + 64 : kRowsDirect + 32;
}

hipError_t launch_csr3_iter(const CsrDev& t1, const CsrDev& t2, const CsrDev& t3, int dim, const IterArgs& a, double a3,
                            int rows_per_block, hipStream_t s) {
  if (rows_per_block == kStreamTile) return launch_csr3_stream(t1, t2, t3, dim, a, a3, s);
  return launch_rows<kLeja, 3>(t1, t2, t3, dim, a, a3, rows_per_block, s);
}

hipError_t launch_csr2_iter(int mode, const CsrDev& t1, const CsrDev& t2, int dim, const IterArgs& a,
                            int rows_per_block, hipStream_t s) {
  if (rows_per_block == kStreamTile) return launch_csr2_stream(mode, t1, t2, dim, a, s);
  if (mode == kSplitComm) return hipErrorInvalidValue;
  const int grid = csr2_grid(dim, rows_per_block);
#define MAGNUS_CSR_CASE(R, M) \
  if (rows_per_block == R && mode == M) { csr2_iter_kernel<R, M><<<grid, kThreads, 0, s>>>(t1, t2, dim, a); return hipGetLastError(); }
  MAGNUS_CSR_CASE(64, kLeja)
  MAGNUS_CSR_CASE(64, kSplit)
  MAGNUS_CSR_CASE(64, kLejaComm)
#undef MAGNUS_CSR_CASE
#define MAGNUS_ROWLANE_CASE(R)                                                                     \
  if (rows_per_block == -R) {                                                                      \
    const int g = csr2_grid(dim, -R);                                                              \
    if (mode == kLeja) csr2_rowlane_kernel<R, kLeja><<<g, kThreads, 0, s>>>(t1, t2, dim, a);       \
    else if (mode == kSplit) csr2_rowlane_kernel<R, kSplit><<<g, kThreads, 0, s>>>(t1, t2, dim, a); \
    else csr2_rowlane_kernel<R, kLejaComm><<<g, kThreads, 0, s>>>(t1, t2, dim, a);                 \
    return hipGetLastError();                                                                      \
  }
  MAGNUS_ROWLANE_CASE(32)
  MAGNUS_ROWLANE_CASE(64)
  MAGNUS_ROWLANE_CASE(128)
#undef MAGNUS_ROWLANE_CASE
#define MAGNUS_WAVE_CASE(R)                                                                         \
  if (rows_per_block == kWaveTile + R) {                                                            \
    const int g = csr2_grid(dim, rows_per_block);                                                   \
    const int ke = csr_keep_entries(dim);                                                           \
    if (mode == kLeja) csr2_wave_kernel<R, kLeja><<<g, kThreads, 0, s>>>(t1, t2, dim, a, ke);       \
    else if (mode == kSplit) csr2_wave_kernel<R, kSplit><<<g, kThreads, 0, s>>>(t1, t2, dim, a, ke); \
    else csr2_wave_kernel<R, kLejaComm><<<g, kThreads, 0, s>>>(t1, t2, dim, a, ke);                 \
    return hipGetLastError();                                                                       \
  }
  MAGNUS_WAVE_CASE(8)
  MAGNUS_WAVE_CASE(16)
#undef MAGNUS_WAVE_CASE
  if (rows_per_block > kRowsDirect) {
    if (mode == kLeja) return launch_rows<kLeja, 2>(t1, t2, t2, dim, a, 0.0, rows_per_block, s);
    if (mode == kSplit) return launch_rows<kSplit, 2>(t1, t2, t2, dim, a, 0.0, rows_per_block, s);
    return launch_rows<kLejaComm, 2>(t1, t2, t2, dim, a, 0.0, rows_per_block, s);
  }
  return hipErrorInvalidValue;
}

int csr_gershgorin_grid(int dim) { return (dim + kThreads - 1) / kThreads; }

hipError_t launch_csr_gershgorin(const CsrDev& t, int dim, long long nnz, double* out, int grid, hipStream_t s) {
  csr_gershgorin_kernel<<<grid, kThreads, 0, s>>>(t, dim, nnz, out);
  return hipGetLastError();
}

int dense_gershgorin_grid(int dim) { return (dim + kThreads / 64 - 1) / (kThreads / 64); }

hipError_t launch_dense_gershgorin(const double2* H, int dim, long long ld, double* out, int grid,
                                   hipStream_t s) {
  dense_gershgorin_kernel<<<grid, kThreads, 0, s>>>(H, dim, ld, out);
  return hipGetLastError();
}

// Two workgroups on every CU, each with an equal share of the rows (one-term
// iteration, us, against a workgroup per 8 rows, whose number is rarely a
// multiple of the CUs': N = 4772 58.5 / 61.8, 5100 64.5 / 82.2, 8192
// 153 / 161; 640 and 1024 workgroups 63.5 and 65.3 at N = 4772); a row each
// where there are fewer rows.
constexpr int kDenseGrid = 512;
int dense2_grid(int dim) { return std::min(dim, std::max(kDenseGrid, (dim + kDenseMaxRows - 1) / kDenseMaxRows)); }

// Rows per wave at a time: one where every workgroup has one row, else 1, 2 or
// 4 (magnus_autotune times them on the caller's terms; 2 by default).

// MALL budget kept for matrix rows: its 256 MiB less a margin and the vectors
// an iteration touches (x, w and p read, w and p written).
constexpr long long kDenseMallKeepBytes = 240LL << 20;

hipError_t launch_dense_assemble_iter(const DenseAssembly& D, int dim, const IterArgs& a, hipStream_t s, int rpw) {
  const int g = dense2_grid(dim);
  if (g <= 0) return hipSuccess;
  if (g == dim) rpw = 1;
#define MAGNUS_DENSE_ASM_CASE(R)                                                        \
  case R:                                                                               \
    if (D.K) dense_assemble_iter_kernel<R, 4 / R, true><<<g, kThreads, 0, s>>>(D, dim, a);      \
    else dense_assemble_iter_kernel<R, 4 / R, false><<<g, kThreads, 0, s>>>(D, dim, a);         \
    break;
  switch (rpw) {
    MAGNUS_DENSE_ASM_CASE(1)
    MAGNUS_DENSE_ASM_CASE(2)
    MAGNUS_DENSE_ASM_CASE(4)
    default: return hipErrorInvalidValue;
  }
#undef MAGNUS_DENSE_ASM_CASE
  return hipGetLastError();
}

hipError_t launch_dense2_iter(const double2* H1, const double2* H2, int dim, long long ld,
                              const IterArgs& a, hipStream_t s, int rpw) {
  const long long row_bytes = 16LL * ld * (H2 ? 2 : 1);
  const long long keep = std::max(0LL, kDenseMallKeepBytes - 80LL * dim) / std::max(1LL, row_bytes);
  const int keep_rows = (int)std::min<long long>(keep, dim);
  const int g = dense2_grid(dim);
  if (g <= 0) return hipSuccess;
  if (g == dim) rpw = 1;
#define MAGNUS_DENSE_CASE(R)                                                             \
  case R:                                                                                \
    if (H2) dense2_iter_kernel<R, 4 / R, 2><<<g, kThreads, 0, s>>>(H1, H2, dim, ld, a, keep_rows); \
    else dense2_iter_kernel<R, R == 1 ? 4 : 8 / R, 1><<<g, kThreads, 0, s>>>(H1, H1, dim, ld, a, keep_rows);    \
    break;
  switch (rpw) {
    MAGNUS_DENSE_CASE(1)
    MAGNUS_DENSE_CASE(2)
    MAGNUS_DENSE_CASE(4)
    default: return hipErrorInvalidValue;
  }
#undef MAGNUS_DENSE_CASE
  return hipGetLastError();
}

hipError_t launch_copy(const double2* src, double2* dst, long long n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const long long grid = (n + kThreads - 1) / kThreads;
  copy_kernel<<<(unsigned)grid, kThreads, 0, s>>>(src, dst, n);
  return hipGetLastError();
}

hipError_t launch_leja_final_check(const IterArgs& a, hipStream_t s) {
  leja_final_check_kernel<<<1, kDecideThreads, 0, s>>>(a);
  return hipGetLastError();
}

hipError_t launch_leja_decide(const IterArgs& a, int grid, hipStream_t s) {
  leja_decide_kernel<<<1, kDecideThreads, 0, s>>>(a, grid);
  return hipGetLastError();
}

hipError_t launch_step_set(int* ctr, int value, hipStream_t s) {
  step_set_kernel<<<1, 1, 0, s>>>(ctr, value);
  return hipGetLastError();
}

hipError_t launch_step_advance(int* ctr, hipStream_t s) {
  step_advance_kernel<<<1, 1, 0, s>>>(ctr);
  return hipGetLastError();
}

hipError_t launch_slot_reset(Slot* slot, int n, hipStream_t s) {
  slot_reset_kernel<<<(n + 63) / 64, 64, 0, s>>>(slot, n);
  return hipGetLastError();
}

}  // namespace magnus

// The commutator K = i [H1, H2] of two CSR terms, assembled once for Method
// M4 (Section 2; Section 4 forms the M4 commutator explicitly), and the Leja
// iteration on the three-term exponent a1 H1 + a2 H2 + a3 K.
//
// Assembly: one wave per row r.  The wave lists every product of row r of
// H1 H2 (H1[r,k] H2[k,c]) and of -H2 H1 (-H2[r,k] H1[k,c]) in LDS, sorts them
// by (column, position in the list) with a bitonic network, and lane 0 sums
// equal columns in that order (deterministic), drops exact zeros and scales
// by i.  A count pass sizes the rows; a fill pass writes them.
//
// Iteration: the wave-tile mapping of the two-term kernel (8 rows per wave,
// 8 lanes per row, each tile's entries of the three terms staged in LDS
// with coalesced non-temporal loads, fixed-order shuffle sums).  Large
// matrices take the streamed three-term kernel instead (LDS-DMA copies one
// chunk ahead), which sums in the same order.
#include <climits>
#include <type_traits>

#include "device_common.h"

namespace magnus {
namespace {

using namespace dev;

constexpr int kCommWaves = 4;

__device__ __forceinline__ void comm_lds_sync() {
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
  __builtin_amdgcn_wave_barrier();
}

template <bool FILL>
__global__ __launch_bounds__(kCommWaves * 64) void csr_commutator_kernel(CsrDev A, CsrDev Bm, int dim, int* counts,
                                                                          const int* rp_out, int* ci_out,
                                                                          double2* val_out, int* overflow) {
  __shared__ long long skey[kCommWaves][kCommCap];
  __shared__ d2 sval[kCommWaves][kCommCap];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int r = blockIdx.x * kCommWaves + wv;
  if (r >= dim) return;  // whole wave; no workgroup barrier below
  const d2* av = reinterpret_cast<const d2*>(A.val);
  const d2* bv = reinterpret_cast<const d2*>(Bm.val);

  // list the products of row r: first A B, then -(B A)
  int n = 0;
  for (int side = 0; side < 2; ++side) {
    const CsrDev& L = side == 0 ? A : Bm;
    const CsrDev& R = side == 0 ? Bm : A;
    const d2* lv = side == 0 ? av : bv;
    const d2* rv = side == 0 ? bv : av;
    const double sg = side == 0 ? 1.0 : -1.0;
    for (int e = L.rp[r]; e < L.rp[r + 1]; ++e) {
      const int k = L.ci[e];
      const d2 lval = lv[e];
      const int b0 = R.rp[k], b1 = R.rp[k + 1];
      for (int j = b0 + lane; j < b1; j += 64) {
        const int idx = n + (j - b0);
        if (idx < kCommCap) {
          skey[wv][idx] = ((long long)R.ci[j] << 32) | (long long)idx;
          sval[wv][idx] = rmul(sg, cmul(lval, rv[j]));
        }
      }
      n += b1 - b0;
    }
  }
  if (n > kCommCap) {
    if (lane == 0) *overflow = 1;  // plain vector store; any writer sets the same value
    return;
  }
  int np2 = 1;
  while (np2 < n) np2 <<= 1;
  for (int i = n + lane; i < np2; i += 64) skey[wv][i] = LLONG_MAX;
  comm_lds_sync();
  // bitonic sort of skey (with sval) ascending
  for (int k = 2; k <= np2; k <<= 1)
    for (int j = k >> 1; j > 0; j >>= 1) {
      for (int i = lane; i < np2; i += 64) {
        const int p = i ^ j;
        if (p > i) {
          const bool up = (i & k) == 0;
          const long long ki = skey[wv][i], kp = skey[wv][p];
          if ((ki > kp) == up) {
            skey[wv][i] = kp;
            skey[wv][p] = ki;
            const d2 t = sval[wv][i];
            sval[wv][i] = sval[wv][p];
            sval[wv][p] = t;
          }
        }
      }
      comm_lds_sync();
    }
  if (lane != 0) return;
  int out = 0;
  const int base = FILL ? rp_out[r] : 0;
  for (int i = 0; i < n;) {
    const int c = (int)(skey[wv][i] >> 32);
    d2 s = {0.0, 0.0};
    for (; i < n && (int)(skey[wv][i] >> 32) == c; ++i) s += sval[wv][i];
    if (s.x != 0.0 || s.y != 0.0) {
      if (FILL) {
        ci_out[base + out] = c;
        val_out[base + out] = make_double2(-s.y, s.x);  // i s
      }
      ++out;
    }
  }
  if (!FILL) counts[r] = out;
}

}  // namespace

hipError_t launch_csr_commutator(bool fill, const CsrDev& A, const CsrDev& Bm, int dim, int* counts,
                                 const int* rp_out, int* ci_out, double2* val_out, int* overflow, hipStream_t s) {
  const int grid = (dim + kCommWaves - 1) / kCommWaves;
  if (fill) csr_commutator_kernel<true><<<grid, kCommWaves * 64, 0, s>>>(A, Bm, dim, counts, rp_out, ci_out, val_out, overflow);
  else csr_commutator_kernel<false><<<grid, kCommWaves * 64, 0, s>>>(A, Bm, dim, counts, rp_out, ci_out, val_out, overflow);
  return hipGetLastError();
}

}  // namespace magnus

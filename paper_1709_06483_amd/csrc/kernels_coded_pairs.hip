// Leja iterations of pairs of states on coded CSR terms (kernels_coded.hip).
//
// The states of a batch are taken two by two, a pair interleaved (element
// (row, c) at 2 row + c): one look-up of a code serves both, and a gather reads
// 32 contiguous bytes.  One launch serves every pair of up to 8 problems (a
// batch of states on one Hamiltonian, the problems of a ragged batch), each
// column with its own coefficients, degree and stop test; or pairs that are the
// block vectors (x, y) of [[H, H2], [0, H]], whose exponential carries the
// Frechet derivative of the matrix exponential.  The stop test of the
// iteration before is made by every workgroup from its pair's norm partials.
#include <algorithm>

#include "coded_device.h"

namespace magnus {
namespace {

using namespace dev;

// The dictionary with each column's coefficient applied; h2 couples column 1
// into column 0 (the second term only).
struct RealPair {
  double h0, h1, h2;
  int offset, pad;
};
struct FullPair {
  double2 h0, h1, h2;
  int offset, pad[3];
};
union PairLds {
  FullPair full[kCodeMax + 1];
  RealPair real[kCodeMax + 1];
};

template <bool FRECHET, int K, class Entry>
__device__ __forceinline__ void pair_rounds(const Entry* dict, const unsigned (&words)[2], unsigned row32,
                                            __amdgpu_buffer_rsrc_t x, d2& s0, d2& s1) {
  d2 g0[K], g1[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const unsigned at = row32 + 2u * (unsigned)dict[(words[k / 4] >> (8 * (k & 3))) & 255u].offset;
    g0[k] = buffer_at(x, at);
    g1[k] = buffer_at(x, at + 16u);
  }
  asm volatile("" ::: "memory");  // the values are read once the gathers are out
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const Entry& e = dict[(words[k / 4] >> (8 * (k & 3))) & 255u];
    s0 += code_mul(e.h0, g0[k]);
    if constexpr (FRECHET) s0 += code_mul(e.h2, g1[k]);
    s1 += code_mul(e.h1, g1[k]);
  }
}

template <bool FRECHET, class Entry>
__device__ __forceinline__ void pair_stream(const Entry* dict, const CodeWords& w, int rd, int end, unsigned row32,
                                            __amdgpu_buffer_rsrc_t x, d2& s0, d2& s1) {
  constexpr bool kWide = sizeof(Entry) == sizeof(RealPair);
#pragma unroll 1
  while (rd < end) {
    const int left = end - rd;
    unsigned words[2];
    code_window(w, rd, words);
    if (kWide && left > 2) {
      if (left < 4) words[0] &= 0xFFFFFFu;
      pair_rounds<FRECHET, 4>(dict, words, row32, x, s0, s1);
      rd += 4;
    } else if (left >= 2) {
      pair_rounds<FRECHET, 2>(dict, words, row32, x, s0, s1);
      rd += 2;
    } else {
      pair_rounds<FRECHET, 1>(dict, words, row32, x, s0, s1);
      rd += 1;
    }
  }
}

// The sums of the previous iteration's norm partials of a pair: w of both
// columns, then v of both (its first iteration only).
struct PairStop {
  double s[4][kStopLoads];
  double vnorm[2], term[2];
  int stopped[2];
};

template <bool FRECHET, int STEPS>
__global__ __launch_bounds__(kThreads, 4) void coded_pair_kernel(PairArgs A) {
  constexpr int NW = kThreads / 64;
  __shared__ PairLds dict;
  __shared__ double red[4][NW];
  __shared__ int was[2];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = lane >> 4, r = lane & 15;
  int pr = 0;
  while (pr + 1 < A.np && (int)blockIdx.x >= A.p[pr + 1].block0) ++pr;  // uniform
  const PairProblem& P = A.p[pr];
  // Eight pairs or more: an XCD takes whole pairs, so its L2 holds their vectors
  // (and no row's partner lies with another XCD); fewer: it takes a range of rows.
  const int id = (int)blockIdx.x - P.block0;
  if (id >= P.blocks * P.npairs) return;
  int pair, L;
  if (P.npairs % 8 == 0) {
    const int k = id >> 3;
    pair = (id & 7) + 8 * (k / P.blocks);
    L = k % P.blocks;
  } else {
    const int j = xcd_remap(id, P.blocks * P.npairs);
    pair = j % P.npairs;
    L = j / P.npairs;
  }
  const CodedDev& C = P.C;
  const int dim = P.dim;
  const d2* x = reinterpret_cast<const d2*>(P.x) + 2 * (long long)dim * pair;
  d2* wout = reinterpret_cast<d2*>(P.wout) + 2 * (long long)dim * pair;
  d2* pacc = reinterpret_cast<d2*>(P.pacc) + 2 * (long long)dim * pair;
  Slot* slots = P.slots + 2 * pair;
  const ColParam* prm = P.prm + 2 * pair;
  const int last_slice = (dim - 1) / 16;
  const bool check = P.iter > 1, vfirst = P.iter == 2;

  PairStop stop;
  if (check) {
    const double* pp = P.prev_partials + 4 * (long long)P.blocks * pair;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      stop.stopped[c] = load_stopped(&slots[c]);
      stop.vnorm[c] = slots[c].vnorm;
      stop.term[c] = slots[c].term[P.iter & 1];
    }
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (c < 2 || vfirst)
#pragma unroll
        for (int u = 0; u < kStopLoads; ++u) stop.s[c][u] = pp[c * P.blocks + min(u * kThreads + tid, P.blocks - 1)];
  }
  const CodeEntry ent = C.dict[(size_t)L * (kCodeMax + 1) + tid];
  const int block = C.block[L];  // -1: not coded
  const ColParam p0 = prm[0], p1 = prm[1];

  unsigned cw[kCodeAhead], head[2];
  auto load_words = [&](int slice) {
    const unsigned* cp = C.codes + ((size_t)min(slice, last_slice) * 64 + lane) * kCodeAhead;
#pragma unroll
    for (int k = 0; k < kCodeAhead; ++k) cw[k] = cp[k];
  };
  auto load_pass = [&](int row0) {
    const int own = min(row0 + (STEPS > 1 ? lane : r), dim - 1);
#pragma unroll
    for (int t = 0; t < 2; ++t) head[t] = C.head[(size_t)(own / 16) * kCodeHead + t];
    load_words(row0 / 16);
  };
  const int first_row = L * C.rows + wv * 16 * STEPS;
  load_pass(first_row);

  // the previous iteration's verdicts, the same in every workgroup of the pair
  bool done[2] = {false, false};
  if (check) {
    if (tid == 0) {
      was[0] = stop.stopped[0];
      was[1] = stop.stopped[1];
    }
    double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (c < 2 || vfirst) {
#pragma unroll
        for (int u = 0; u < kStopLoads; ++u)
          if (u * kThreads + tid < P.blocks) s[c] += stop.s[c][u];
        s[c] = wave_sum(s[c]);
        if (lane == 0) red[c][wv] = s[c];
      }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      s[c] = 0.0;
      if (c < 2 || vfirst)
        for (int k = 0; k < NW; ++k) s[c] += red[c][k];
    }
    if (FRECHET) {  // one block vector
      s[0] = s[1] = s[0] + s[1];
      s[2] = s[3] = s[2] + s[3];
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      done[c] = was[c] != 0;
      if (done[c]) continue;
      const ColParam& pc = P.prev[2 * pair + c];
      const double vn = vfirst ? sqrt(s[2 + c]) : stop.vnorm[c];
      const double prev = vfirst ? pc.d0abs * vn : stop.term[c];
      const double term = pc.dabs * sqrt(s[c]);
      const double est = term + prev;
      const bool bad = !isfinite(s[c]) || !isfinite(vn);
      done[c] = bad || (P.early && est <= P.tol * vn);
      if (L == 0 && tid == 0) {
        Slot* S = &slots[c];
        if (bad) S->status |= 1;
        if (vfirst) S->vnorm = vn;
        S->term[(P.iter - 1) & 1] = term;
        S->last_est = est;
        if (done[c]) {
          S->stopped = 1;
        } else {
          S->iters_sub = P.iter;
          S->iters_total += 1;
        }
      }
    }
    if (done[0] && done[1]) return;  // uniform over the workgroup
  } else if (L == 0 && tid == 0) {  // a substep's first iteration always runs
    for (int c = 0; c < 2; ++c) {
      slots[c].stopped = 0;
      slots[c].iters_sub = 1;
      slots[c].iters_total += 1;
    }
  }

  const bool one_real = block >= 0 && (block & kCodeOneReal);
  const bool used = block >= 0 && tid > 0 && tid <= (block & 255);
  {
    const double a0 = ent.term == 0 ? p0.a1 : p0.a2, a1 = ent.term == 0 ? p1.a1 : p1.a2;
    const double a2 = FRECHET && ent.term == 1 ? p0.coup : 0.0;
    const int off = used ? ent.offset : kNoEntry;
    if (one_real) {
      const double v = used ? (ent.val.x != 0.0 ? ent.val.x : ent.val.y) : 0.0;
      dict.real[tid] = RealPair{a0 * v, a1 * v, a2 * v, off, 0};
    } else {
      const d2 v = used ? tod2(ent.val) : d2{0.0, 0.0};
      dict.full[tid] = FullPair{fromd2(rmul(a0, v)), fromd2(rmul(a1, v)), fromd2(rmul(a2, v)), off, {0, 0, 0}};
    }
  }
  __syncthreads();

  const __amdgpu_buffer_rsrc_t buf =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<d2*>(x), 0, (int)(32u * (unsigned)dim), 0x00020000);
  double nw[2] = {0.0, 0.0}, nv[2] = {0.0, 0.0};
  const int row_end = min((L + 1) * C.rows, dim);
  for (int row0 = first_row; row0 < row_end; row0 += NW * 16 * STEPS) {
    if (row0 != first_row) load_pass(row0);
    const int own = row0 + (STEPS > 1 ? lane : r);
    const bool mine = own < dim && q < STEPS;
    const int own_ld = min(own, dim - 1);
    SliceSums<STEPS> sums[2];
    d2 w_old[2], p_old[2];
    double diag[2];
#pragma unroll 1
    for (int j = 0; j < STEPS; ++j) {
      const int row = row0 + 16 * j + r;
      CodeWords w;
#pragma unroll
      for (int k = 0; k < kCodeAhead; ++k) w.ahead[k] = cw[k];
      if (j + 1 < STEPS) {
        load_words(row0 / 16 + j + 1);
      } else {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          w_old[c] = x[2 * (long long)own_ld + c];
          p_old[c] = P.first ? d2{0.0, 0.0} : pacc[2 * (long long)own_ld + c];
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) diag[t] = C.diag[(size_t)t * C.diag_stride + own_ld];
      }
      d2 sum[2] = {{0.0, 0.0}, {0.0, 0.0}};
      if (row0 + 16 * j >= dim) {  // (uniform) no rows left
      } else if (block >= 0) {
        const int slice = row0 / 16 + j;
        const int end0 = (int)(__builtin_amdgcn_readlane(head[0], 16 * j) & 255u);
        const int end1 = (int)(__builtin_amdgcn_readlane(head[1], 16 * j) & 255u);
        const unsigned row32 = 32u * (unsigned)min(row, dim - 1);
        w.first = C.codes + ((size_t)slice * 64 + lane) * kCodeAhead;
        w.more = C.more + (size_t)slice * (kCodeMore * 64) + lane;
        w.rounds = end1;
        const bool i0 = one_real && (block & kCodeImag), i1 = one_real && (block & (kCodeImag << 1));
        int rd = 0;
#pragma unroll 1
        for (int t = 0; t < 2; ++t) {
          if (t == 0 && i0 == i1) continue;  // terms of one kind are one stream of rounds
          const int e = t == 0 ? end0 : end1;
          d2 s0 = {0.0, 0.0}, s1 = {0.0, 0.0};
          if (one_real) pair_stream<FRECHET>(dict.real, w, rd, e, row32, buf, s0, s1);
          else pair_stream<FRECHET>(dict.full, w, rd, e, row32, buf, s0, s1);
          if (t == 0 ? i0 : i1) {
            s0 = d2{-s0.y, s0.x};
            s1 = d2{-s1.y, s1.x};
          }
          sum[0] += s0;
          sum[1] += s1;
          rd = e;
        }
      } else if (row < dim) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const CsrDev& M = t == 0 ? P.t1 : P.t2;
          const d2* v = reinterpret_cast<const d2*>(M.val);
          d2 s0 = {0.0, 0.0}, s1 = {0.0, 0.0};
          const int e1 = M.rp[row + 1];
          for (int e = M.rp[row] + q; e < e1; e += 4) {
            const d2* xe = x + 2 * (long long)M.ci[e];
            s0 += cmul(v[e], xe[0]);
            s1 += cmul(v[e], xe[1]);
          }
          sum[0] += rmul(t == 0 ? p0.a1 : p0.a2, s0);
          if (FRECHET && t == 1) sum[0] += rmul(p0.coup, s1);
          sum[1] += rmul(t == 0 ? p1.a1 : p1.a2, s1);
        }
      }
      sums[0].put(j, sum[0]);
      sums[1].put(j, sum[1]);
    }
    d2 y[2] = {sums[0].total(q), sums[1].total(q)};
    if (mine) {
      if (block >= 0) {
        if (head[0] >> 8) {
          y[0] += rmul(p0.a1 * diag[0], w_old[0]);
          y[1] += rmul(p1.a1 * diag[0], w_old[1]);
        }
        if (head[1] >> 8) {
          y[0] += rmul(p0.a2 * diag[1], w_old[0]);
          if (FRECHET) y[0] += rmul(p0.coup * diag[1], w_old[1]);
          y[1] += rmul(p1.a2 * diag[1], w_old[1]);
        }
      }
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const ColParam& pc = c == 0 ? p0 : p1;
        const d2 wn = y[c] - rmul(pc.sigma, w_old[c]);
        const d2 dd = {pc.dre, pc.dim};
        d2 p = p_old[c];
        if (P.first) {
          p = cmul(d2{pc.d0re, pc.d0im}, w_old[c]) + cmul(dd, wn);
          nv[c] += nrm2(w_old[c]);
        } else if (!done[c]) {
          p += cmul(dd, wn);
        }
        wout[2 * (long long)own + c] = wn;
        pacc[2 * (long long)own + c] = p;
        nw[c] += nrm2(wn);
      }
    }
  }
  const double norms[4] = {wave_sum(nw[0]), wave_sum(nw[1]), wave_sum(nv[0]), wave_sum(nv[1])};
  __syncthreads();  // red is free again
  if (lane == 0)
    for (int c = 0; c < 4; ++c) red[c][wv] = norms[c];
  __syncthreads();
  if (tid < 4) {
    double t = 0.0;
    for (int k = 0; k < NW; ++k) t += red[tid][k];
    P.partials[4 * (long long)P.blocks * pair + tid * P.blocks + L] = t;
  }
}

// After the last iteration of a call: flag non-finite norms of the columns that
// had not stopped before it (one workgroup per pair; P.partials are its sums).
__global__ __launch_bounds__(kThreads) void coded_pair_check_kernel(PairArgs A) {
  __shared__ double red[4][kThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  int pr = 0, pair = blockIdx.x;
  while (pr + 1 < A.np && pair >= A.p[pr].npairs) pair -= A.p[pr++].npairs;  // uniform
  const PairProblem& P = A.p[pr];
  const double* pp = P.partials + 4 * (long long)P.blocks * pair;
  for (int c = 0; c < 4; ++c) {
    double s = 0.0;
    if (c < 2 || P.first)
      for (int k = tid; k < P.blocks; k += kThreads) s += pp[c * P.blocks + k];
    s = wave_sum(s);
    if (lane == 0) red[c][wv] = s;
  }
  __syncthreads();
  if (tid < 2) {
    Slot* S = P.slots + 2 * pair + tid;
    double w = 0.0, v = 0.0;
    for (int k = 0; k < kThreads / 64; ++k) {
      w += red[tid][k];
      v += red[2 + tid][k];
    }
    if (!load_stopped(S) && (!isfinite(w) || !isfinite(v))) S->status |= 1;
  }
}

__global__ void pack_pairs_kernel(const double2* __restrict__ src, double2* __restrict__ dst, int dim, int npairs) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;  // (pair, row)
  if (i >= (long long)dim * npairs) return;
  const long long pair = i / dim, row = i % dim;
  dst[2 * i] = src[2 * pair * dim + row];
  dst[2 * i + 1] = src[(2 * pair + 1) * dim + row];
}

__global__ void unpack_pairs_kernel(const double2* __restrict__ src, double2* __restrict__ dst, int dim, int npairs) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (long long)dim * npairs) return;
  const long long pair = i / dim, row = i % dim;
  dst[2 * pair * dim + row] = src[2 * i];
  dst[(2 * pair + 1) * dim + row] = src[2 * i + 1];
}

// The block vectors [0; u] and [0; v], interleaved pairs.
__global__ void frechet_pairs_init_kernel(const double2* __restrict__ u, const double2* __restrict__ v,
                                          double2* __restrict__ dst, int dim) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= dim) return;
  dst[2 * (long long)i] = make_double2(0.0, 0.0);
  dst[2 * (long long)i + 1] = u[i];
  dst[2 * ((long long)dim + i)] = make_double2(0.0, 0.0);
  dst[2 * ((long long)dim + i) + 1] = v[i];
}

}  // namespace

// A block's dictionary is read by every workgroup that takes the block, 8 KiB for
// as little as 64 rows, so blocks grow until about three workgroups to a CU are
// left, past 256 rows (where a wave takes its four slices more than once) until
// four are, and past 512 only where rows are short.  Against blocks that leave
// 2,048 workgroups, batches of 16 on 16,384 rows of 7 / 15 / 21 entries are 1.45,
// 1.45 and 1.36 times as fast, of 8 on the ring of 15 sites 1.32, of 4 on 65,535
// rows of 21 entries 1.30 times; 512 to 1,024 rows per block, 16 states on 90,001
// rows of 7 / 15 / 21 entries 1.10, 1.12 and 1.04, 8 on 200,003 rows of 31 0.88.
// A single state that is left over runs on the same blocks and wants small ones.
// So does a single pair whose rows reach over 4 MB of states, an XCD's L2, and
// more: 512 workgroups hide too little of the gathers that miss it.  Two states,
// 3 steps, 128 / 256 rows per block, chain of 17 sites 838 / 872 us, ring 773 /
// 797; columns near the rows (lattices of no power of two) gain instead, 150,001
// rows of 15 entries 494 / 477.
int code_pair_rows(int dim, int npairs, int min_rows, long long nnz, bool single_too) {
  int r = std::max(min_rows, code_rows(dim));  // (partial sums of at most kFuseMaxGrid blocks each)
  auto grow = [&](int limit, long long target) {
    while (r < limit && (long long)((dim + r - 1) / r) * npairs > target) r *= 2;
  };
  const bool reaches = npairs == 1 && dim >= 1 << 17 && (dim & (dim - 1)) == 0;  // (as flips of spins do)
  if (!single_too && !reaches) {
    grow(256, 768);
    grow(512, 1024);
    if (nnz < 16LL * dim) grow(1024, 1024);
  }
  grow(1024, 2048);
  return r;
}

hipError_t launch_coded_pairs(bool frechet, PairArgs& A, hipStream_t s) {
  if (A.np < 1 || A.np > kMaxPairProblems) return hipErrorInvalidValue;
  int blocks = 0;
  bool small = true, mid = true;  // 64 (128) rows per block in every problem: one (two) slices to a wave
  for (int q = 0; q < A.np; ++q) {
    PairProblem& P = A.p[q];
    P.blocks = (P.dim + P.C.rows - 1) / P.C.rows;
    if (P.npairs < 1 || P.blocks > kFuseMaxGrid) return hipErrorInvalidValue;
    P.block0 = blocks;
    blocks += (P.blocks * P.npairs + 7) / 8 * 8;  // whole rounds of the 8 XCDs
    small = small && P.C.rows == 64;
    mid = mid && P.C.rows <= 128;
  }
  const int steps = small ? 1 : mid ? 2 : 4;
#define MAGNUS_PAIRS(F, S) coded_pair_kernel<F, S><<<blocks, kThreads, 0, s>>>(A)
  if (frechet) {
    if (steps == 1) MAGNUS_PAIRS(true, 1);
    else if (steps == 2) MAGNUS_PAIRS(true, 2);
    else MAGNUS_PAIRS(true, 4);
  } else {
    if (steps == 1) MAGNUS_PAIRS(false, 1);
    else if (steps == 2) MAGNUS_PAIRS(false, 2);
    else MAGNUS_PAIRS(false, 4);
  }
#undef MAGNUS_PAIRS
  return hipGetLastError();
}

hipError_t launch_coded_pairs_check(const PairArgs& A, hipStream_t s) {
  int pairs = 0;
  for (int q = 0; q < A.np; ++q) pairs += A.p[q].npairs;
  coded_pair_check_kernel<<<pairs, kThreads, 0, s>>>(A);
  return hipGetLastError();
}

hipError_t launch_pack_pairs(const double2* src, double2* dst, int dim, int npairs, hipStream_t s) {
  const long long n = (long long)dim * npairs;
  pack_pairs_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(src, dst, dim, npairs);
  return hipGetLastError();
}

hipError_t launch_unpack_pairs(const double2* src, double2* dst, int dim, int npairs, hipStream_t s) {
  const long long n = (long long)dim * npairs;
  unpack_pairs_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(src, dst, dim, npairs);
  return hipGetLastError();
}

hipError_t launch_frechet_pairs_init(const double2* u, const double2* v, double2* dst, int dim, hipStream_t s) {
  frechet_pairs_init_kernel<<<(dim + 255) / 256, 256, 0, s>>>(u, v, dst, dim);
  return hipGetLastError();
}

}  // namespace magnus

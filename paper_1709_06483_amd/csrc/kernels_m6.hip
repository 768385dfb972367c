// One Leja iteration of Method M6 on CSR terms, in three passes or two.
//
// The exponent of a step is a combination of H1, H2, K = i[H1,H2], P_a = -i[H_a,K],
// U_ab = i[H_a,P_b] and R_a = -i[K,P_a], with coefficients c0..c9 in the order
// H1, H2, K, P1, P2, U11, U12, U22, R1, R2.  P_a and what is nested deeper fill
// in, so only H1, H2 and K are multiplied, in three passes over the rows:
//   pass 0: a1 = H1 w, a2 = H2 w, a3 = K w, z = c6 a1 + c7 a2;
//   pass 1: with q1 = i P1 w = H1 a3 - K a1 and q2 = i P2 w = H2 a3 - K a2,
//     v1 = c0 w - i c3 a3 + c5 q1 + c6 q2 + c8 K a3 - c5 K a1
//     v2 = c1 w - i c4 a3 + c7 q2 + c9 K a3 - c6 K a1 - c7 K a2
//     v3 = c2 w + i (c3 a1 + c4 a2) - c8 q1 - c9 q2 - c8 H1 a3 + c5 H1 a1 - c9 H2 a3 + H2 z;
//   pass 2: y = H1 v1 + H2 v2 + K v3, the Leja update and the norm partials.
// (Every nested commutator expanded into products and collected by the matrix
// that is applied last.)  Two passes over H1, H2, K, P1 and P2 read up to three
// times as many entries, and with P1 and P2 a block of rows has more distinct
// couplings than its codes can name; they are taken where the rows of P1 and P2
// are short, above all in small states, whose iteration is a chain of launches.
//
// Measured, us per iteration, two passes / three on the CSR arrays / three on coded
// terms.  Chains, n = 8 17 / 19 / 19, n = 12 26 / 22 / 20, n = 14 42 / 26 / 21, n = 16
// 122 / 58 / 30; rings, n = 12 19 / 21 / 19, n = 14 30 / 24 / 19, n = 16 72 / 56 / 29;
// long-range couplings, n = 12 23 / 22, n = 16 106 / 53.  Up to n = 16 a coded pass
// is bound by its chain of dependent loads (about 7 us of 9), the CSR passes by the
// matrix entries from the MALL (44 MB in 19 us at n = 16) and the gathers.
#include "coded_device.h"

namespace magnus {
namespace {

using namespace dev;

__device__ __forceinline__ d2 times_i(d2 v) { return d2{-v.y, v.x}; }

constexpr int m6_sums(int stage) { return stage == 0 ? 3 : stage == 1 ? 7 : 1; }
// products of pass 1, in the order of the sums
enum { kH1a1, kH1a3, kH2z, kH2a3, kKa1, kKa2, kKa3 };

// What a row needs of its own besides the products.
struct M6Own {
  d2 w, a1, a2, a3;
};

// The result of the row that lane group `part` writes (pass 0: four, pass 1: three).
__device__ __forceinline__ void m6_store_a(const M6Args& M, int part, int r, const d2 (&s)[3]) {
  const d2 out = part == 0 ? s[0] : part == 1 ? s[1] : part == 2 ? s[2] : rmul(M.c[6], s[0]) + rmul(M.c[7], s[1]);
  double2* dst = part == 0 ? M.a[0] : part == 1 ? M.a[1] : part == 2 ? M.a[2] : M.a[3];
  dst[r] = fromd2(out);
}
__device__ __forceinline__ void m6_store_b(const M6Args& M, int part, int r, const M6Own& o, const d2 (&s)[7]) {
  const double* c = M.c;
  const d2 q1 = s[kH1a3] - s[kKa1], q2 = s[kH2a3] - s[kKa2];
  d2 out;
  double2* dst;
  if (part == 0) {
    out = rmul(c[0], o.w) - times_i(rmul(c[3], o.a3)) + rmul(c[5], q1) + rmul(c[6], q2) + rmul(c[8], s[kKa3]) -
          rmul(c[5], s[kKa1]);
    dst = M.v[0];
  } else if (part == 1) {
    out = rmul(c[1], o.w) - times_i(rmul(c[4], o.a3)) + rmul(c[7], q2) + rmul(c[9], s[kKa3]) - rmul(c[6], s[kKa1]) -
          rmul(c[7], s[kKa2]);
    dst = M.v[1];
  } else {
    out = rmul(c[2], o.w) + times_i(rmul(c[3], o.a1) + rmul(c[4], o.a2)) - rmul(c[8], q1) - rmul(c[9], q2) -
          rmul(c[8], s[kH1a3]) + rmul(c[5], s[kH1a1]) - rmul(c[9], s[kH2a3]) + s[kH2z];
    dst = M.v[2];
  }
  dst[r] = fromd2(out);
}
template <int STAGE>
__device__ __forceinline__ M6Own m6_own(const M6Args& M, const IterArgs& a, int r) {
  M6Own o;
  o.w = o.a1 = o.a2 = o.a3 = d2{0.0, 0.0};
  if (STAGE < 2) o.w = tod2(a.wcur[r]);
  if (STAGE == 1) {
    o.a1 = tod2(M.a[0][r]);
    o.a2 = tod2(M.a[1][r]);
    o.a3 = tod2(M.a[2][r]);
  }
  return o;
}

// Whether this launch has nothing to do (pass 0 makes the verdict where the test is fused).
template <int STAGE>
__device__ __forceinline__ bool m6_stopped(const IterArgs& a, double* fz) {
  if (STAGE == 0) return iteration_stopped(a, fz);
  return a.check_stop && load_stopped(a.slot);
}

// ---------------------------------------------------------------------------
// On the CSR arrays: kM6Lanes lanes per row.  Consecutive passes go through the
// rows in opposite order: a pass starts on the rows the last one ended on,
// whose entries are still in the MALL.  A lane loads its row's bounds in all
// matrices before the first product, so those loads are in flight together.
// ---------------------------------------------------------------------------
constexpr int kM6Lanes = 8;

template <int NV>
__device__ __forceinline__ void m6_row(const CsrDev& T, int e, int end, const d2* const (&x)[NV], d2* sum) {
  const d2* av = reinterpret_cast<const d2*>(T.val);
#pragma unroll
  for (int k = 0; k < NV; ++k) sum[k] = d2{0.0, 0.0};
  for (; e < end; e += kM6Lanes) {
    const d2 h = av[e];
    const int c = T.ci[e];
#pragma unroll
    for (int k = 0; k < NV; ++k) sum[k] += cmul(h, x[k][c]);
  }
}

template <int STAGE>
__global__ __launch_bounds__(kThreads) void m6_kernel(CodeTerms T, int dim, M6Args M, IterArgs a) {
  __shared__ double fz[kFuseLds];
  if (m6_stopped<STAGE>(a, fz)) return;
  constexpr int NS = m6_sums(STAGE);
  const long long t = (long long)blockIdx.x * kThreads + threadIdx.x;
  const int r0 = (int)(t / kM6Lanes), q = (int)(t % kM6Lanes);
  const bool up = ((a.iter + STAGE) & 1) == 0;
  const int r = up || r0 >= dim ? r0 : dim - 1 - r0;
  d2 sum[NS];
  double pw = 0.0, pv = 0.0;
  int rs[3] = {0, 0, 0}, re[3] = {0, 0, 0};
#pragma unroll
  for (int k = 0; k < 3; ++k)
    if (r < dim) {
      rs[k] = T.m[k].rp[r];
      re[k] = T.m[k].rp[r + 1];
    }
  auto vec = [](const double2* p) { return reinterpret_cast<const d2*>(p); };
  if constexpr (STAGE == 1) {
    const d2* const h1[2] = {vec(M.a[0]), vec(M.a[2])};
    const d2* const h2[2] = {vec(M.a[3]), vec(M.a[2])};
    const d2* const k[3] = {vec(M.a[0]), vec(M.a[1]), vec(M.a[2])};
    m6_row<2>(T.m[0], rs[0] + q, re[0], h1, sum + kH1a1);
    m6_row<2>(T.m[1], rs[1] + q, re[1], h2, sum + kH2z);
    m6_row<3>(T.m[2], rs[2] + q, re[2], k, sum + kKa1);
  } else {
    d2 one[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const d2* const x[1] = {STAGE == 0 ? vec(a.wcur) : vec(M.v[k])};
      m6_row<1>(T.m[k], rs[k] + q, re[k], x, one + k);
    }
    if constexpr (STAGE == 0) {
      for (int k = 0; k < 3; ++k) sum[k] = one[k];
    } else {
      sum[0] = one[0] + one[1] + one[2];
    }
  }
#pragma unroll
  for (int k = 0; k < NS; ++k)
#pragma unroll
    for (int off = kM6Lanes / 2; off > 0; off >>= 1) {
      sum[k].x += __shfl_xor(sum[k].x, off, 64);
      sum[k].y += __shfl_xor(sum[k].y, off, 64);
    }
  if (r < dim) {
    if constexpr (STAGE == 0) {
      if (q < 4) m6_store_a(M, q, r, sum);
    } else if constexpr (STAGE == 1) {
      if (q < 3) m6_store_b(M, q, r, m6_own<1>(M, a, r), sum);
    } else {
      if (q == 0) leja_row(a, r, rmul(M.scale, sum[0]), pw, pv);
    }
  }
  if constexpr (STAGE == 2) block_partials(a, pw, pv);
}

// ---------------------------------------------------------------------------
// Two passes over H1, H2, K, P1 and P2 (the assembled P_a).  Pass 0 forms the row's five products s_k = M_k w,
//   y0 = c0 s0 + c1 s1 + c2 s2 + c3 s3 + c4 s4, u1 = i(c5 s3 + c6 s4), u2 = i c7 s4,
//   u3 = -i(c8 s3 + c9 s4), u4 = i(c8 s2 - c5 s0), u5 = i(c9 s2 - c6 s0 - c7 s1);
// pass 1: y = y0 + H1 u1 + H2 u2 + K u3 + P1 u4 + P2 u5, then the Leja update.
// ---------------------------------------------------------------------------
template <int STAGE>
__global__ __launch_bounds__(kThreads, 8) void m6_two_kernel(CodeTerms T, int dim, M6Args M, IterArgs a) {
  __shared__ double fz[kFuseLds];
  if (m6_stopped<STAGE>(a, fz)) return;
  const long long t = (long long)blockIdx.x * kThreads + threadIdx.x;
  const int r0 = (int)(t / kM6Lanes), q = (int)(t % kM6Lanes);
  const int r = STAGE == 0 || r0 >= dim ? r0 : dim - 1 - r0;  // (the second pass starts on the rows the first ended on)
  // M.a[0..3], M.v[0..1]: u1 .. u5 and y0
  double2* const u[6] = {M.a[0], M.a[1], M.a[2], M.a[3], M.v[0], M.v[1]};
  int rs[5], re[5];
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    rs[k] = r < dim ? T.m[k].rp[r] : 0;
    re[k] = r < dim ? T.m[k].rp[r + 1] : 0;
  }
  auto row_sum = [](d2 v) {  // over the row's lanes, in all of them
#pragma unroll
    for (int off = kM6Lanes / 2; off > 0; off >>= 1) {
      v.x += __shfl_xor(v.x, off, 64);
      v.y += __shfl_xor(v.y, off, 64);
    }
    return v;
  };
  d2 s[5], acc = {0.0, 0.0};
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    const d2* val = reinterpret_cast<const d2*>(T.m[k].val);
    const d2* x = reinterpret_cast<const d2*>(STAGE == 0 ? a.wcur : u[k]);
    if (STAGE == 0) acc = d2{0.0, 0.0};
    for (int e = rs[k] + q; e < re[k]; e += kM6Lanes) acc += cmul(val[e], x[T.m[k].ci[e]]);
    if (STAGE == 0) s[k] = row_sum(acc);
  }
  if constexpr (STAGE == 0) {
    if (r >= dim || q >= 6) return;
    const double* c = M.c;  // lane q of the row writes vector q
    d2 out;
    switch (q) {
      case 0: out = times_i(rmul(c[5], s[3]) + rmul(c[6], s[4])); break;
      case 1: out = times_i(rmul(c[7], s[4])); break;
      case 2: out = times_i(rmul(-c[8], s[3]) - rmul(c[9], s[4])); break;
      case 3: out = times_i(rmul(c[8], s[2]) - rmul(c[5], s[0])); break;
      case 4: out = times_i(rmul(c[9], s[2]) - rmul(c[6], s[0]) - rmul(c[7], s[1])); break;
      default: out = rmul(c[0], s[0]) + rmul(c[1], s[1]) + rmul(c[2], s[2]) + rmul(c[3], s[3]) + rmul(c[4], s[4]);
    }
    double2* dst = u[0];
#pragma unroll
    for (int k = 1; k < 6; ++k) dst = q == k ? u[k] : dst;
    dst[r] = fromd2(out);
  } else {
    acc = row_sum(acc);
    double pw = 0.0, pv = 0.0;
    if (r < dim && q == 0) leja_row(a, r, rmul(M.scale, tod2(u[5][r]) + acc), pw, pv);
    block_partials(a, pw, pv);
  }
}

// ---------------------------------------------------------------------------
// On coded terms (H1, H2, K): a wave takes a slice of 16 rows, lane 16 q + r
// quarter q of row r's entries, as in the other coded iterations.
// ---------------------------------------------------------------------------
// Products of rounds [rd, end) with NV vectors, four rounds at a time (two
// where values are complex, whose registers would spill), all their gathers
// issued before the first product (codes past the end are 0: no entry, no access).
template <int NV, class Entry>
__device__ __forceinline__ void m6_stream(const Entry* dict, const CodeWords& w, int rd, int end, unsigned row16,
                                          const __amdgpu_buffer_rsrc_t (&x)[NV], d2* sum) {
  constexpr int U = sizeof(Entry) == sizeof(RealEntry) ? 4 : 2;
#pragma unroll
  for (int k = 0; k < NV; ++k) sum[k] = d2{0.0, 0.0};
#pragma unroll 1
  for (; rd < end; rd += U) {
    unsigned words[2];
    code_window(w, rd, words);
    unsigned c = words[0];
    if (end - rd < U) c &= (1u << (8 * (end - rd))) - 1u;
    d2 g[U][NV];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const unsigned at = row16 + (unsigned)dict[(c >> (8 * u)) & 255u].offset;
#pragma unroll
      for (int k = 0; k < NV; ++k) g[u][k] = buffer_at(x[k], at);
    }
    asm volatile("" ::: "memory");
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const auto h = dict[(c >> (8 * u)) & 255u].val;
#pragma unroll
      for (int k = 0; k < NV; ++k) sum[k] += code_mul(h, g[u][k]);
    }
  }
}

template <int NV>
__device__ __forceinline__ void m6_plain(const CsrDev& T, int row, int dim, int q, const d2* const (&x)[NV], d2* sum) {
#pragma unroll
  for (int k = 0; k < NV; ++k) sum[k] = plain_row(T, row, dim, q, x[k]);
}

template <int STAGE>
__global__ __launch_bounds__(kThreads, 4) void coded_m6_kernel(CodeTerms T, int dim, CodedDev C, M6Args M, IterArgs a) {
  constexpr int NS = m6_sums(STAGE);
  __shared__ DictLds dict;
  __shared__ double fz[kFuseLds];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int L = xcd_remap(blockIdx.x, gridDim.x);
  const int q = lane >> 4, rl = lane & 15;
  const int last_slice = (dim - 1) / 16;

  // everything that needs no other load's result, together
  StopLoads<> stop;
  int stopped = 0;
  if (STAGE == 0) stop_loads(a, stop);
  else if (a.check_stop) stopped = load_stopped(a.slot);
  static_assert(kThreads > kCodeMax, "a thread per dictionary entry");
  const CodeEntry& ent = C.dict[(size_t)L * (kCodeMax + 1) + (tid & kCodeMax)];
  const d2 ent_val = tod2(ent.val);
  const int ent_off = ent.offset;
  const int block = C.block[L];  // -1: not coded
  CodeWords w;
  unsigned head[3];
  double diag[3];
  M6Own own;
  d2 x2[3];  // pass 2: the row's own v1, v2, v3; pass 1: its z
  auto load_slice = [&](int row0) {
    const int slice = min(row0 / 16, last_slice), row = min(row0 + rl, dim - 1);
    w.first = C.codes + ((size_t)slice * 64 + lane) * kCodeAhead;
    w.more = C.more + (size_t)slice * (kCodeMore * 64) + lane;
#pragma unroll
    for (int k = 0; k < kCodeAhead; ++k) w.ahead[k] = w.first[k];
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      head[t] = C.head[(size_t)slice * kCodeHead + t];
      diag[t] = C.diag[(size_t)t * C.diag_stride + row];
    }
    own = m6_own<STAGE>(M, a, row);
    if (STAGE == 1) x2[0] = tod2(M.a[3][row]);
    if (STAGE == 2)
#pragma unroll
      for (int t = 0; t < 3; ++t) x2[t] = tod2(M.v[t][row]);
  };
  const int first = L * C.rows + wv * 16;
  load_slice(first);
  if (STAGE == 0) {
    if (stop_verdict(a, stop, fz)) return;
  } else if (stopped) {
    return;
  }
  const bool one_real = block >= 0 && (block & kCodeOneReal);
  const bool used = block >= 0 && tid > 0 && tid <= (block & 255);
  if (tid > kCodeMax) {
  } else if (one_real) {
    dict.real[tid].val = used ? (ent_val.x != 0.0 ? ent_val.x : ent_val.y) : 0.0;
    dict.real[tid].offset = used ? ent_off : kNoEntry;
  } else {
    dict.full[tid].val = used ? fromd2(ent_val) : make_double2(0.0, 0.0);
    dict.full[tid].offset = used ? ent_off : kNoEntry;
  }
  __syncthreads();

  double pw = 0.0, pv = 0.0;
  const int row_end = min((L + 1) * C.rows, dim);
  for (int row0 = first; row0 < row_end; row0 += kThreads / 4) {
    if (row0 != first) load_slice(row0);
    const int row = row0 + rl;
    const unsigned row16 = 16u * (unsigned)min(row, dim - 1);
    d2 sum[NS];
    if (block >= 0) {
      int end[3];
#pragma unroll
      for (int t = 0; t < 3; ++t) end[t] = (int)(__builtin_amdgcn_readfirstlane(head[t]) & 255u);
      w.rounds = end[2];
      auto turned = [&](int t, d2 y) { return one_real && (block & (kCodeImag << t)) ? times_i(y) : y; };
      auto buf = [&](const double2* p) { return state_buffer(reinterpret_cast<const d2*>(p), dim); };
      auto stream1 = [&](int rd, int e, const double2* p) {
        const __amdgpu_buffer_rsrc_t x = buf(p);
        return one_real ? code_stream(dict.real, w, rd, e, row16, x) : code_stream(dict.full, w, rd, e, row16, x);
      };
      if constexpr (STAGE == 1) {
#pragma unroll 1
        for (int t = 0; t < 2; ++t) {
          const __amdgpu_buffer_rsrc_t x[2] = {buf(t == 0 ? M.a[0] : M.a[3]), buf(M.a[2])};
          d2 y[2];
          if (one_real) m6_stream<2>(dict.real, w, t == 0 ? 0 : end[0], t == 0 ? end[0] : end[1], row16, x, y);
          else m6_stream<2>(dict.full, w, t == 0 ? 0 : end[0], t == 0 ? end[0] : end[1], row16, x, y);
          if (t == 0) {
            sum[kH1a1] = turned(0, y[0]);
            sum[kH1a3] = turned(0, y[1]);
          } else {
            sum[kH2z] = turned(1, y[0]);
            sum[kH2a3] = turned(1, y[1]);
          }
        }
        const __amdgpu_buffer_rsrc_t x[3] = {buf(M.a[0]), buf(M.a[1]), buf(M.a[2])};
        d2 y[3];
        if (one_real) m6_stream<3>(dict.real, w, end[1], end[2], row16, x, y);
        else m6_stream<3>(dict.full, w, end[1], end[2], row16, x, y);
        for (int k = 0; k < 3; ++k) sum[kKa1 + k] = turned(2, y[k]);
      } else {
        d2 total = {0.0, 0.0};
#pragma unroll 1
        for (int t = 0; t < 3; ++t) {
          const int rd = t == 0 ? 0 : t == 1 ? end[0] : end[1], e = t == 0 ? end[0] : t == 1 ? end[1] : end[2];
          const double2* p = STAGE == 0 ? a.wcur : t == 0 ? M.v[0] : t == 1 ? M.v[1] : M.v[2];
          const d2 y = turned(t, stream1(rd, e, p));
          if constexpr (STAGE == 0) {
            if (t == 0) sum[0] = y;
            else if (t == 1) sum[1] = y;
            else sum[2] = y;
          } else {
            total += y;
          }
        }
        if constexpr (STAGE == 2) sum[0] = total;
      }
    } else {
      auto vec = [](const double2* p) { return reinterpret_cast<const d2*>(p); };
      if constexpr (STAGE == 0) {
        for (int t = 0; t < 3; ++t) sum[t] = plain_row(T.m[t], row, dim, q, vec(a.wcur));
      } else if constexpr (STAGE == 1) {
        const d2* const h1[2] = {vec(M.a[0]), vec(M.a[2])};
        const d2* const h2[2] = {vec(M.a[3]), vec(M.a[2])};
        const d2* const k[3] = {vec(M.a[0]), vec(M.a[1]), vec(M.a[2])};
        m6_plain<2>(T.m[0], row, dim, q, h1, sum + kH1a1);
        m6_plain<2>(T.m[1], row, dim, q, h2, sum + kH2z);
        m6_plain<3>(T.m[2], row, dim, q, k, sum + kKa1);
      } else {
        sum[0] = d2{0.0, 0.0};
        for (int t = 0; t < 3; ++t) sum[0] += plain_row(T.m[t], row, dim, q, vec(M.v[t]));
      }
    }
#pragma unroll
    for (int k = 0; k < NS; ++k)
#pragma unroll
      for (int off = 32; off >= 16; off >>= 1) {
        sum[k].x += __shfl_xor(sum[k].x, off, 64);
        sum[k].y += __shfl_xor(sum[k].y, off, 64);
      }
    if (block >= 0) {
      double d[3];
#pragma unroll
      for (int t = 0; t < 3; ++t) d[t] = diag[t];
      const bool has[3] = {(head[0] >> 8) != 0, (head[1] >> 8) != 0, (head[2] >> 8) != 0};
      if constexpr (STAGE == 0) {
        for (int t = 0; t < 3; ++t)
          if (has[t]) sum[t] += rmul(d[t], own.w);
      } else if constexpr (STAGE == 1) {
        if (has[0]) {
          sum[kH1a1] += rmul(d[0], own.a1);
          sum[kH1a3] += rmul(d[0], own.a3);
        }
        if (has[1]) {
          sum[kH2z] += rmul(d[1], x2[0]);
          sum[kH2a3] += rmul(d[1], own.a3);
        }
        if (has[2]) {
          sum[kKa1] += rmul(d[2], own.a1);
          sum[kKa2] += rmul(d[2], own.a2);
          sum[kKa3] += rmul(d[2], own.a3);
        }
      } else {
        for (int t = 0; t < 3; ++t)
          if (has[t]) sum[0] += rmul(d[t], x2[t]);
      }
    }
    if (row < dim) {
      if constexpr (STAGE == 0) {
        m6_store_a(M, q, row, sum);
      } else if constexpr (STAGE == 1) {
        if (q < 3) m6_store_b(M, q, row, own, sum);
      } else {
        if (q == 0) leja_row(a, row, rmul(M.scale, sum[0]), pw, pv);
      }
    }
  }
  if constexpr (STAGE == 2) block_partials(a, pw, pv);
}

}  // namespace

int m6_grid(int dim) { return (int)(((long long)dim * kM6Lanes + kThreads - 1) / kThreads); }

hipError_t launch_m6(int stage, const CodeTerms& T, int dim, const M6Args& M, const IterArgs& a, hipStream_t s) {
  if (dim <= 0) return hipSuccess;
  if (T.n != 3) return hipErrorInvalidValue;
  const int g = m6_grid(dim);
  if (stage == 0) m6_kernel<0><<<g, kThreads, 0, s>>>(T, dim, M, a);
  else if (stage == 1) m6_kernel<1><<<g, kThreads, 0, s>>>(T, dim, M, a);
  else m6_kernel<2><<<g, kThreads, 0, s>>>(T, dim, M, a);
  return hipGetLastError();
}

hipError_t launch_m6_two(int stage, const CodeTerms& T, int dim, const M6Args& M, const IterArgs& a, hipStream_t s) {
  if (dim <= 0) return hipSuccess;
  if (T.n != 5) return hipErrorInvalidValue;
  const int g = m6_grid(dim);
  if (stage == 0) m6_two_kernel<0><<<g, kThreads, 0, s>>>(T, dim, M, a);
  else m6_two_kernel<1><<<g, kThreads, 0, s>>>(T, dim, M, a);
  return hipGetLastError();
}

hipError_t launch_coded_m6(int stage, const CodeTerms& T, int dim, const CodedDev& C, const M6Args& M,
                           const IterArgs& a, hipStream_t s) {
  if (dim <= 0) return hipSuccess;
  if (T.n != 3) return hipErrorInvalidValue;
  const int g = code_grid(dim, C.rows);
  if (stage == 0) coded_m6_kernel<0><<<g, kThreads, 0, s>>>(T, dim, C, M, a);
  else if (stage == 1) coded_m6_kernel<1><<<g, kThreads, 0, s>>>(T, dim, C, M, a);
  else coded_m6_kernel<2><<<g, kThreads, 0, s>>>(T, dim, C, M, a);
  return hipGetLastError();
}

}  // namespace magnus

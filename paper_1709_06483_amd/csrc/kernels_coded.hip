// CSR Leja iteration on coded terms.
//
// A Hamiltonian of a lattice or spin system repeats a few couplings: in the
// rows of one block the triples (term, column - row, value) take a few dozen
// distinct values although the block holds tens of thousands of entries.  Once
// per call the terms are rewritten in that form (code_build_kernel): per block
// of rows a dictionary of at most 255 of them, and per off-diagonal entry one
// byte; real diagonals are kept apart, 8 bytes a row.  An iteration then reads
// about one byte per entry instead of 20.  The dictionary holds the entries'
// own doubles; a block that does not fit the form (more than 255 triples, more
// than 128 entries in a row, two diagonal entries of a term in a row, a diagonal
// entry with an imaginary part) is marked and read from the CSR arrays by the
// same kernel.  Nothing is kept between calls: each codes its terms as they are.
//
// Measured, Cf4 on spin chains, a call's time over its iterations, us, with the
// CSR mapping that each size takes by default / coded (and the coding, once per
// call): n = 14 6.0 / 5.8 (15), n = 15 7.4 / 6.5, n = 16 14.9 / 8.1 (22),
// n = 17 22.9 / 9.9 (36), n = 18 35 / 15 (53), n = 20 152 / 45 (194).  At n = 20 an
// iteration moves 243 MB past the L2s (counted; 847 streamed from the CSR arrays);
// what bounds it there is the latency of the gathers that leave the L2, at four
// waves per SIMD.  Measured slower: non-temporal loads and stores of the operands used
// once (48 us; they give up the MALL), 2,048 workgroups (47), a row to a lane
// (52), all code paths unrolled by the number of rounds (code of 28 KB, fetched
// cold by every launch: the three-term iteration at n = 14 20 us, 6.4 now).
#include <type_traits>

#include "coded_device.h"

namespace magnus {
namespace {

using namespace dev;

// Hash slots of a block's dictionary (at most 255 used): so few are taken that
// nearly every key lies in the slot of its hash or in the next one.
constexpr int kHash = 1024;
constexpr int kBW = kThreads / 64;
constexpr int kRoundBytes = 64;  // a round: one entry of each of a row's four lanes, 16 rows

// The dictionary of a block while it is built: a slot's key and its code (0:
// free, -1: being written).  A key equal to the one looked for has been written
// whole, in whatever order its parts are read: free slots hold a place (0) and
// parts (kNoValue, a NaN) that no entry has (a block with such a value is not coded).
constexpr long long kNoValue = 0x7FF8A5C3D00DFEEDll;
struct DictKey {
  long long re, im;
};
struct DictTag {
  int where, code;  // where: (column - row) * 8 + term
};
struct BuildLds {
  DictKey key[kHash];
  DictTag tag[kHash];
  int n, bad;
  int mixed;   // bit 2 t: a value of term t has a real part, bit 2 t + 1: an imaginary part
  unsigned tile[kBW][kCodeRounds * kRoundBytes / 4];
  double diag[kBW][16];
};

__device__ __forceinline__ unsigned code_hash(int where, long long re, long long im) {
  const unsigned rh = (unsigned)(re >> 32), ih = (unsigned)(im >> 32);
  const unsigned v = ((rh << 7 | rh >> 25) ^ (unsigned)re) + ((ih << 19 | ih >> 13) ^ (unsigned)im);
  return ((unsigned)where + v) * 0x9E3779B1u >> 22;
}
static_assert(kHash == 1 << 10, "code_hash returns ten bits");

__device__ __forceinline__ bool code_bad(BuildLds& S) {
  return __hip_atomic_load(&S.bad, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) != 0;
}
__device__ __forceinline__ void code_set_bad(BuildLds& S) {
  __hip_atomic_store(&S.bad, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// The codes of the lanes' keys (lanes with want), inserting those that are
// missing.  A lane that meets a free slot claims it, writes the key and its
// code before the loop goes round; one that meets a slot being written by
// another wave, which runs on by itself, looks again.  So every round trip of
// the loop settles a lane or lets another wave settle one; the bound on them
// only guards against a mistake.
__device__ __forceinline__ int code_get(BuildLds& S, bool want, int where, long long re, long long im) {
  unsigned h = code_hash(where, re, im);
  int found = 0;
  for (int t = 0; t < (1 << 20); ++t) {
    if (!__any(want && found == 0)) return found;
    if (code_bad(S)) return 0;
    if (want && found == 0) {
      const int c = __hip_atomic_load(&S.tag[h].code, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
      if (c > 0 && S.tag[h].where == where && S.key[h].re == re && S.key[h].im == im) {
        found = c;
      } else if (c > 0) {
        h = (h + 1) & (kHash - 1);
      } else if (c == 0) {
        int expected = 0;
        if (__hip_atomic_compare_exchange_strong(&S.tag[h].code, &expected, -1, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_WORKGROUP)) {
          const int mine = __hip_atomic_fetch_add(&S.n, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) + 1;
          S.key[h].re = re;
          S.key[h].im = im;
          S.tag[h].where = where;
          if (mine > kCodeMax) code_set_bad(S);
          else __hip_atomic_store(&S.tag[h].code, mine, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
          found = mine;
        }
      }
    }
  }
  code_set_bad(S);
  return 0;
}

// One workgroup per block of rows; a wave codes one slice of 16 rows at a time,
// term by term, four lanes to a row (so loads are runs of consecutive entries),
// the codes collected in LDS in the order the iteration reads them.  A batch is
// 4 U entries of each row; the next batch (of the same term or the next) is
// loaded while one is coded.
template <int NT>
__global__ __launch_bounds__(kThreads, 4) void code_build_kernel(CodeTerms T, int dim, CodedDev C, int* bad_blocks,
                                                                  const double* flags, int nflags) {
  __shared__ BuildLds S;
  const int tid = threadIdx.x, lane = tid & 63;
  if (nflags > 0) {  // (uniform)
    int malformed = 0;
    for (int k = tid; k < nflags; k += kThreads) malformed |= flags[3 * k + 2] != 0.0;
    if (__syncthreads_or(malformed)) {
      if (tid == 0) {
        C.block[xcd_remap(blockIdx.x, gridDim.x)] = -1;
        if (bad_blocks) atomicAdd(bad_blocks, 1);
      }
      return;
    }
  }
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int L = xcd_remap(blockIdx.x, gridDim.x);
  CodeEntry* dict = C.dict + (size_t)L * (kCodeMax + 1);
  for (int k = tid; k < kHash; k += kThreads) {
    S.key[k] = DictKey{kNoValue, kNoValue};
    S.tag[k] = DictTag{0, 0};
  }
  if (tid == 0) {
    S.n = 0;
    S.bad = 0;
    S.mixed = 0;
  }
  __syncthreads();
  constexpr int U = 4;
  const int rl = lane >> 2, q = lane & 3;
  unsigned char* bytes = reinterpret_cast<unsigned char*>(&S.tile[wv][0]);
  for (int sb = wv; sb < C.rows / 16; sb += kBW) {
    const int slice = L * (C.rows / 16) + sb;
    const int row0 = slice * 16;
    if (row0 >= dim || code_bad(S)) break;
    const int row = row0 + rl;
    int st[NT], len[NT], most[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      st[t] = len[t] = 0;
      if (row < dim) {
        st[t] = T.m[t].rp[row];
        len[t] = T.m[t].rp[row + 1];
      }
    }
    for (int k = lane; k < kCodeRounds * kRoundBytes / 4; k += 64) S.tile[wv][k] = 0;
    if (lane < 16) S.diag[wv][lane] = 0.0;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      len[t] -= st[t];
      int m = len[t];
#pragma unroll
      for (int off = 32; off >= 4; off >>= 1) m = max(m, __shfl_xor(m, off, 64));
      most[t] = __builtin_amdgcn_readfirstlane(m);
    }
    int ncol[U];
    d2 nv[U];
    auto load = [&](const CsrDev& M, int s, int l, int p0) {
      const d2* val = reinterpret_cast<const d2*>(M.val);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int pos = p0 + 4 * u + q;
        ncol[u] = 0;
        nv[u] = d2{0.0, 0.0};
        if (pos < l) {
          ncol[u] = M.ci[s + pos];
          nv[u] = val[s + pos];
        }
      }
    };
    int r0 = 0;  // rounds of the terms done
    bool fail = false;
    load(T.m[0], st[0], len[0], 0);
    wave_lds_sync();
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int l = len[t], m = most[t];
      if (r0 + ((m + 3) >> 2) > kCodeRounds) fail = true;
      if (__any(fail)) break;
      bool seen = false;  // the row's diagonal entry has been met
      bool has_re = false, has_im = false;
      int p0 = 0;
      do {
      int col[U];
      d2 v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        col[u] = ncol[u];
        v[u] = nv[u];
      }
      if (p0 + 4 * U < m) load(T.m[t], st[t], l, p0 + 4 * U);
      else if (t + 1 < NT) load(T.m[t + 1 < NT ? t + 1 : t], st[t + 1 < NT ? t + 1 : t], len[t + 1 < NT ? t + 1 : t], 0);
      int c[U];
      bool want[U];
      asm volatile("" ::: "memory");  // the dictionary grows as other waves insert
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int delta = col[u] - row;
        want[u] = p0 + 4 * u + q < l && delta != 0;
        const long long re = __double_as_longlong(v[u].x), im = __double_as_longlong(v[u].y);
        if (want[u] && (re == kNoValue || im == kNoValue)) fail = true;
        const int where = delta * 8 + t;
        const unsigned h = code_hash(where, re, im);
        const DictTag tag = S.tag[h];
        const DictKey key = S.key[h];
        c[u] = want[u] && tag.where == where && key.re == re && key.im == im ? max(tag.code, 0) : 0;
        if (__any(want[u] && c[u] == 0)) {
          const unsigned h2 = (h + 1) & (kHash - 1);
          const DictTag tag2 = S.tag[h2];
          const DictKey key2 = S.key[h2];
          if (want[u] && c[u] == 0 && tag2.where == where && key2.re == re && key2.im == im) c[u] = max(tag2.code, 0);
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (p0 + 4 * u >= m) break;  // uniform
        const int pos = p0 + 4 * u + q;
        const int delta = col[u] - row;
        const bool is_diag = pos < l && delta == 0;
        const unsigned dm = (unsigned)(__ballot(is_diag) >> (lane & ~3)) & 0xfu;
        const int slot = pos - ((seen || (dm & ((1u << q) - 1u))) ? 1 : 0);
        if (__popc(dm) + (seen ? 1 : 0) > 1) fail = true;
        seen = seen || dm != 0;
        if (is_diag) {
          if (v[u].y != 0.0) fail = true;
          S.diag[wv][rl] = v[u].x;
        }
        const long long re = __double_as_longlong(v[u].x), im = __double_as_longlong(v[u].y);
        if (__any(want[u] && c[u] == 0)) {
          const int got = code_get(S, want[u] && c[u] == 0, delta * 8 + t, re, im);
          if (want[u] && c[u] == 0) c[u] = got;
        }
        has_re = has_re || (want[u] && v[u].x != 0.0);
        has_im = has_im || (want[u] && v[u].y != 0.0);
        // round slot / 4 of the term, lane quarter slot % 4: byte round % 4 of word 16 quarter + row
        const int rd = r0 + (slot >> 2);
        if (want[u]) bytes[((rd >> 2) * 64 + (slot & 3) * 16 + rl) * 4 + (rd & 3)] = (unsigned char)c[u];
      }
      p0 += 4 * U;
      } while (p0 < m);
      int top = l - (seen ? 1 : 0);  // the slice's longest row
#pragma unroll
      for (int off = 32; off >= 4; off >>= 1) top = max(top, __shfl_xor(top, off, 64));
      r0 += (__builtin_amdgcn_readfirstlane(top) + 3) >> 2;
      const bool any = __any(seen);
      wave_lds_sync();
      if (any && lane < 16) {
        if (row0 + lane < dim) C.diag[(size_t)t * C.diag_stride + row0 + lane] = S.diag[wv][lane];
        S.diag[wv][lane] = 0.0;
      }
      const int parts = (__any(has_re) ? 1 : 0) | (__any(has_im) ? 2 : 0);
      if (lane == 0) {
        C.head[(size_t)slice * kCodeHead + t] = (unsigned)r0 | (any ? 1u << 8 : 0u);
        __hip_atomic_fetch_or(&S.mixed, parts << (2 * t), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
      wave_lds_sync();
    }
    if (__any(fail)) code_set_bad(S);
    if (code_bad(S)) break;
    wave_lds_sync();
    // (the iteration reads kCodeAhead words whatever the rounds: the tile is zero past them)
    struct Ahead {
      unsigned w[kCodeAhead];
    } first;
#pragma unroll
    for (int g = 0; g < kCodeAhead; ++g) first.w[g] = S.tile[wv][g * 64 + lane];
    reinterpret_cast<Ahead*>(C.codes)[(size_t)slice * 64 + lane] = first;
    for (int g = kCodeAhead; 4 * g < r0; ++g)
      C.more[((size_t)slice * kCodeMore + (g - kCodeAhead)) * 64 + lane] = S.tile[wv][g * 64 + lane];
    wave_lds_sync();  // the tile is free for the next slice
  }
  __syncthreads();
  for (int k = tid; k < kHash; k += kThreads) {
    const int c = S.tag[k].code;
    if (c > 0 && c <= kCodeMax) {
      dict[c].val = make_double2(__longlong_as_double(S.key[k].re), __longlong_as_double(S.key[k].im));
      dict[c].offset = (S.tag[k].where >> 3) * 16;
      dict[c].term = S.tag[k].where & 7;
    }
  }
  if (tid == 0) {
    dict[0].val = make_double2(0.0, 0.0);
    dict[0].offset = kNoEntry;
    dict[0].term = 0;
    // a term whose values are all real or all imaginary needs one number per value
    int flags = kCodeOneReal;
    for (int t = 0; t < NT; ++t) {
      const int parts = S.mixed >> (2 * t) & 3;
      if (parts == 3) flags &= ~kCodeOneReal;
      if (parts == 2) flags |= kCodeImag << t;
    }
    C.block[L] = S.bad ? -1 : S.n | flags;
    if (S.bad && bad_blocks) atomicAdd(bad_blocks, 1);
  }
}

// MODE kLeja: y = a1 H1 x1 + a2 H2 x2 (+ a3 K x1 with NT = 3), then the Leja
// update; kSplitComm as in the streamed kernel.  A wave takes STEPS slices of
// 16 rows at a time, four lanes to a row (lane = 16 q + r; lane q takes the
// entries q, q + 4, ... of each term, one a round), so a gather instruction
// reads four runs of 16 neighbouring rows; a row's four sums are combined in a
// fixed order, and lane 16 j + r makes the update of row r of slice j.
//
// What bounds it up to about 2^18 rows is the chain of dependent loads, each a
// round trip to memory that the previous launch or another XCD wrote: so
// everything that needs no other load's result (codes, ends of the terms'
// rounds, own-row operands, dictionary, the stop test's inputs) is loaded
// together first, and a slice's gathers are all issued before the first product.
template <int MODE, int NT, int STEPS, int THREADS>
__global__ __launch_bounds__(THREADS, 4) void coded_iter_kernel(CodeTerms T, int dim, CodedDev C, IterArgs a_in,
                                                                double a3_arg) {
  const IterArgs a = resolve_args(a_in);
  const double a3 = a_in.coef ? a.kap : a3_arg;
  constexpr int NW = THREADS / 64;
  __shared__ DictLds dict;
  __shared__ double red[2][NW];
  __shared__ double fz[kFuseLds];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int L = xcd_remap(blockIdx.x, gridDim.x);
  const int q = lane >> 4, r = lane & 15;
  const d2* xs[3] = {reinterpret_cast<const d2*>(a.x1), reinterpret_cast<const d2*>(a.x2),
                     reinterpret_cast<const d2*>(a.x1)};
  const int last_slice = (dim - 1) / 16;

  StopLoads<> stop;
  stop_loads(a, stop);
  static_assert(THREADS > kCodeMax, "a thread per dictionary entry");
  const d2 ent_val = tod2(C.dict[(size_t)L * (kCodeMax + 1) + (tid & kCodeMax)].val);
  const int ent_off = C.dict[(size_t)L * (kCodeMax + 1) + (tid & kCodeMax)].offset;
  const int ent_term = C.dict[(size_t)L * (kCodeMax + 1) + (tid & kCodeMax)].term;
  const int block = C.block[L];  // -1: not coded

  // what a pass of the wave needs (rows and slices past the end read the last ones)
  d2 w_old, p_old = {0.0, 0.0};
  double diag[NT];
  unsigned head[NT];  // of the lane's own slice: the term's rounds end at head & 255, bit 8: a diagonal
  unsigned cw[kCodeAhead];  // of the slice that comes next
  auto load_words = [&](int slice) {
    const unsigned* cp = C.codes + ((size_t)min(slice, last_slice) * 64 + lane) * kCodeAhead;
#pragma unroll
    for (int k = 0; k < kCodeAhead; ++k) cw[k] = cp[k];
  };
  auto load_own = [&](int row0) {
    const int own = min(row0 + (STEPS > 1 ? lane : r), dim - 1);
    w_old = tod2(a.wcur[own]);
    if (MODE == kLeja && !a.first) p_old = tod2(a.pacc[own]);
#pragma unroll
    for (int t = 0; t < NT; ++t) diag[t] = C.diag[(size_t)t * C.diag_stride + own];
  };
  auto load_pass = [&](int row0) {
    const int own = min(row0 + (STEPS > 1 ? lane : r), dim - 1);
#pragma unroll
    for (int t = 0; t < NT; ++t) head[t] = C.head[(size_t)(own / 16) * kCodeHead + t];
    load_words(row0 / 16);
    if (STEPS == 1) load_own(row0);  // (else before the last slice: held through all of them they cost waves)
  };
  const int first = L * C.rows + wv * 16 * STEPS;
  load_pass(first);
  if (stop_verdict(a, stop, fz)) return;
  const bool one_real = block >= 0 && (block & kCodeOneReal);
  const bool used = block >= 0 && tid > 0 && tid <= (block & 255);
  const int off = used ? ent_off : kNoEntry;
  const double coef = MODE == kSplitComm ? 1.0 : ent_term == 0 ? a.a1 : ent_term == 1 ? a.a2 : a3;
  if (tid > kCodeMax) {
  } else if (one_real) {
    dict.real[tid].val = used ? coef * (ent_val.x != 0.0 ? ent_val.x : ent_val.y) : 0.0;
    dict.real[tid].offset = off;
  } else {
    dict.full[tid].val = used ? fromd2(rmul(coef, ent_val)) : make_double2(0.0, 0.0);
    dict.full[tid].offset = off;
  }
  __syncthreads();

  double pw = 0.0, pv = 0.0;
  const int row_end = min((L + 1) * C.rows, dim);
  for (int row0 = first; row0 < row_end; row0 += NW * 16 * STEPS) {
    if (row0 != first) load_pass(row0);
    const int own = row0 + (STEPS > 1 ? lane : r);
    const bool mine = own < dim && q < STEPS;
    // kLeja: the terms' sum with their coefficients; kSplitComm: both products
    constexpr int NR = MODE == kSplitComm ? 2 : 1;
    SliceSums<STEPS> sums[NR];
#pragma unroll 1
    for (int j = 0; j < STEPS; ++j) {
      const int row = row0 + 16 * j + r;
      CodeWords w;
#pragma unroll
      for (int k = 0; k < kCodeAhead; ++k) w.ahead[k] = cw[k];
      if (j + 1 < STEPS) load_words(row0 / 16 + j + 1);
      else if (STEPS > 1) load_own(row0);
      d2 sum[NR];
#pragma unroll
      for (int i = 0; i < NR; ++i) sum[i] = d2{0.0, 0.0};
      if (row0 + 16 * j >= dim) {  // (uniform) no rows left
      } else if (block >= 0) {
        const int slice = row0 / 16 + j;
        int end[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) end[t] = (int)(__builtin_amdgcn_readlane(head[t], 16 * j) & 255u);
        const unsigned row16 = 16u * (unsigned)min(row, dim - 1);
        w.first = C.codes + ((size_t)slice * 64 + lane) * kCodeAhead;
        w.more = C.more + (size_t)slice * (kCodeMore * 64) + lane;
        w.rounds = end[NT - 1];
        // neighbouring terms of one kind on one vector are one stream of rounds
        int rd = 0;
#pragma unroll 1
        for (int t = 0; t < NT; ++t) {
          const int e = t == 0 ? end[0] : t == 1 ? end[1] : end[NT - 1];
          const bool imag = one_real && (block & (kCodeImag << t));
          const d2* x = t == 1 ? xs[1] : xs[0];
          if (MODE == kLeja && t + 1 < NT) {
            const bool next_imag = one_real && (block & (kCodeImag << (t + 1)));
            if (next_imag == imag && (t + 1 == 1 ? xs[1] : xs[0]) == x) continue;
          }
          const __amdgpu_buffer_rsrc_t buf = state_buffer(x, dim);
          const d2 y = one_real ? code_stream(dict.real, w, rd, e, row16, buf) : code_stream(dict.full, w, rd, e, row16, buf);
          const d2 z = imag ? d2{-y.y, y.x} : y;
          if (NR == 2 && t == 1) sum[NR - 1] = z;
          else sum[0] += z;
          rd = e;
        }
      } else {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const d2 y = plain_row(T.m[t], row, dim, q, xs[t]);
          if (NR == 2) sum[t < NR ? t : 0] = y;
          else sum[0] += rmul(t == 0 ? a.a1 : t == 1 ? a.a2 : a3, y);
        }
      }
#pragma unroll
      for (int i = 0; i < NR; ++i) sums[i].put(j, sum[i]);
    }
    d2 res[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) res[i] = sums[i].total(q);
    if (mine) {
      auto diag_part = [&](int t) {
        d2 x = w_old;
        if (xs[t] != reinterpret_cast<const d2*>(a.wcur)) x = xs[t][own];
        return rmul(diag[t], x);
      };
      const bool has[3] = {block >= 0 && (head[0] >> 8), block >= 0 && (head[1] >> 8), NT == 3 && block >= 0 && (head[NT - 1] >> 8)};
      if constexpr (MODE == kSplitComm) {
        if (has[0]) res[0] += diag_part(0);
        if (has[1]) res[1] += diag_part(1);
        a.wout[own] = fromd2(rmul(a.a1, w_old) + rmul(a.kap, d2{-res[1].y, res[1].x}));
        a.pacc[own] = fromd2(rmul(a.a2, w_old) - rmul(a.kap, d2{-res[0].y, res[0].x}));
      } else {
        d2 y = res[0];
        if (has[0]) y += rmul(a.a1, diag_part(0));
        if (has[1]) y += rmul(a.a2, diag_part(1));
        if (NT == 3 && has[2]) y += rmul(a3, diag_part(2));
        const d2 wn = y - rmul(a.sigma, w_old);
        d2 p;
        if (a.first) {
          p = cmul(tod2(a.d0), w_old) + cmul(tod2(a.d), wn);
          pv += nrm2(w_old);
        } else {
          p = p_old + cmul(tod2(a.d), wn);
        }
        a.wout[own] = fromd2(wn);
        a.pacc[own] = fromd2(p);
        pw += nrm2(wn);
      }
    }
  }
  if constexpr (MODE == kLeja) {
    pw = wave_sum(pw);
    pv = wave_sum(pv);
    if (lane == 0) {
      red[0][wv] = pw;
      red[1][wv] = pv;
    }
    __syncthreads();
    if (tid == 0) {
      double bw = 0.0, bv = 0.0;
      for (int k = 0; k < NW; ++k) {
        bw += red[0][k];
        bv += red[1][k];
      }
      a.partials[blockIdx.x] = bw;
      if (a.first) a.partials[gridDim.x + blockIdx.x] = bv;
    }
  }
}

}  // namespace

int code_rows(int dim) {
  int r = 64;
  while ((dim + r - 1) / r > kFuseMaxGrid) r *= 2;
  return r;
}

int code_grid(int dim, int rows) { return (dim + rows - 1) / rows; }

hipError_t launch_code_build(const CodeTerms& T, int dim, const CodedDev& C, int* bad_blocks, hipStream_t s,
                             const double* flags, int nflags) {
  const int g = code_grid(dim, C.rows);
  if (T.n == 2) code_build_kernel<2><<<g, kThreads, 0, s>>>(T, dim, C, bad_blocks, flags, nflags);
  else if (T.n == 3) code_build_kernel<3><<<g, kThreads, 0, s>>>(T, dim, C, bad_blocks, flags, nflags);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_coded_iter(int mode, const CodeTerms& T, int dim, const CodedDev& C, const IterArgs& a, double a3,
                             hipStream_t s) {
  const int g = code_grid(dim, C.rows);
#define MAGNUS_CODED(M, N)                                                                  \
  do {                                                                                      \
    if (C.rows == 64) coded_iter_kernel<M, N, 1, 256><<<g, 256, 0, s>>>(T, dim, C, a, a3);  \
    else if (C.rows == 128) coded_iter_kernel<M, N, 2, 256><<<g, 256, 0, s>>>(T, dim, C, a, a3);  \
    else coded_iter_kernel<M, N, 4, 256><<<g, 256, 0, s>>>(T, dim, C, a, a3);               \
    return hipGetLastError();                                                               \
  } while (0)
  if (T.n < 2 || T.n > 3) return hipErrorInvalidValue;
  if (mode == kSplitComm) MAGNUS_CODED(kSplitComm, 2);
  if (mode == kLeja && T.n == 2) MAGNUS_CODED(kLeja, 2);
  if (mode == kLeja) MAGNUS_CODED(kLeja, 3);
#undef MAGNUS_CODED
  return hipErrorInvalidValue;
}

}  // namespace magnus

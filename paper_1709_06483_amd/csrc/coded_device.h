// Device parts shared by the kernels that iterate on coded CSR terms
// (kernels_coded.hip describes the form).
#pragma once

#include "device_common.h"

namespace magnus {
namespace dev {

// A row of a block that is not coded, from the CSR arrays (its quarter q of the entries).
__device__ __forceinline__ d2 plain_row(const CsrDev& M, int row, int dim, int q, const d2* x) {
  d2 acc = {0.0, 0.0};
  if (row < dim) {
    const d2* v = reinterpret_cast<const d2*>(M.val);
    const int e1 = M.rp[row + 1];
    for (int e = M.rp[row] + q; e < e1; e += 4) acc += cmul(v[e], x[M.ci[e]]);
  }
  return acc;
}

// The dictionary as an iteration uses it, values times their term's coefficient.
struct RealEntry {
  double val;
  int offset, pad;
};
struct FullEntry {
  double2 val;
  int offset, pad[3];
};
union DictLds {
  FullEntry full[kCodeMax + 1];
  RealEntry real[kCodeMax + 1];
};

__device__ __forceinline__ d2 code_mul(double2 h, d2 x) { return cmul(tod2(h), x); }
__device__ __forceinline__ d2 code_mul(double h, d2 x) { return rmul(h, x); }

// A state as a buffer of num_records bytes: a load outside it returns zeros
// without an access, which is what a lane without an entry (offset kNoEntry) does.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t state_buffer(const d2* x, int dim) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<d2*>(x), 0, dim * 16, 0x00020000);
}
__device__ __forceinline__ d2 buffer_at(__amdgpu_buffer_rsrc_t x, unsigned offset) {
  typedef unsigned u4 __attribute__((ext_vector_type(4)));
  const u4 v = __builtin_amdgcn_raw_buffer_load_b128(x, (int)offset, 0, 0);
  return __builtin_bit_cast(d2, v);
}

// The next K rounds, a code to a byte of `words`: all gathers issued before the first product.
template <int K, class Entry>
__device__ __forceinline__ void code_rounds(const Entry* dict, const unsigned (&words)[2], unsigned row16,
                                            __amdgpu_buffer_rsrc_t x, d2& sum) {
  d2 g[K];
#pragma unroll
  for (int k = 0; k < K; ++k)
    g[k] = buffer_at(x, row16 + (unsigned)dict[(words[k / 4] >> (8 * (k & 3))) & 255u].offset);
  asm volatile("" ::: "memory");  // the values are read once the gathers are out: held with them they cost waves
#pragma unroll
  for (int k = 0; k < K; ++k) sum += code_mul(dict[(words[k / 4] >> (8 * (k & 3))) & 255u].val, g[k]);
}

// A slice's codes: the words loaded ahead, and where to find all of them.
struct CodeWords {
  unsigned ahead[kCodeAhead];
  const unsigned* first;  // word k < kCodeAhead at first[k]
  const unsigned* more;   // word k at more[(k - kCodeAhead) * 64] after them
  int rounds;             // of the slice
};

// The codes of the eight rounds from rd on (uniform; bytes past the slice's rounds are not used).
__device__ __forceinline__ void code_window(const CodeWords& w, int rd, unsigned (&out)[2]) {
  const int i = rd >> 2;
  unsigned a[3];
  static_assert(kCodeAhead == 3, "three words ahead");
  if (w.rounds <= 4 * kCodeAhead) {
    a[0] = i == 0 ? w.ahead[0] : i == 1 ? w.ahead[1] : w.ahead[2];
    a[1] = i == 0 ? w.ahead[1] : w.ahead[2];
    a[2] = w.ahead[2];
  } else {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int g = min(i + k, (w.rounds - 1) >> 2);
      a[k] = g < kCodeAhead ? w.first[g] : w.more[(g - kCodeAhead) * 64];
    }
  }
  out[0] = __builtin_amdgcn_alignbyte(a[1], a[0], rd & 3);
  out[1] = __builtin_amdgcn_alignbyte(a[2], a[1], rd & 3);
}

// The lane's products over rounds [rd, end) of a slice, in pieces of eight
// rounds (four where values are complex, whose registers would leave fewer
// waves), then of 4, 2 or 1.
template <class Entry>
__device__ __forceinline__ d2 code_stream(const Entry* dict, const CodeWords& w, int rd, int end, unsigned row16,
                                          __amdgpu_buffer_rsrc_t x) {
  constexpr bool kWide = sizeof(Entry) == sizeof(RealEntry);
  d2 sum = {0.0, 0.0};
#pragma unroll 1
  while (rd < end) {
    const int left = end - rd;
    unsigned words[2];
    code_window(w, rd, words);
    if (kWide && left > 4) {
      if (left < 8) words[1] &= (1u << (8 * (left - 4))) - 1u;
      code_rounds<8>(dict, words, row16, x, sum);
      rd += 8;
    } else if (left > 2) {
      if (left < 4) words[0] &= 0xFFFFFFu;
      code_rounds<4>(dict, words, row16, x, sum);
      rd += 4;
    } else if (left == 2) {
      code_rounds<2>(dict, words, row16, x, sum);
      rd += 2;
    } else {
      code_rounds<1>(dict, words, row16, x, sum);
      rd += 1;
    }
  }
  return sum;
}

__device__ __forceinline__ void swap32(double& a, double& b) {
  typedef unsigned u2 __attribute__((ext_vector_type(2)));
  union { double d; unsigned u[2]; } x{a}, y{b};
  for (int k = 0; k < 2; ++k) {
    const u2 r = __builtin_amdgcn_permlane32_swap(x.u[k], y.u[k], false, false);
    x.u[k] = r.x;
    y.u[k] = r.y;
  }
  a = x.d;
  b = y.d;
}
__device__ __forceinline__ void swap16(double& a, double& b) {
  typedef unsigned u2 __attribute__((ext_vector_type(2)));
  union { double d; unsigned u[2]; } x{a}, y{b};
  for (int k = 0; k < 2; ++k) {
    const u2 r = __builtin_amdgcn_permlane16_swap(x.u[k], y.u[k], false, false);
    x.u[k] = r.x;
    y.u[k] = r.y;
  }
  a = x.d;
  b = y.d;
}

// A transposing reduction: lane 16 j + r gets the sum of y_j over the lanes
// 16 q + r, j < 4, as quarter_sum(half_sum(y0, y2), half_sum(y1, y3)): two
// exchanges instead of eight shuffles and adds.
__device__ __forceinline__ double half_sum(double y0, double y2) {
  swap32(y0, y2);  // y0: quarters 0, 1 of y0, then of y2; y2: quarters 2, 3 likewise
  return y0 + y2;
}
__device__ __forceinline__ double quarter_sum(double y02, double y13) {
  swap16(y02, y13);  // quarters 0 + 2 of y0, y1, y2, y3; quarters 1 + 3
  return y02 + y13;
}

// The sums of a wave's slices, STEPS = 1, 2 or 4 of them, each lane's share put
// in slice by slice (j uniform); total() is the sum of row r of slice j at lane
// 16 j + r (STEPS = 1: at every quarter).
template <int STEPS>
struct SliceSums {
  d2 v[STEPS == 1 ? 1 : 2];
  __device__ __forceinline__ void put(int j, d2 y) {
    if (j == 0) v[0] = y;
    if constexpr (STEPS > 1) {
      if (j == 1) v[1] = y;
    }
    if constexpr (STEPS == 4) {
      if (j == 2) v[0] = d2{half_sum(v[0].x, y.x), half_sum(v[0].y, y.y)};
      if (j == 3) v[1] = d2{half_sum(v[1].x, y.x), half_sum(v[1].y, y.y)};
    }
  }
  __device__ __forceinline__ d2 total(int quarter) const {
    if constexpr (STEPS == 4) {
      return d2{quarter_sum(v[0].x, v[1].x), quarter_sum(v[0].y, v[1].y)};
    } else {
      d2 t = {0.0, 0.0};
#pragma unroll
      for (int j = 0; j < STEPS; ++j) {
        d2 y = v[j];
#pragma unroll
        for (int off = 32; off >= 16; off >>= 1) {
          y.x += __shfl_xor(y.x, off, 64);
          y.y += __shfl_xor(y.y, off, 64);
        }
        if (STEPS == 1 || quarter == j) t = y;
      }
      return t;
    }
  }
};

}  // namespace dev
}  // namespace magnus

// Coefficients of the two-site MPO apply, one workgroup's share.  Every entry
// of a coefficient row (class, output o) is the sum of its W1*W2 terms in a
// fixed order; the row is written dense (coef64/coef32) and compacted to its
// nonzero entries in increasing input order (cnt, idx, val64, val32) for the
// sparse apply.
//
// The work is a few microseconds of dependent loads on a handful of
// workgroups, and nothing before the MPO apply needs it, so it has no launch of
// its own: these workgroups run beside the splits or beside L.psi (a launch
// between dependent kernels costs 4 to 5 us on the GPU and 2 on the host; the
// float64 apply at chi = 2048 went from 67.2 to 61.7 us).
#pragma once
#include "bst_internal.h"

namespace bst {

inline int64_t hcoef_blocks(const HCoefLaunch& c) { return (c.nentries + 255) / 256; }
inline bool hcoef_valid(const HCoefLaunch& c) {
  return c.nentries == 0 || (c.nmax > 0 && 256 % c.nmax == 0 && c.nentries % c.nmax == 0);
}

// 256 lanes; cs: 256 doubles of LDS
__device__ __forceinline__ void hcoef_block(const HCoefLaunch& c, int64_t block, double* cs) {
  // one lane per entry, then one lane per row compacts the row (nmax
  // divides 256, so a workgroup holds whole rows)
  const int tid = threadIdx.x, nmax = c.nmax;
  const int64_t e = block * 256 + tid;
  double sum = 0.0;
  if (e < c.nentries) {
    for (int32_t k = c.entry_begin[e]; k < c.entry_begin[e + 1]; ++k) {
      const HTerm t = c.terms[k];
      const double w1 = ((const BST_G double*)(c.ptrs[t.w1_buf]))[t.w1_off];
      const double w2 = ((const BST_G double*)(c.ptrs[t.w2_buf]))[t.w2_off];
      sum += w1 * w2;
    }
    c.coef64[e] = sum;
    c.coef32[e] = (float)sum;
  }
  cs[tid] = sum;
  __syncthreads();
  const int rpb = 256 / nmax;
  if (tid >= rpb) return;
  const int64_t row = block * rpb + tid;
  if (row * nmax >= c.nentries) return;
  int32_t n = 0;
  for (int i = 0; i < nmax; ++i) {
    const double v = cs[tid * nmax + i];
    if (v != 0.0) {
      c.idx[row * nmax + n] = i;
      c.val64[row * nmax + n] = v;
      c.val32[row * nmax + n] = (float)v;
      ++n;
    }
  }
  c.cnt[row] = n;
}

}  // namespace bst

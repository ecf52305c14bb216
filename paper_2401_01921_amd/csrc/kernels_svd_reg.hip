// Symmetric SVD of sector matrices that fit one workgroup's registers.
//
// A sector's tall matrix X (p x r, p >= r) goes through three kernels:
//
// 1. svd_panel_kernel / svd_trail_kernel: the rows of X, ordered by falling
//    norm, and its columns, by falling largest element (P), are reduced to lower trapezoidal form by
//    Householder reflections from the right, X <- X P Q, and V <- P Q starts as
//    that orthogonal factor.  Jacobi on X P Q needs about half the sweeps of
//    Jacobi on X (Drmac and Veselic, SIAM J. Matrix Anal. Appl. 2008: the Gram
//    matrix of the triangular factor is one LR step nearer to diagonal).  Both
//    orders count for the small singular values: a reflection leaves an error of
//    the rounding of its row's large elements in all of them, which a small
//    column bears only if it comes after the large ones (Cox and Higham, on
//    Householder QR of row-wise graded matrices, 1998).  24 x 20, columns of 1 to 1e-20 in any order, largest relative
//    error of a singular value: rows ordered alone 100, both 5e-15, Jacobi on X
//    itself 2e-15.
// 2. svd_reg_kernel: one-sided Jacobi with X in registers, one workgroup per
//    sector.  It logs its rotations.
// 3. svd_apply_kernel: the logged rotations on the rows of V, which are
//    independent of each other and spread over the device.
//
// Measured, kernels only: a two-site spin-1/2 state at chi = 256 (15 sectors
// to 52 x 52), 1.62 ms in the one-workgroup LDS kernel before, now 37 us (1) +
// 164 us (2) + 27 us (3); at chi = 1024 (to 204 x 204), 23 ms of one launch per
// round before, now 7 x (45 + 13) us (1) + 2.28 ms (2) + 0.14 ms (3).
//
// The squares of a row or column have to stay inside float64's range: below it a
// reflection is not orthogonal, and V with it (entries of 1e-160: |V V^T - 1| =
// 1e-3).  A sector whose largest element is outside 2^-128 .. 2^128 is worked on
// times a power of two (exact), and so is the reflection of a row that is tiny
// even then.
//
// Layout of a sector in the workspace: p + r rows of ld doubles, the rows of
// X (sorted) and then those of V; ld is the padded column count N.  Its part of
// rowpos: the place of every row of X and the inverse, then of every column.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>
#include <type_traits>

#include "plan.h"

#include "svd.h"

namespace bst {

namespace {

// ---- cross-lane helpers ----------------------------------------------------
template <int CTRL>
__device__ __forceinline__ double dpp_zero(double v) {   // lanes without a source get 0
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}
constexpr int kWaveShl1 = 0x130;   // lane i takes lane i + 1
constexpr int kWaveShr1 = 0x138;   // lane i takes lane i - 1
constexpr int kRowRor = 0x120;     // + n: rotation within 16 lanes

// The lane, formed anew at every use: where the columns take nearly all
// registers, an index kept across them would be spilled.
__device__ __forceinline__ int fresh_lane() {
  int l;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=&v"(l));
  return l;
}
__device__ __forceinline__ double uniform(double v) {
  return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)),
                          __builtin_amdgcn_readfirstlane(__double2loint(v)));
}

// 1 / sqrt(q) to rounding: the hardware's estimate (some 26 bits) and one
// third-order step, fewer dependent operations than sqrt and a division.
__device__ __forceinline__ double rsqrt_step(double q) {
  const double c = __builtin_amdgcn_rsq(q);
  const double e = fma(-q * c, c, 1.0);
  return fma(c * e, fma(0.375, e, 0.5), c);
}

// Sum over 16 lanes, the same value in each.
__device__ __forceinline__ double row_sum(double v) {
  v += dpp_zero<kRowRor + 8>(v);
  v += dpp_zero<kRowRor + 4>(v);
  v += dpp_zero<kRowRor + 2>(v);
  v += dpp_zero<kRowRor + 1>(v);
  return v;
}

// Order of non-negative values by their bits; NaN sorts first, so that a
// ranking by it is a permutation whatever the values are.
__device__ __forceinline__ unsigned long long order_key(double v) {
  return (unsigned long long)__double_as_longlong(v) & 0x7FFFFFFFFFFFFFFFull;
}

}  // namespace

// Householder rows [k0, k0 + rows) of one sector per workgroup, held in LDS:
// the reflections of rows k0 .. k0 + nref - 1 on all later rows of the range.
// A sector whose rows of X and V all fit is done in one launch; otherwise its
// rows come nb at a time and svd_trail_kernel carries the reflections (kept in
// ubuf) to the rest.  Panel 0 first orders the rows and columns of X.
//
// A row takes 16 lanes (E column pairs each), so that a sum along it is four
// moves within them, and a wave four rows at a time.  Wave 0 takes the four
// rows after the reflected one and from the first of them forms the next
// reflection, while the other waves bring the rest of the rows up to date: one
// barrier per reflection.  Bound: the latency of that chain (read u, dot,
// update, norm, two reciprocal roots, write u).
namespace {

template <int E>
__device__ __forceinline__ void load_pairs(double2 (&x)[E], const double* row, int l16) {
#pragma unroll
  for (int j = 0; j < E; ++j) x[j] = *reinterpret_cast<const double2*>(row + 2 * l16 + 32 * j);
}
template <int E>
__device__ __forceinline__ void store_pairs(const double2 (&x)[E], double* row, int l16) {
#pragma unroll
  for (int j = 0; j < E; ++j) *reinterpret_cast<double2*>(row + 2 * l16 + 32 * j) = x[j];
}
// x <- x - (x.u) u along a row
template <int E>
__device__ __forceinline__ void reflect(double2 (&x)[E], const double2 (&u)[E]) {
  double w0 = 0.0, w1 = 0.0;
#pragma unroll
  for (int j = 0; j < E; ++j) {
    w0 = fma(x[j].x, u[j].x, w0);
    w1 = fma(x[j].y, u[j].y, w1);
  }
  const double w = row_sum(w0 + w1);
#pragma unroll
  for (int j = 0; j < E; ++j) {
    x[j].x = fma(-w, u[j].x, x[j].x);
    x[j].y = fma(-w, u[j].y, x[j].y);
  }
}
// The reflection H = I - u u^T, |u|^2 = 2, that takes row x from column c0 on
// to a multiple of e_c0: u, and x as it leaves it.  A zero row gives u = 0; u of
// one whose square would lose digits comes from the row times 2^800.
template <int E>
__device__ __forceinline__ void reflector(double2 (&x)[E], double2 (&u)[E], double x0, int c0, int l16) {
  double q0 = 0.0, q1 = 0.0;
#pragma unroll
  for (int j = 0; j < E; ++j) {
    const int c = 2 * l16 + 32 * j;
    u[j].x = c >= c0 ? x[j].x : 0.0;
    u[j].y = c + 1 >= c0 ? x[j].y : 0.0;
    q0 = fma(u[j].x, u[j].x, q0);
    q1 = fma(u[j].y, u[j].y, q1);
  }
  const double q = row_sum(q0 + q1);
  const bool zero = q == 0.0;
  const double nrm = q * rsqrt_step(q);
  const double s = copysign(nrm, x0);
  double sc = zero ? 0.0 : rsqrt_step(nrm * (nrm + fabs(x0)));
  double diag = zero ? 0.0 : -s, head = zero ? 0.0 : (x0 + s) * sc;
  // (decided on last, off the chain; 16 lanes agree)
  if (__builtin_expect(__ballot(q < 0x1p-900) != 0ull, 0) && q < 0x1p-900) {
    x0 *= 0x1p800;
    q0 = q1 = 0.0;
#pragma unroll
    for (int j = 0; j < E; ++j) {
      u[j].x *= 0x1p800;
      u[j].y *= 0x1p800;
      q0 = fma(u[j].x, u[j].x, q0);
      q1 = fma(u[j].y, u[j].y, q1);
    }
    const double qq = row_sum(q0 + q1), n = qq * rsqrt_step(qq), ss = copysign(n, x0);
    if (qq > 0.0) {
      sc = rsqrt_step(n * (n + fabs(x0)));
      diag = -ss * 0x1p-800;
      head = (x0 + ss) * sc;
    }
  }
#pragma unroll
  for (int j = 0; j < E; ++j) {
    const int c = 2 * l16 + 32 * j;
    u[j].x = c == c0 ? head : u[j].x * sc;
    u[j].y = c + 1 == c0 ? head : u[j].y * sc;
    x[j].x = c == c0 ? diag : c > c0 ? 0.0 : x[j].x;
    x[j].y = c + 1 == c0 ? diag : c + 1 > c0 ? 0.0 : x[j].y;
  }
}

// ub: two rows of LDS for u, in turn.
template <int E>
__device__ __forceinline__ void panel_rows(double* lds, double* ub, double* ubuf, int ld, int k0, int nref,
                                           int rows) {
  constexpr int NW = 16, LDL = 32 * E;
  const int l16 = threadIdx.x & 15, grp = (threadIdx.x >> 4) & 3;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // the reflection of row i from x in the wave's first 16 lanes (the others
  // idle along), x0 its element on the diagonal
  auto form = [&](double2 (&x)[E], double x0, int i) {
    double2 u[E];
    reflector<E>(x, u, x0, k0 + i, l16);
    if (grp == 0) {
      store_pairs<E>(x, lds + i * LDL, l16);
      store_pairs<E>(u, ub + (i & 1) * LDL, l16);
      if (ubuf) {
#pragma unroll
        for (int j = 0; j < E; ++j)
          if (2 * l16 + 32 * j < ld)
            *reinterpret_cast<double2*>(ubuf + (int64_t)(k0 + i) * ld + 2 * l16 + 32 * j) = u[j];
      }
    }
  };
  if (wave == 0) {
    double2 x[E];
    load_pairs<E>(x, lds, l16);
    form(x, lds[k0], 0);
  }
  __syncthreads();
  for (int i = 0; i < nref; ++i) {
    double2 u[E], x[E];
    load_pairs<E>(u, ub + (i & 1) * LDL, l16);
    if (wave == 0) {
      const int q = i + 1 + grp;
      load_pairs<E>(x, lds + min(q, rows - 1) * LDL, l16);
      reflect<E>(x, u);
      if (q < rows) store_pairs<E>(x, lds + q * LDL, l16);
      if (i + 1 < nref) form(x, lds[(i + 1) * LDL + k0 + i + 1], i + 1);
    } else {
      for (int q0 = i + 5 + 4 * (wave - 1); q0 < rows; q0 += 4 * (NW - 1)) {
        const int q = q0 + grp;
        load_pairs<E>(x, lds + min(q, rows - 1) * LDL, l16);
        reflect<E>(x, u);
        if (q < rows) store_pairs<E>(x, lds + q * LDL, l16);
      }
    }
    __syncthreads();
  }
}
}  // namespace

__global__ __launch_bounds__(1024) void svd_panel_kernel(const SvdSec* __restrict__ secs,
                                                         const int32_t* __restrict__ list, double* D,
                                                         double* scratch, int32_t* rowpos, int32_t* ctrl,
                                                         int panel) {
  const SvdSec S = secs[list[blockIdx.x]];
  const int p = S.m >= S.n ? S.m : S.n, r = S.m >= S.n ? S.n : S.m;
  const int k0 = panel * S.nb;
  if (k0 >= r) return;
  const bool whole = S.nb >= r;
  const int ld = S.ld, nref = min(S.nb, r - k0);
  const int rows = whole ? p + r : nref;
  const int tid = threadIdx.x;
  const int ldl = svd_panel_ld(ld);
  __shared__ __attribute__((aligned(16))) double lds[kSvdPanelLds / sizeof(double)];
  __shared__ __attribute__((aligned(16))) double ub[2 * kSvdRegMaxCols];
  __shared__ double nrm[kSvdRegMaxRows];
  __shared__ unsigned long long cmax[kSvdRegMaxCols];
  __shared__ int inv[kSvdRegMaxRows], cpos[kSvdRegMaxCols];
  double* const X = D + S.x_off;
  const double* const X0 = scratch + S.log_off;                  // as gathered
  double* const ubuf = scratch + S.log_off + (int64_t)p * ld;    // row i: the u of reflection i
  int32_t* const pos = rowpos + S.p_off;   // [0, p): sorted place of a row; [p, 2p): its inverse
  int32_t* const pos_c = pos + 2 * p;      // the same of the r columns
  const int l16 = tid & 15;
  int ex = 0;   // X is held times 2^-ex
  if (panel == 0) {
    // |row|^2 and the largest element of every column
    constexpr int NC = kSvdRegRows2 / 16;   // columns of a lane, at most
    static_assert(kSvdRegCols1 <= 16 * NC && kSvdRegMaxRows <= 256, "lanes of a row");
    if (tid < r) cmax[tid] = 0ull;
    double cm[NC];
#pragma unroll
    for (int j = 0; j < NC; ++j) cm[j] = 0.0;
    for (int q = tid >> 4; q < p; q += 64) {
      double a = 0.0, v[NC];
#pragma unroll
      for (int j = 0; j < NC; ++j)
        if (16 * j < r) v[j] = X0[(int64_t)q * ld + min(l16 + 16 * j, r - 1)];
#pragma unroll
      for (int j = 0; j < NC; ++j) {
        if (16 * j >= r) break;
        a = l16 + 16 * j < r ? fma(v[j], v[j], a) : a;
        cm[j] = fmax(cm[j], fabs(v[j]));
      }
      a = row_sum(a);
      if (l16 == 0) nrm[q] = a;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      if (16 * j >= r) break;
      if (l16 + 16 * j < r && tid >> 4 < p) atomicMax(&cmax[l16 + 16 * j], order_key(cm[j]));
    }
    __syncthreads();
    // four lanes per row and column count those before it (p >= r)
    const int q = tid >> 2;
    int rank = 0, rank_c = 0;
    unsigned long long top = 0ull;   // the largest element, in every lane
    {
      const unsigned long long k = q < p ? order_key(nrm[q]) : 0ull, kc = q < r ? cmax[q] : 0ull;
      for (int i = tid & 3; i < p; i += 4) {
        const unsigned long long w = order_key(nrm[i]), wc = i < r ? cmax[i] : 0ull;
        rank += (w > k || (w == k && i < q)) ? 1 : 0;
        rank_c += i < r && (wc > kc || (wc == kc && i < q)) ? 1 : 0;
        top = max(top, wc);
      }
    }
    top = max(top, (unsigned long long)__shfl_xor(top, 1, 4));
    top = max(top, (unsigned long long)__shfl_xor(top, 2, 4));
    const double t = __longlong_as_double((long long)top);
    if (t > 0.0 && t <= DBL_MAX && (t < 0x1p-128 || t > 0x1p128)) {
      ex = ilogb(t);
      __syncthreads();   // (every lane has read the norms)
      for (int i = tid >> 4; i < p; i += 64) {
        double a = 0.0;
        for (int c = l16; c < r; c += 16) {
          const double v = ldexp(X0[(int64_t)i * ld + c], -ex);
          a = fma(v, v, a);
        }
        a = row_sum(a);
        if (l16 == 0) nrm[i] = a;
      }
      __syncthreads();
      rank = 0;
      const unsigned long long k = q < p ? order_key(nrm[q]) : 0ull;
      for (int i = tid & 3; i < p; i += 4) {
        const unsigned long long w = order_key(nrm[i]);
        rank += (w > k || (w == k && i < q)) ? 1 : 0;
      }
    }
    if (tid == 0) ctrl[kSvdCtrl * blockIdx.x + 2] = ex;
    rank += __shfl_xor(rank, 1, 4);
    rank += __shfl_xor(rank, 2, 4);
    rank_c += __shfl_xor(rank_c, 1, 4);
    rank_c += __shfl_xor(rank_c, 2, 4);
    if ((tid & 3) == 0 && q < p) {
      inv[rank] = q;
      pos[q] = rank;
      pos[p + rank] = q;
    }
    if ((tid & 3) == 0 && q < r) {
      cpos[q] = rank_c;
      pos_c[q] = rank_c;
      pos_c[r + rank_c] = q;
    }
    __syncthreads();
  }
  // 16 lanes per row, all of a row's loads at once
  for (int q = tid >> 4; q < rows; q += 64) {
    const int g = k0 + q;
    const bool unit = panel == 0 && g >= p;   // a row of P
    const double* const src = panel == 0 ? X0 + (int64_t)inv[min(g, p - 1)] * ld : X + (int64_t)g * ld;
    const int one = unit ? cpos[g - p] : -1;
    double2 x[7];
#pragma unroll
    for (int j = 0; j < 7; ++j)
      if (32 * j < ldl) x[j] = *reinterpret_cast<const double2*>(src + min(2 * l16 + 32 * j, ld - 2));
#pragma unroll
    for (int j = 0; j < 7; ++j) {
      const int c = 2 * l16 + 32 * j;
      if (32 * j >= ldl) break;
      double2 v = x[j];
      if (ex != 0) v = double2{ldexp(v.x, -ex), ldexp(v.y, -ex)};
      if (unit) v = double2{c == one ? 1.0 : 0.0, c + 1 == one ? 1.0 : 0.0};
      if (c >= r) v.x = 0.0;
      if (c + 1 >= r) v.y = 0.0;
      double* const row = lds + q * ldl;
      if (panel == 0 && !unit) {   // each column to its place
        row[c < r ? cpos[c] : c] = v.x;
        row[c + 1 < r ? cpos[c + 1] : c + 1] = v.y;
      } else {
        *reinterpret_cast<double2*>(row + c) = v;
      }
    }
  }
  __syncthreads();
  double* const keep = whole ? nullptr : ubuf;
  if (ldl == 32) panel_rows<1>(lds, ub, keep, ld, k0, nref, rows);
  else if (ldl == 64) panel_rows<2>(lds, ub, keep, ld, k0, nref, rows);
  else if (ldl == 128) panel_rows<4>(lds, ub, keep, ld, k0, nref, rows);
  else panel_rows<7>(lds, ub, keep, ld, k0, nref, rows);
  __syncthreads();
  for (int q = tid >> 4; q < rows; q += 64)
    for (int c = 2 * (tid & 15); c < ld; c += 32)
      *reinterpret_cast<double2*>(X + (int64_t)(k0 + q) * ld + c) = *reinterpret_cast<double2*>(lds + q * ldl + c);
}

// The reflections of one panel on the rows after it (those of X and all of
// V's), 16 lanes per row as above, two rows per lane group in registers and
// the panel's u in LDS.  Panel 0 takes X from the gathered copy in sorted order
// (pos: that order, as in the panel kernel) and starts V from P.  Bound: latency of the sum
// along a row, hidden by the second row and the other waves.
namespace {
template <int E>
__device__ __forceinline__ void trail_rows(const SvdSec& S, double* X, const double* X0, const int32_t* pos,
                                           int ex, const double* ul, int panel, int nref, int q0) {
  constexpr int LDL = 32 * E;
  const int p = S.m >= S.n ? S.m : S.n, r = S.m >= S.n ? S.n : S.m, ld = S.ld;
  const int l16 = threadIdx.x & 15;
  const int32_t *const inv = pos + p, *const pos_c = pos + 2 * p;
  double2 x[2][E];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int g = min(q0 + t, p + r - 1);
    if (panel > 0) {
#pragma unroll
      for (int j = 0; j < E; ++j) {
        const int c = 2 * l16 + 32 * j;
        const double2 v = *reinterpret_cast<const double2*>(X + (int64_t)g * ld + min(c, ld - 2));
        x[t][j] = double2{c < r ? v.x : 0.0, c + 1 < r ? v.y : 0.0};
      }
    } else {
      const bool unit = g >= p;
      const int one = unit ? pos_c[g - p] : -1;
      const double* const src = X0 + (int64_t)inv[min(g, p - 1)] * ld;
#pragma unroll
      for (int j = 0; j < E; ++j) {
        const int c = 2 * l16 + 32 * j;
        double v0 = src[pos_c[r + min(c, r - 1)]], v1 = src[pos_c[r + min(c + 1, r - 1)]];
        if (ex != 0) {
          v0 = ldexp(v0, -ex);
          v1 = ldexp(v1, -ex);
        }
        x[t][j].x = unit ? (c == one ? 1.0 : 0.0) : c < r ? v0 : 0.0;
        x[t][j].y = unit ? (c + 1 == one ? 1.0 : 0.0) : c + 1 < r ? v1 : 0.0;
      }
    }
  }
  for (int i = 0; i < nref; ++i) {
    double2 u[E];
    load_pairs<E>(u, ul + i * LDL, l16);
    reflect<E>(x[0], u);
    reflect<E>(x[1], u);
  }
#pragma unroll
  for (int t = 0; t < 2; ++t)
    if (q0 + t < p + r) {
#pragma unroll
      for (int j = 0; j < E; ++j)
        if (2 * l16 + 32 * j < ld)
          *reinterpret_cast<double2*>(X + (int64_t)(q0 + t) * ld + 2 * l16 + 32 * j) = x[t][j];
    }
}
}  // namespace

__global__ __launch_bounds__(256) void svd_trail_kernel(const SvdSec* __restrict__ secs,
                                                        const int32_t* __restrict__ list, double* D,
                                                        const double* scratch, const int32_t* rowpos,
                                                        const int32_t* ctrl, int panel) {
  __shared__ __attribute__((aligned(16))) double ul[kSvdPanelRefl * 32 * 7];
  const SvdSec S = secs[list[blockIdx.y]];
  const int p = S.m >= S.n ? S.m : S.n, r = S.m >= S.n ? S.n : S.m;
  const int k0 = panel * S.nb, ld = S.ld;
  if (k0 >= r || S.nb >= r) return;
  const int nref = min(S.nb, r - k0);
  const int b0 = k0 + nref + blockIdx.x * kSvdTrailRows;
  if (b0 >= p + r) return;
  double* const X = D + S.x_off;
  const double* const X0 = scratch + S.log_off;
  const double* const ubuf = scratch + S.log_off + (int64_t)p * ld;
  const int32_t* const pos = rowpos + S.p_off;
  const int ex = ctrl[kSvdCtrl * blockIdx.y + 2];
  const int ldl = svd_panel_ld(ld);
  for (int i = threadIdx.x >> 4; i < nref; i += 16) {
    const double* const src = ubuf + (int64_t)(k0 + i) * ld;
#pragma unroll
    for (int j = 0; j < 7; ++j) {
      const int c = 2 * (threadIdx.x & 15) + 32 * j;
      if (32 * j >= ldl) break;
      double2 v = *reinterpret_cast<const double2*>(src + min(c, ld - 2));
      if (c >= ld) v = double2{0.0, 0.0};
      *reinterpret_cast<double2*>(ul + i * ldl + c) = v;
    }
  }
  __syncthreads();
  const int q0 = b0 + 2 * (threadIdx.x >> 4);
  if (ldl == 32) trail_rows<1>(S, X, X0, pos, ex, ul, panel, nref, q0);
  else if (ldl == 64) trail_rows<2>(S, X, X0, pos, ex, ul, panel, nref, q0);
  else if (ldl == 128) trail_rows<4>(S, X, X0, pos, ex, ul, panel, nref, q0);
  else trail_rows<7>(S, X, X0, pos, ex, ul, panel, nref, q0);
}

// ---- Jacobi in registers ---------------------------------------------------
//
// The columns stand at N positions (r and up to 2U - 1 zero columns) and are
// rotated in the odd-even order: steps of kind A pair the positions (2P,
// 2P + 1), steps of kind B the positions (2P + 1, 2P + 2), and every pair
// changes places.  After N steps each pair has met once and the order is
// reversed.  A lane holds the 2U columns of U neighbouring pairs, right-
// aligned in the wave (the last pair in lane 63), for RW rows; a wave holds RW
// rows of every column.  So a dot product is RW local products and one sum
// over the waves through LDS, and a step of kind B moves one column by one
// lane, with wave-wide DPP moves and no LDS.
//
// A pair (x, y) is rotated by two in-place products,
//   y <- y + beta x,  x <- x - alpha y,
// which is the plane rotation x' = c x - s y, y' = s x + c y up to a factor
// c on y' and 1 / c on x': with factors d per column, beta = t d_x / d_y and
// alpha = c s d_y / d_x give d_y' = c d_y and d_x' = d_x / c.  The factors are
// multiplied in, and the norms formed afresh, once per sweep; within a sweep
// the norms follow the rotations (|x'|^2 = a - t g, |y'|^2 = b + t g).  A
// sweep that rotated nothing has decided on fresh norms throughout.  The
// angle need not be exact (an error of it leaves a smaller dot product for the
// next sweep), c^2 (1 + t^2) = 1 does.
//
// The places at the ends pair with nothing in a step of kind B: the last lane
// takes its own x (beta = 1 onto the zeros that the move left), and the lane
// before the first one hands back the column that the move took there
// (alpha = -1 onto its zeros).  One lane must be free for that.
//
// Bound: with X in registers the FP64 units (3 products per element and
// step), below about 128 columns the chain of one step: dot, LDS sum,
// rotation parameters (one wave per pair of a lane), LDS broadcast.
namespace {

struct RegShared {
  double part[kSvdRegWaves][4][64];
  double2 cf[2][64];
  double na[kSvdRegMaxCols], d[kSvdRegMaxCols], e[kSvdRegMaxCols];
  int rotated[2];
};

// What a column carries through a sweep: |x|^2, its factor and the reciprocal.
struct ColState {
  double a, d, e;
};

// The rotation of a pair with states x, y and (scaled) dot product g, and the
// states after it.  Without rotation (on = false, or the columns orthogonal to
// tol) both coefficients are 0.
__device__ __forceinline__ bool rotate(ColState& x, ColState& y, double g, bool on, double tol, double2& cf) {
  g *= x.d * y.d;
  const bool need = on && fabs(g) * (__builtin_amdgcn_rsq(x.a) * __builtin_amdgcn_rsq(y.a)) > tol;
  const double z = (y.a - x.a) * 0.5 * __builtin_amdgcn_rcp(g);
  const double az = fmin(fabs(z), 1e100), q0 = fma(az, az, 1.0);
  double t = copysign(__builtin_amdgcn_rcp(fma(q0, __builtin_amdgcn_rsq(q0), az)), z);
  t = need ? t : 0.0;
  const double q = fma(t, t, 1.0);
  const double c = need ? rsqrt_step(q) : 1.0, ic = q * c;
  cf.x = t * (x.d * y.e);
  cf.y = t * (y.d * x.e) * (c * c);
  y.d *= c;
  y.e *= ic;
  x.d *= ic;
  x.e *= c;
  const double xa = x.a, ya = y.a, tg = need ? t * g : 0.0;
  x.a = fmax(xa - tg, 1e-32 * xa);
  y.a = fmax(ya + tg, 1e-32 * ya);
  return need;
}

// The pairs of one wave of the two-pair layout, states in LDS by position.
template <int U>
__device__ __forceinline__ bool pair_params(RegShared& sh, int u, int lane, int f, int N, bool kind_b, double tol,
                                            double2& cf) {
  const int k = lane - f;
  const int left = 2 * (U * k + u) + (kind_b ? 1 : 0), right = left + 1;
  const bool active = k >= 0 && right < N;
  double s0 = 0.0, s1 = 0.0;
#pragma unroll
  for (int w = 0; w < kSvdRegWaves; w += 2) {
    s0 += sh.part[w][u][lane];
    s1 += sh.part[w + 1][u][lane];
  }
  const int l = active ? left : 0, r = active ? right : 1;
  ColState x{sh.na[l], sh.d[l], sh.e[l]}, y{sh.na[r], sh.d[r], sh.e[r]};
  const bool need = rotate(x, y, s0 + s1, active, tol, cf);
  if (active) {   // the columns change places
    sh.na[left] = y.a;
    sh.na[right] = x.a;
    sh.d[left] = y.d;
    sh.d[right] = x.d;
    sh.e[left] = y.e;
    sh.e[right] = x.e;
  }
  if (kind_b && u == U - 1) {
    if (lane == 63) cf.x = 1.0;
    if (lane == f - 1) cf.y = -1.0;
  }
  return need;
}

template <int RW>
__device__ __forceinline__ void lift(double (&x)[RW], double (&y)[RW], double2 cf) {
#pragma unroll
  for (int i = 0; i < RW; ++i) {
    y[i] = fma(cf.x, x[i], y[i]);
    x[i] = fma(-cf.y, y[i], x[i]);
  }
  __builtin_amdgcn_sched_barrier(0);   // mixed phases take registers that the columns need
}
template <int CTRL, int RW>
__device__ __forceinline__ void move(double (&x)[RW]) {
#pragma unroll
  for (int i = 0; i < RW; ++i) x[i] = dpp_zero<CTRL>(x[i]);
  __builtin_amdgcn_sched_barrier(0);
}
template <int RW>
__device__ __forceinline__ double dot(const double (&x)[RW], const double (&y)[RW]) {
  double s0 = 0.0, s1 = 0.0;
#pragma unroll
  for (int i = 0; i < RW; i += 2) {
    s0 = fma(x[i], y[i], s0);
    if (i + 1 < RW) s1 = fma(x[i + 1], y[i + 1], s1);
  }
  return s0 + s1;
}

// The columns of this lane: v[j][i] is column 2U k + j of row row0 + i (row0
// the same for the whole wave); zero in lanes with k < 0 and beyond nrows.
template <int U, int RW>
__device__ __forceinline__ void load_rows(double (&v)[2 * U][RW], const double* base, int row0, int nrows, int ld,
                                          int k) {
  // addresses and row tests formed here, not kept from or for another call
  asm volatile("" : "+v"(k), "+s"(row0), "+s"(nrows));
  const double* const col = base + 2 * U * max(k, 0);
#pragma unroll
  for (int i = 0; i < RW; ++i) {
    const bool in = k >= 0 && row0 + i < nrows;
    const double* const row = col + (int64_t)min(row0 + i, nrows - 1) * ld;
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const double2 w = *reinterpret_cast<const double2*>(row + 2 * j);
      v[2 * j][i] = in ? w.x : 0.0;
      v[2 * j + 1][i] = in ? w.y : 0.0;
    }
  }
}
// ... and back; reversed: to the mirrored columns.
template <int U, int RW>
__device__ __forceinline__ void store_rows(const double (&v)[2 * U][RW], double* base, int row0, int nrows, int ld,
                                           int k, bool reversed) {
  asm volatile("" : "+v"(k), "+s"(row0), "+s"(nrows));
  if (k < 0) return;
  double* const col = base + (reversed ? ld - 2 * U * (k + 1) : 2 * U * k);
#pragma unroll
  for (int i = 0; i < RW; ++i) {
    if (row0 + i >= nrows) break;
    double* const row = col + (int64_t)(row0 + i) * ld;
#pragma unroll
    for (int j = 0; j < U; ++j) {
      if (reversed)
        *reinterpret_cast<double2*>(row + 2 * (U - 1 - j)) = double2{v[2 * j + 1][i], v[2 * j][i]};
      else
        *reinterpret_cast<double2*>(row + 2 * j) = double2{v[2 * j][i], v[2 * j + 1][i]};
    }
  }
}

// The steps of one (U = 1: A, B) or two (U = 2: A, B, A, B) double steps with
// the columns' roles as they change places; step(u-th pair's x and y, kind).
template <int U, int RW, typename Step>
__device__ __forceinline__ void double_steps(double (&v)[2 * U][RW], Step&& step) {
  if constexpr (U == 1) {
    step(v[0], v[1], v[0], v[1], 0);
    move<kWaveShl1>(v[1]);
    step(v[0], v[1], v[0], v[1], 1);
    move<kWaveShr1>(v[0]);
  } else {
    step(v[0], v[1], v[2], v[3], 0);
    move<kWaveShl1>(v[1]);
    step(v[0], v[3], v[2], v[1], 1);
    move<kWaveShr1>(v[2]);
    step(v[2], v[3], v[0], v[1], 2);
    move<kWaveShl1>(v[3]);
    step(v[2], v[1], v[0], v[3], 3);
    move<kWaveShr1>(v[0]);
  }
}

// `sweeps` logged sweeps on rows row0 .. row0 + RW - 1 of base (one wave).
// Log of a sweep: N steps of U x LL pairs (beta, alpha) of the wave's last LL
// lanes (svd_log_lanes), then N factors.
template <int U, int RW>
__device__ __forceinline__ void apply_log(double* base, int row0, int nrows, int N, int lane, const double* log, int sweeps,
                          bool reversed) {
  const int f = 64 - N / (2 * U), k = lane - f;
  double v[2 * U][RW];
  load_rows<U, RW>(v, base, row0, nrows, N, k);
  const int64_t stride = svd_log_sweep(N, U);
  const int LL = svd_log_lanes(N, U);
  // The log of the next AHEAD groups of 2U steps is in flight: a group takes
  // some 150 cycles, the load several times that.
  constexpr int PER = 2 * U, AHEAD = 4 / U;
  const int groups = N / PER;
  for (int s = 0; s < sweeps; ++s) {
    const double2* const cf = reinterpret_cast<const double2*>(log + s * stride) + max(lane - (64 - LL), 0);
    const double* const fac = log + s * stride + (int64_t)N * U * LL * 2;
    double2 c[AHEAD][PER * U];
#pragma unroll
    for (int a = 0; a < AHEAD; ++a)
#pragma unroll
      for (int q = 0; q < PER * U; ++q) c[a][q] = cf[LL * (min(a, groups - 1) * PER * U + q)];
    for (int g = 0; g < groups; g += AHEAD) {
#pragma unroll
      for (int a = 0; a < AHEAD; ++a) {
        if (g + a >= groups) break;
        double_steps<U, RW>(v, [&](double (&x0)[RW], double (&y0)[RW], double (&x1)[RW], double (&y1)[RW], int w) {
          lift<RW>(x0, y0, c[a][w * U]);
          if constexpr (U == 2) lift<RW>(x1, y1, c[a][w * U + 1]);
        });
        const int next = min(g + a + AHEAD, groups - 1);
#pragma unroll
        for (int q = 0; q < PER * U; ++q) c[a][q] = cf[LL * (next * PER * U + q)];
      }
    }
#pragma unroll
    for (int j = 0; j < 2 * U; ++j) {
      const double dj = k >= 0 ? fac[2 * U * k + j] : 0.0;
#pragma unroll
      for (int i = 0; i < RW; ++i) v[j][i] *= dj;
    }
  }
  store_rows<U, RW>(v, base, row0, nrows, N, k, reversed);
}

// All rows of V by the calling workgroup (rare; apart, for its registers).
template <int U>
__device__ __noinline__ void apply_log_all(double* base, int nrows, int N, const double* log, int sweeps,
                                            int waves) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  nrows = __builtin_amdgcn_readfirstlane(nrows);
  waves = __builtin_amdgcn_readfirstlane(waves);
  for (int q = wave * 4; q < nrows; q += 4 * waves)
    apply_log<U, 4>(base, q, nrows, N, threadIdx.x & 63, log, sweeps, false);
}

// U = 1: every wave forms all parameters for itself from the partial sums
// (one barrier per step), the states in registers beside the columns.  U = 2
// has no registers for that: one wave per pair of a lane forms them, the
// states in LDS, and a second barrier hands them out.
template <int U, int RW, int W>
__device__ __forceinline__ void jacobi_reg(RegShared& sh, double* X, int p, int r, int N, double* log, int logcap,
                                           int32_t* ctrl, int32_t* sweeps, double* sig, double* sorted,
                                           int32_t* perm) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int f = 64 - N / (2 * U), k = lane - f;
  const double tol = uniform(4.0 * DBL_EPSILON * sqrt((double)p));
  double v[2 * U][RW];
  ColState st[2];
  load_rows<U, RW>(v, X, wave * RW, p, N, k);
  // the norms of all columns, from the registers; the factors 1
  auto norms = [&]() {
#pragma unroll
    for (int j = 0; j < 2 * U; ++j) sh.part[wave][j][lane] = dot<RW>(v[j], v[j]);
    __syncthreads();
    if constexpr (U == 1) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < W; ++w) s += sh.part[w][j][lane];
        st[j] = ColState{s, 1.0, 1.0};
      }
    }
    for (int c = tid; c < N; c += 64 * W) {
      double s = 0.0;
      for (int w = 0; w < W; ++w) s += sh.part[w][c % (2 * U)][f + c / (2 * U)];
      sh.na[c] = s;
      sh.d[c] = 1.0;
      sh.e[c] = 1.0;
    }
    __syncthreads();
  };
  int sw = 0, logged = 0, turns = 0;
  const int64_t stride = svd_log_sweep(N, U);
  const int LL = svd_log_lanes(N, U);
  for (; sw < kSvdMaxSweeps && r > 1; ++sw) {
    norms();
    double2* const lg = reinterpret_cast<double2*>(log + logged * stride);
    // this lane's place in it (lanes before the stored ones all write the first one's zeros)
    double2* lw = lg + max(lane - (64 - LL), 0);
    unsigned long long rot = 0ull;   // lanes that rotated
    for (int s0 = 0; s0 < N; s0 += 2 * U) {
      if constexpr (U == 1) {
        // kind A, then B; the partial sums in two places in turn
#pragma unroll
        for (int w = 0; w < 2; ++w) {
          if (w == 1) {
            move<kWaveShl1>(v[1]);
            st[1] = ColState{dpp_zero<kWaveShl1>(st[1].a), dpp_zero<kWaveShl1>(st[1].d),
                             dpp_zero<kWaveShl1>(st[1].e)};
          }
          sh.part[wave][2 + w][lane] = dot<RW>(v[0], v[1]);
          __syncthreads();
          double g0 = 0.0, g1 = 0.0;
#pragma unroll
          for (int i = 0; i < W; i += 2) {
            g0 += sh.part[i][2 + w][lane];
            g1 += sh.part[i + 1][2 + w][lane];
          }
          double2 c;
          rot |= __ballot(rotate(st[0], st[1], g0 + g1, k >= 0 && (w == 0 || lane < 63), tol, c));
          if (w == 1) {
            if (lane == 63) {
              c.x = 1.0;
              st[1] = st[0];
            }
            if (lane == f - 1) {
              c.y = -1.0;
              st[0] = st[1];
            }
          }
          if (wave == W - 1) *lw = c;
          lw += LL;
          lift<RW>(v[0], v[1], c);
          if (w == 1) {
            move<kWaveShr1>(v[0]);
            st[0] = ColState{dpp_zero<kWaveShr1>(st[0].a), dpp_zero<kWaveShr1>(st[0].d),
                             dpp_zero<kWaveShr1>(st[0].e)};
          }
        }
      } else {
        double_steps<U, RW>(v, [&](double (&x0)[RW], double (&y0)[RW], double (&x1)[RW], double (&y1)[RW], int w) {
          const double g0 = dot<RW>(x0, y0), g1 = dot<RW>(x1, y1);
          const int la = fresh_lane();
          sh.part[wave][0][la] = g0;
          sh.part[wave][1][la] = g1;
          __syncthreads();
          if (wave < U) {
            const int lb = fresh_lane();
            double2 c;
            rot |= __ballot(pair_params<U>(sh, wave, lb, f, N, w & 1, tol, c));
            sh.cf[wave][lb] = c;
            (lg + (int64_t)LL * ((s0 + w) * U + wave))[(uint32_t)max(lb - (64 - LL), 0)] = c;
          }
          __syncthreads();
          const int lc = fresh_lane();
          lift<RW>(x0, y0, sh.cf[0][lc]);
          lift<RW>(x1, y1, sh.cf[1][lc]);
        });
      }
    }
    ++turns;   // every sweep reverses the order
    if (wave < U) {
      if (lane == 0) sh.rotated[wave] = rot != 0ull ? 1 : 0;
      if (U == 1 && k >= 0) {
        sh.d[2 * k] = st[0].d;
        sh.d[2 * k + 1] = st[1].d;
      }
    }
    __syncthreads();
    const bool again = sh.rotated[0] || (U == 2 && sh.rotated[1]);
    if (!again) break;
    for (int c = tid; c < N; c += 64 * W) log[logged * stride + (int64_t)N * U * LL * 2 + c] = sh.d[c];
#pragma unroll
    for (int j = 0; j < 2 * U; ++j) {
      const double dj = k >= 0 ? sh.d[2 * U * k + j] : 0.0;
#pragma unroll
      for (int i = 0; i < RW; ++i) v[j][i] *= dj;
    }
    ++logged;
    __syncthreads();
    if (logged == logcap && sw + 1 < kSvdMaxSweeps) {
      // the log is full: this workgroup brings V up to date itself
      store_rows<U, RW>(v, X, wave * RW, p, N, k, false);
      __threadfence_block();
      __syncthreads();
      apply_log_all<U>(X + (int64_t)p * N, r, N, log, logged, W);
      logged = 0;
      __syncthreads();
      load_rows<U, RW>(v, X, wave * RW, p, N, k);
    }
  }
  norms();
  const int ex = __builtin_amdgcn_readfirstlane(ctrl[2]);   // X back to its own scale
  if (ex != 0) {
#pragma unroll
    for (int j = 0; j < 2 * U; ++j)
#pragma unroll
      for (int i = 0; i < RW; ++i) v[j][i] = ldexp(v[j][i], ex);
  }
  store_rows<U, RW>(v, X, wave * RW, p, N, k, false);
  // zero columns that only pad: r .. N - 1 at the start, mirrored with every sweep
  const int pad = N - r, lo = turns & 1 ? pad : 0, hi = turns & 1 ? N : r;
  double* const sg = &sh.part[0][0][0];
  for (int c = tid; c < N; c += 64 * W) sg[c] = sqrt(sh.na[c]);
  __syncthreads();
  for (int c = lo + tid; c < hi; c += 64 * W) {
    const unsigned long long key = order_key(sg[c]);
    int rank = 0;
    for (int i = lo; i < hi; ++i) {
      const unsigned long long w = order_key(sg[i]);
      rank += (w > key || (w == key && i < c)) ? 1 : 0;
    }
    perm[rank] = c;
    sorted[rank] = sig[c - lo] = ldexp(sg[c], ex);
  }
  if (tid == 0) {
    *sweeps = sw;
    ctrl[0] = logged;
    ctrl[1] = turns > sw ? 1 : 0;   // the last sweep, without rotations, is not in the log
  }
}

}  // namespace

__global__ __launch_bounds__(64 * kSvdRegWaves) void svd_reg_kernel(const SvdSec* __restrict__ secs,
                                                                   const int32_t* __restrict__ list, double* D,
                                                                   double* scratch, int logcap, int32_t* ctrl,
                                                                   int32_t* sweeps, double* sig, double* sorted,
                                                                   int32_t* perm) {
  __shared__ RegShared sh;
  const int id = list[blockIdx.x];
  const SvdSec S = secs[id];
  const int p = S.m >= S.n ? S.m : S.n, r = S.m >= S.n ? S.n : S.m;
  double* const X = D + S.x_off;
  double* const log = scratch + S.log_off;
  auto go = [&](auto u, auto rw, auto w) {
    constexpr int W = decltype(w)::value;
    if (W < kSvdRegWaves && threadIdx.x >= 64 * W) return;
    jacobi_reg<decltype(u)::value, decltype(rw)::value, W>(sh, X, p, r, S.ld, log, logcap, ctrl + kSvdCtrl * blockIdx.x,
                                                           sweeps + id, sig + S.s_off, sorted + S.s_off,
                                                           perm + S.s_off);
  };
  using std::integral_constant;
  const integral_constant<int, 1> one;
  const integral_constant<int, 2> two;
  const integral_constant<int, 4> w4;
  const integral_constant<int, 8> w8;
  if (S.pairs == 1) {
    // four waves, one per SIMD, while the rows fit: a step is bound by its
    // chain, which more waves of a SIMD would share its cycles with
    if (p <= 32) go(one, integral_constant<int, 8>(), w4);
    else if (p <= 64) go(one, integral_constant<int, 16>(), w4);
    else if (p <= 128) go(one, integral_constant<int, 32>(), w4);
    else go(one, integral_constant<int, 32>(), w8);
  } else {
    if (p <= 160) go(two, integral_constant<int, 20>(), w8);
    else go(two, integral_constant<int, 26>(), w8);
  }
}

constexpr int kSvdApplyRows = 2;
// The logged rotations on the rows of V, two rows per wave.  Bound: latency
// of a step (two dependent products and a move), hidden by the other waves of
// the SIMD; the log is read once per wave, from L2: with 4, 2 and 1 rows a wave
// 160, 128 and 188 us at chi = 1024, 31, 27 and 26 us at chi = 256 (a log of 64
// lanes per step; of those with columns 143 and 27 us, 2 rows a wave).
__global__ __launch_bounds__(256) void svd_apply_kernel(const SvdSec* __restrict__ secs,
                                                        const int32_t* __restrict__ list, double* D,
                                                        const double* scratch, const int32_t* __restrict__ ctrl) {
  const SvdSec S = secs[list[blockIdx.y]];
  const int p = S.m >= S.n ? S.m : S.n, r = S.m >= S.n ? S.n : S.m;
  const int lane = threadIdx.x & 63, q = (blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * kSvdApplyRows;
  if (q >= r) return;
  double* const V = D + S.x_off + (int64_t)p * S.ld;
  const double* const log = scratch + S.log_off;
  const int sweeps = ctrl[kSvdCtrl * blockIdx.y];
  const bool rev = ctrl[kSvdCtrl * blockIdx.y + 1] != 0;
  if (S.pairs == 1)
    apply_log<1, kSvdApplyRows>(V, q, r, S.ld, lane, log, sweeps, rev);
  else
    apply_log<2, kSvdApplyRows>(V, q, r, S.ld, lane, log, sweeps, rev);
}

hipError_t launch_svd_reg(const SvdLaunch& l, hipStream_t s) {
  if (l.logcap < 1) return hipErrorInvalidValue;
  // a grid's second dimension holds 65535 sectors
  for (int32_t k = 0; k < l.nreg; k += 65535) {
    const unsigned n = (unsigned)std::min(l.nreg - k, 65535);
    const int32_t* const list = l.reg + k;
    int32_t* const ctrl = l.ctrl + (int64_t)kSvdCtrl * k;
    const unsigned trail = (unsigned)((l.trail_rows + kSvdTrailRows - 1) / kSvdTrailRows);
    const unsigned apply = (unsigned)((l.reg_cols + 4 * kSvdApplyRows - 1) / (4 * kSvdApplyRows));
    for (int q = 0; q < l.panels; ++q) {
      hipLaunchKernelGGL(svd_panel_kernel, dim3(n), dim3(1024), 0, s, l.secs, list, l.X, l.scratch, l.rowpos, ctrl, q);
      if (trail > 0)
        hipLaunchKernelGGL(svd_trail_kernel, dim3(trail, n), dim3(256), 0, s, l.secs, list, l.X, l.scratch, l.rowpos,
                           ctrl, q);
    }
    hipLaunchKernelGGL(svd_reg_kernel, dim3(n), dim3(64 * kSvdRegWaves), 0, s, l.secs, list, l.X, l.scratch, l.logcap,
                       ctrl, l.sweeps, l.sig, l.sorted, l.perm);
    hipLaunchKernelGGL(svd_apply_kernel, dim3(apply, n), dim3(256), 0, s, l.secs, list, l.X, l.scratch, ctrl);
  }
  return hipGetLastError();
}

}  // namespace bst

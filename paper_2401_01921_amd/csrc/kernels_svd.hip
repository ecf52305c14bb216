// Symmetric SVD kernels (Sec. "Singular value decomposition"): the block
// matrices of every charge sector are gathered into the tall orientation X,
// each sector's SVD runs as one-sided Jacobi (Hestenes), the truncation is
// selected across all sectors by one workgroup, and the kept columns are
// written into the block layouts of U and V^dagger.  Sectors that fit a
// workgroup's registers are rotated in kernels_svd_reg.hip; here are the paths
// of the others.
//
// One-sided Jacobi: for a pair of columns (x_i, x_j) with a = |x_i|^2,
// b = |x_j|^2, g = x_i.x_j, the plane rotation
//   x_i <- c x_i - s x_j,  x_j <- s x_i + c x_j,
//   t = s / c the root of smaller magnitude of t^2 + 2 zeta t - 1 = 0,
//   zeta = (b - a) / (2 g),
// makes the two columns orthogonal; the same rotation applied to the
// columns of Vh (starting from the identity) accumulates X_0 Vh = X.  Sweeps
// visit every pair once in the round-robin (circle) order, all pairs of a
// round at once (one lane group each, disjoint columns); they stop after a sweep
// without a rotation (|g| <= tol sqrt(a b)).  Then sigma_j = |x_j|.  The
// arithmetic of every pair is a fixed sequence, so results repeat bit for
// bit.  A sector whose X does not fit LDS would pull every round's columns
// through one CU's L2; such sectors instead run a round per launch, each
// pair of the round on a workgroup of its own (svd_round_kernel).
#include <algorithm>
#include <cfloat>
#include <type_traits>

#include "plan.h"

#include "svd.h"

namespace bst {

namespace {
__device__ __forceinline__ double wave_allsum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}
}  // namespace

__global__ __launch_bounds__(256) void svd_gather_kernel(const SvdGather* __restrict__ jobs,
                                                         const SvdWork* __restrict__ work,
                                                         const double* __restrict__ in, double* __restrict__ X,
                                                         double* __restrict__ scratch) {
  const SvdWork w = work[blockIdx.x];
  const SvdGather j = jobs[w.job];
  double* const out = (j.scratch ? scratch : X) + j.x_off;
  const int64_t total = (int64_t)j.rows * j.cols;
  for (int e = threadIdx.x; e < kSvdGatherChunk; e += 256) {
    const int64_t idx = (int64_t)w.start + e;
    if (idx >= total) break;
    const int64_t r = idx / j.cols, c = idx % j.cols;
    out[(j.row0 + r) * j.rs + (j.col0 + c) * j.cs] = in[j.in_off + idx];
  }
}

#define BST_LDS __attribute__((address_space(3)))

// Sum over groups of LP lanes (LP = 32, 64; every lane of a group gets the
// same value).
template <int LP>
__device__ __forceinline__ double group_allsum(double v) {
#pragma unroll
  for (int off = LP / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, LP);
  return v;
}

// The sweeps of one sector on X (p x r, column-major, in LDS) and Vh (r x r):
// PV is a pointer to global memory or, where Vh is held in LDS too, an
// LDS-addressed one (so that the compiler issues LDS accesses, not generic
// ones).  One group of LP lanes per pair of a round.  Returns the sweeps used.
template <int LP, typename PV>
__device__ int jacobi_sweeps(BST_LDS double* x, PV vh, int p, int r, int* rotated) {
  constexpr int NH = 64 * kSvdWaves / LP;   // lane groups of the workgroup
  const int tid = threadIdx.x, hl = tid % LP, half = tid / LP;
  const double tol = 4.0 * DBL_EPSILON * sqrt((double)p);
  const int rr = r + (r & 1);   // an odd count gets one idle slot
  int sw = 0;
  for (; sw < kSvdMaxSweeps && r > 1; ++sw) {
    for (int t = 0; t < rr - 1; ++t) {
      for (int k = half; k < rr / 2; k += NH) {
        // circle method: slot 0 stays, the others advance by one per round
        const int s0 = k, s1 = rr - 1 - k;
        int i = s0 == 0 ? 0 : (s0 - 1 + t) % (rr - 1) + 1;
        int j = (s1 - 1 + t) % (rr - 1) + 1;
        if (i > j) {
          const int q = i;
          i = j;
          j = q;
        }
        if (j >= r) continue;
        BST_LDS double* xi = x + (int64_t)i * p;
        BST_LDS double* xj = x + (int64_t)j * p;
        double a = 0.0, b = 0.0, g = 0.0;
        for (int e = hl; e < p; e += LP) {
          const double u = xi[e], v = xj[e];
          a += u * u;
          b += v * v;
          g += u * v;
        }
        a = group_allsum<LP>(a);
        b = group_allsum<LP>(b);
        g = group_allsum<LP>(g);
        if (a == 0.0 || b == 0.0 || !(fabs(g) > tol * sqrt(a) * sqrt(b))) continue;
        const double zeta = (b - a) / (2.0 * g);
        const double tt = (zeta >= 0.0 ? 1.0 : -1.0) / (fabs(zeta) + sqrt(1.0 + zeta * zeta));
        const double c = 1.0 / sqrt(1.0 + tt * tt), s = c * tt;
        for (int e = hl; e < p; e += LP) {
          const double u = xi[e], v = xj[e];
          xi[e] = c * u - s * v;
          xj[e] = s * u + c * v;
        }
        PV vi = vh + (int64_t)i * r;
        PV vj = vh + (int64_t)j * r;
        for (int e = hl; e < r; e += LP) {
          const double u = vi[e], v = vj[e];
          vi[e] = c * u - s * v;
          vj[e] = s * u + c * v;
        }
        if (hl == 0) *rotated = 1;
      }
      __syncthreads();
    }
    const bool done = *rotated == 0;
    __syncthreads();
    if (tid == 0) *rotated = 0;
    __syncthreads();
    if (done) break;
  }
  return sw;
}

__global__ __launch_bounds__(64 * kSvdWaves) void svd_jacobi_kernel(const SvdSec* __restrict__ secs, double* X,
                                                                   double* __restrict__ sig,
                                                                   double* __restrict__ sorted,
                                                                   int32_t* __restrict__ perm,
                                                                   int32_t* __restrict__ sweeps, int path) {
  constexpr int NT = 64 * kSvdWaves;
  const SvdSec S = secs[blockIdx.x];
  const int p = S.m >= S.n ? S.m : S.n, r = S.m >= S.n ? S.n : S.m;
  // the sectors that fit LDS (their sweeps), or the big ones (sigma and order
  // after their rounds)
  if (S.path != path) return;
  double* const xg = X + S.x_off;
  double* const vg = X + S.v_off;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  __shared__ int rotated;
  // X is rotated in LDS, and Vh with it when both fit; else Vh works in global
  // memory (the three dots of a pair read X only, so X in LDS keeps them off
  // global latency).  Copied back at the end.  X of a big sector, and a single
  // column, which is not rotated, may be larger and stay where they are.
  __shared__ double lds[kSvdLdsBytes / sizeof(double)];
  const bool x_lds = (int64_t)p * r * (int64_t)sizeof(double) <= kSvdLdsBytes;
  const bool v_lds = x_lds && ((int64_t)p * r + (int64_t)r * r) * (int64_t)sizeof(double) <= kSvdLdsBytes;
  BST_LDS double* xl = (BST_LDS double*)lds;
  BST_LDS double* vl = xl + (int64_t)p * r;
  // a big sector arrives rotated (svd_round_kernel), its sweeps counted
  const bool pre = path == kSvdPathRounds;
  if (x_lds)
    for (int64_t e = tid; e < (int64_t)p * r; e += NT) xl[e] = xg[e];
  if (v_lds)
    for (int64_t e = tid; e < (int64_t)r * r; e += NT) vl[e] = (e % r == e / r) ? 1.0 : 0.0;
  else if (!pre)
    for (int64_t e = tid; e < (int64_t)r * r; e += NT) vg[e] = (e % r == e / r) ? 1.0 : 0.0;
  if (tid == 0) rotated = 0;
  __syncthreads();
  // the widest lane groups that still give every pair of a round its own group:
  // 32 lanes do for all, as X has more rows than the register path takes
  static_assert(kSvdLdsBytes / 8 / (kSvdRegMaxRows + 1) <= 2 * (NT / 32), "pairs of a round");
  const int npairs = (r + 1) / 2;
  int sw = 0;
  if (pre)
    sw = sweeps[blockIdx.x];
  else if (npairs <= NT / 64)
    sw = v_lds ? jacobi_sweeps<64>(xl, vl, p, r, &rotated) : jacobi_sweeps<64>(xl, vg, p, r, &rotated);
  else
    sw = v_lds ? jacobi_sweeps<32>(xl, vl, p, r, &rotated) : jacobi_sweeps<32>(xl, vg, p, r, &rotated);
  // sigma_j = |x_j| (one column per wave), from where the sweeps left X
  for (int j = wave; j < r; j += kSvdWaves) {
    double a = 0.0;
    if (x_lds) {
      for (int e = lane; e < p; e += 64) a += xl[(int64_t)j * p + e] * xl[(int64_t)j * p + e];
    } else {
      for (int e = lane; e < p; e += 64) a += xg[(int64_t)j * p + e] * xg[(int64_t)j * p + e];
    }
    a = wave_allsum(a);
    if (lane == 0) sig[S.s_off + j] = sqrt(a);
  }
  if (x_lds)
    for (int64_t e = tid; e < (int64_t)p * r; e += NT) xg[e] = xl[e];
  if (v_lds)
    for (int64_t e = tid; e < (int64_t)r * r; e += NT) vg[e] = vl[e];
  __syncthreads();
  // descending order, ties by column: rank of every value
  for (int j = tid; j < r; j += NT) {
    const double v = sig[S.s_off + j];
    int rank = 0;
    for (int i = 0; i < r; ++i) {
      const double w = sig[S.s_off + i];
      rank += (w > v || (w == v && i < j)) ? 1 : 0;
    }
    perm[S.s_off + rank] = j;
    sorted[S.s_off + rank] = v;
  }
  if (tid == 0) sweeps[blockIdx.x] = sw;
}

// Rounds of the big sectors, a launch per round.  Block (k, b) takes pair k
// of round t of big sector b (the circle order of jacobi_sweeps) with 256
// lanes: the three sums over the column (lane-strided, then the wave sums
// and the four waves in order), the same test and rotation, both columns of
// X and of Vh updated.  Any rotation sets the sector's flag for the sweep.
__global__ __launch_bounds__(256) void svd_round_kernel(const SvdSec* __restrict__ secs,
                                                        const int32_t* __restrict__ big, double* X, int t,
                                                        int32_t* flags) {
  const int b = blockIdx.y;
  if (flags[2 * b + 1]) return;   // converged
  const SvdSec S = secs[big[b]];
  const int p = S.m >= S.n ? S.m : S.n, r = S.m >= S.n ? S.n : S.m;
  const int rr = r + (r & 1);
  const int k = blockIdx.x;
  if (t >= rr - 1 || k >= rr / 2) return;
  const int s0 = k, s1 = rr - 1 - k;
  int i = s0 == 0 ? 0 : (s0 - 1 + t) % (rr - 1) + 1;
  int j = (s1 - 1 + t) % (rr - 1) + 1;
  if (i > j) {
    const int q = i;
    i = j;
    j = q;
  }
  if (j >= r) return;
  double* const xi = X + S.x_off + (int64_t)i * p;
  double* const xj = X + S.x_off + (int64_t)j * p;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double a = 0.0, bb = 0.0, g = 0.0;
  for (int e = tid; e < p; e += 256) {
    const double u = xi[e], v = xj[e];
    a += u * u;
    bb += v * v;
    g += u * v;
  }
  a = wave_allsum(a);
  bb = wave_allsum(bb);
  g = wave_allsum(g);
  __shared__ double red[3][4];
  if (lane == 0) {
    red[0][wave] = a;
    red[1][wave] = bb;
    red[2][wave] = g;
  }
  __syncthreads();
  a = ((red[0][0] + red[0][1]) + red[0][2]) + red[0][3];
  bb = ((red[1][0] + red[1][1]) + red[1][2]) + red[1][3];
  g = ((red[2][0] + red[2][1]) + red[2][2]) + red[2][3];
  const double tol = 4.0 * DBL_EPSILON * sqrt((double)p);
  if (a == 0.0 || bb == 0.0 || !(fabs(g) > tol * sqrt(a) * sqrt(bb))) return;
  const double zeta = (bb - a) / (2.0 * g);
  const double tt = (zeta >= 0.0 ? 1.0 : -1.0) / (fabs(zeta) + sqrt(1.0 + zeta * zeta));
  const double c = 1.0 / sqrt(1.0 + tt * tt), sn = c * tt;
  for (int e = tid; e < p; e += 256) {
    const double u = xi[e], v = xj[e];
    xi[e] = c * u - sn * v;
    xj[e] = sn * u + c * v;
  }
  double* const vi = X + S.v_off + (int64_t)i * r;
  double* const vj = X + S.v_off + (int64_t)j * r;
  for (int e = tid; e < r; e += 256) {
    const double u = vi[e], v = vj[e];
    vi[e] = c * u - sn * v;
    vj[e] = sn * u + c * v;
  }
  if (tid == 0) flags[2 * b] = 1;
}

// Identity Vh and cleared flags and counts of the big sectors (grid y: the
// sector, x: pieces of its r x r).
__global__ __launch_bounds__(256) void svd_big_init_kernel(const SvdSec* __restrict__ secs,
                                                           const int32_t* __restrict__ big, double* V,
                                                           int32_t* flags, int32_t* sweeps) {
  const int b = blockIdx.y;
  const SvdSec S = secs[big[b]];
  const int64_t r = S.m >= S.n ? S.n : S.m;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < r * r; e += (int64_t)gridDim.x * 256)
    V[S.v_off + e] = (e % r == e / r) ? 1.0 : 0.0;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    flags[2 * b] = 0;
    flags[2 * b + 1] = 0;
    sweeps[big[b]] = 0;
  }
}

// End of a sweep of the big sectors: a sector that rotated counts the
// sweep, one that did not is converged (as jacobi_sweeps stops).
__global__ __launch_bounds__(256) void svd_sweep_end_kernel(int nbig, const int32_t* __restrict__ big,
                                                            int32_t* flags, int32_t* sweeps) {
  for (int b = blockIdx.x * 256 + threadIdx.x; b < nbig; b += gridDim.x * 256) {
    if (!flags[2 * b + 1]) {
      if (flags[2 * b])
        sweeps[big[b]] += 1;
      else
        flags[2 * b + 1] = 1;
    }
    flags[2 * b] = 0;
  }
}

hipError_t launch_svd_gather(const SvdLaunch& l, hipStream_t s) {
  if (l.ngwork > 0x7FFFFFFF || l.nsec < 0 || l.nbig < 0 || l.nbig > 65535) return hipErrorInvalidValue;
  if (l.ngwork > 0)
    hipLaunchKernelGGL(svd_gather_kernel, dim3((unsigned)l.ngwork), dim3(256), 0, s, l.gjobs, l.gwork, l.in, l.X,
                       l.scratch);
  if (l.nbig > 0) {
    const int64_t gx = std::min<int64_t>(std::max<int64_t>((l.vmax + 4095) / 4096, 1), 1024);
    hipLaunchKernelGGL(svd_big_init_kernel, dim3((unsigned)gx, (unsigned)l.nbig), dim3(256), 0, s, l.secs, l.big,
                       l.X, l.flags, l.sweeps);
  }
  return hipGetLastError();
}

hipError_t launch_svd_sweep(const SvdLaunch& l, hipStream_t s) {
  if (l.nbig <= 0) return hipSuccess;
  if (l.nbig > 65535 || l.pairs <= 0 || l.rounds <= 0) return hipErrorInvalidValue;
  for (int t = 0; t < l.rounds; ++t)
    hipLaunchKernelGGL(svd_round_kernel, dim3((unsigned)l.pairs, (unsigned)l.nbig), dim3(256), 0, s, l.secs, l.big,
                       l.X, t, l.flags);
  hipLaunchKernelGGL(svd_sweep_end_kernel, dim3((unsigned)((l.nbig + 255) / 256)), dim3(256), 0, s, l.nbig, l.big,
                     l.flags, l.sweeps);
  return hipGetLastError();
}

hipError_t launch_svd_finish(const SvdLaunch& l, hipStream_t s, int path) {
  if (l.nsec < 0 || (path != kSvdPathLds && path != kSvdPathRounds)) return hipErrorInvalidValue;
  if (l.nsec > 0)
    hipLaunchKernelGGL(svd_jacobi_kernel, dim3((unsigned)l.nsec), dim3(64 * kSvdWaves), 0, s, l.secs, l.X,
                       l.sig, l.sorted, l.perm, l.sweeps, path);
  return hipGetLastError();
}

// ------------------------------------------------------------------------
// Truncation across sectors (one workgroup).  Every sector first keeps its
// min_blockdim largest values; the other values not below err are the
// candidates, ordered by value (descending), then sector, then position; the
// first keepdim - (forced) of them are kept.  The cut is found on the bit
// pattern of the values (non-negative doubles order like their bits), four
// bits at a time: each wave counts the candidates not below one of the 16
// next digits, and a sector's count is a binary search, since its values are
// sorted.  It is found when exactly the wanted number lie at or above it;
// where equal values leave no such cut, the last of them go by sector.
//
// Bound: latency, a round is one search in LDS and a barrier.  A two-site
// state at chi = 256 (15 sectors, 510 values): 292 us with a scan of all values
// for each bit, now 12 us.
// ------------------------------------------------------------------------
constexpr int kSelectMaxSectors = 4096;
constexpr int kSelectLdsValues = 8192;   // values staged in LDS when they all fit

__global__ __launch_bounds__(1024) void svd_select_kernel(const SvdSec* __restrict__ secs, int nsec,
                                                         const double* __restrict__ sorted,
                                                         const int64_t* __restrict__ min_blockdim,
                                                         int64_t keepdim, double err, int64_t* __restrict__ kept,
                                                         double* __restrict__ s_err) {
  constexpr unsigned long long kInf = 0x7FF0000000000000ull;
  __shared__ double vals[kSelectLdsValues];
  // per sector: value offset (below 2^31: the plan refuses more values), the
  // candidates' range of positions, forced count, values equal to the cut
  __shared__ int soff[kSelectMaxSectors], base[kSelectMaxSectors], cap[kSelectMaxSectors], cnt[kSelectMaxSectors];
  __shared__ long long red[17];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  auto rank_of = [&](int q) {
    const SvdSec& S = secs[q];
    return S.m < S.n ? S.m : S.n;
  };
  auto forced = [&](int q, int r) -> int {
    const int64_t f = min_blockdim ? min_blockdim[q] : 0;
    return (int)(f < 0 ? 0 : (f < r ? f : r));
  };
  const long long total = secs[nsec - 1].s_off + rank_of(nsec - 1);
  const bool staged = total <= kSelectLdsValues;
  if (staged)
    for (int e = tid; e < total; e += 1024) vals[e] = sorted[e];
  for (int q = tid; q < nsec; q += 1024) {
    soff[q] = (int)secs[q].s_off;
    cap[q] = rank_of(q);
  }
  __syncthreads();
  // entries of sector q in [lo, hi) whose bits are t or more: a prefix
  auto search = [](const auto* v, int lo, int hi, unsigned long long t) {
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      const double x = v[mid];
      if (((unsigned long long)__double_as_longlong(x) & 0x7FFFFFFFFFFFFFFFull) >= t) lo = mid + 1;
      else hi = mid;
    }
    return lo;
  };
  auto prefix = [&](int q, int lo, int hi, unsigned long long t) {
    return staged ? search((const BST_LDS double*)vals + soff[q], lo, hi, t) : search(sorted + soff[q], lo, hi, t);
  };
  // sum over the wave (the values' count is below 2^31)
  auto wave_total = [&](int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x128, 0xF, 0xF, true);   // rotations by 8, 4, 2, 1 within 16 lanes
    v += __builtin_amdgcn_update_dpp(0, v, 0x124, 0xF, 0xF, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x122, 0xF, 0xF, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x121, 0xF, 0xF, true);
    return __builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16) + __builtin_amdgcn_readlane(v, 32) +
           __builtin_amdgcn_readlane(v, 48);
  };
  // sums over all threads
  auto block_total = [&](int n) {
    const long long v = wave_total(n);
    __syncthreads();
    if (lane == 0) red[wave] = v;
    __syncthreads();
    long long t = 0;
    for (int w = 0; w < 16; ++w) t += red[w];
    return t;
  };
  // candidates: after the forced values (and any NaN, sorted first), down to err
  int f_mine = 0, c_mine = 0;
  const unsigned long long ebits = (unsigned long long)__double_as_longlong(err + 0.0) & 0x7FFFFFFFFFFFFFFFull;
  for (int q = tid; q < nsec; q += 1024) {
    const int r = cap[q], f = forced(q, r);
    const int b = max(f, prefix(q, 0, r, kInf + 1));
    const int c = max(b, prefix(q, b, r, ebits));
    base[q] = b;
    cap[q] = c;
    cnt[q] = 0;
    f_mine += f;
    c_mine += c - b;
  }
  const long long room = keepdim - block_total(f_mine);
  const long long ncand = block_total(c_mine);
  const bool all = room >= ncand, none = room <= 0;
  // the room-th largest candidate: the largest t with count(t) >= room
  auto count = [&](unsigned long long t) {   // by one wave
    int c = 0;
    for (int q = lane; q < nsec; q += 64) c += prefix(q, base[q], cap[q], t) - base[q];
    return wave_total(c);
  };
  unsigned long long cut = 0ull;
  bool exact = false;   // count(cut) == room
  if (!all && !none) {
    for (int shift = 60; shift >= 0 && !exact; shift -= 4) {
      const long long c = count(cut | ((unsigned long long)wave << shift));
      __syncthreads();
      if (lane == 0) red[wave] = c;
      __syncthreads();
      int d = 0;   // the counts fall with the digit; that of 0 is room or more
      for (int w = 1; w < 16; ++w) d = red[w] >= room ? w : d;
      cut |= (unsigned long long)d << shift;
      exact = red[d] == room;
    }
    __syncthreads();
  }
  if (!all && !none && !exact) {
    if (wave == 0) {
      const long long c = count(cut + 1);
      if (lane == 0) red[16] = room - c;
    }
    __syncthreads();
    for (int q = tid; q < nsec; q += 1024) {
      const int gt = prefix(q, base[q], cap[q], cut + 1), ge = prefix(q, base[q], cap[q], cut);
      cnt[q] = ge - gt;
    }
    __syncthreads();
    if (tid == 0) {
      long long need = red[16];   // of the values equal to the cut
      for (int q = 0; q < nsec; ++q) {
        cnt[q] = (int)(cnt[q] < need ? cnt[q] : need);
        need -= cnt[q];
      }
    }
    __syncthreads();
  }
  double e = 0.0;
  for (int q = tid; q < nsec; q += 1024) {
    const int r = rank_of(q), f = forced(q, r);
    int k = f;
    if (all) k = f + cap[q] - base[q];
    else if (!none) k = f + prefix(q, base[q], cap[q], exact ? cut : cut + 1) - base[q] + cnt[q];
    kept[q] = k;
    if (k < r) e = fmax(e, sorted[soff[q] + k]);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) e = fmax(e, __shfl_xor(e, off, 64));
  __syncthreads();
  double* const re = reinterpret_cast<double*>(red);
  if (lane == 0) re[wave] = e;
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < 16; ++w) e = fmax(e, re[w]);
    *s_err = e;
  }
}

hipError_t launch_svd_select(const SvdSelectLaunch& l, hipStream_t s) {
  if (l.nsec < 0 || l.nsec > kSelectMaxSectors) return hipErrorInvalidValue;
  hipLaunchKernelGGL(svd_select_kernel, dim3(1), dim3(1024), 0, s, l.secs, l.nsec, l.sorted, l.min_blockdim,
                     l.keepdim, l.err, l.kept, l.s_err);
  return hipGetLastError();
}

// ------------------------------------------------------------------------
// Kept columns into the output factors
// ------------------------------------------------------------------------
__global__ __launch_bounds__(256) void svd_write_kernel(const SvdWrite* __restrict__ jobs,
                                                        const SvdWriteWork* __restrict__ work,
                                                        const SvdSec* __restrict__ secs, const double* __restrict__ X,
                                                        const int32_t* __restrict__ rowpos,
                                                        const double* __restrict__ sorted,
                                                        const int32_t* __restrict__ perm, int absorb, double* U,
                                                        double* Vd, double* Sv) {
  const SvdWriteWork w = work[blockIdx.x];
  const SvdWrite j = jobs[w.job];
  const SvdSec S = secs[j.sec];
  const bool tall = S.m >= S.n;
  const int64_t total = j.kind == 2 ? j.k : (int64_t)j.ext * j.k;
  for (int e = threadIdx.x; e < kSvdGatherChunk; e += 256) {
    const int64_t idx = (int64_t)w.start + e;
    if (idx >= total) break;
    if (j.kind == 2) {
      Sv[j.out_off + idx] = sorted[S.s_off + idx];
      continue;
    }
    // U: (row, c) = (idx / k, idx % k); V^dagger: (c, col) = (idx / ext, idx % ext)
    const int64_t c = j.kind == 0 ? idx % j.k : idx / j.ext;
    const int64_t row = j.off0 + (j.kind == 0 ? idx / j.k : idx % j.ext);
    const int64_t col = perm[S.s_off + c];
    const double sg = sorted[S.s_off + c];
    // U = x_j / sigma_j (tall) or Vh (wide); V = Vh (tall) or x_j / sigma_j (wide)
    const bool from_x = (j.kind == 0) == tall;
    double v;
    if (from_x) {
      const int64_t xr = S.path == kSvdPathReg ? rowpos[S.p_off + row] : row;
      v = sg > 0.0 ? X[S.x_off + xr * S.x_rs + col * S.x_cs] / sg : 0.0;
    } else {
      v = X[S.v_off + row * S.v_rs + col * S.v_cs];
    }
    if ((j.kind == 0 && absorb == 1) || (j.kind == 1 && absorb == 2)) v *= sg;
    (j.kind == 0 ? U : Vd)[j.out_off + idx] = v;
  }
}

hipError_t launch_svd_write(const SvdWriteLaunch& l, hipStream_t s) {
  if (l.nwork <= 0) return hipSuccess;
  if (l.nwork > 0x7FFFFFFF) return hipErrorInvalidValue;
  hipLaunchKernelGGL(svd_write_kernel, dim3((unsigned)l.nwork), dim3(256), 0, s, l.jobs, l.work, l.secs, l.X, l.rowpos,
                     l.sorted, l.perm, l.absorb, l.U, l.Vd, l.S);
  return hipGetLastError();
}

}  // namespace bst

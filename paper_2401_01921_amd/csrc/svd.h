// Symmetric SVD (Sec. "Singular value decomposition"): device records shared
// by the host plan (svd.cpp) and the kernels (kernels_svd.hip).
//
// A tensor seen as a matrix (first rowrank legs = rows) splits into one block
// matrix M_q per charge q of the new bond.  Each M_q (m x n) is held in the
// workspace as X, the "tall" orientation (p x r, p = max(m, n), r = min(m, n)):
// X = M_q when m >= n, X = M_q^T otherwise.  One-sided Jacobi rotates the
// columns of X until they are orthogonal and accumulates the rotations in Vh
// (r x r); then sigma_j = |x_j|, and
//   tall: U = x_j / sigma_j, V = Vh;      wide: U = Vh, V = x_j / sigma_j.
// Three paths do the sweeps; a sector's size chooses one (svd_path).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace bst {

// One block of the input, copied into its sector's matrix: element (R, C) of
// M_q goes to x_off + R * rs + C * cs of the X region, or of the scratch
// region (register path: the rows are ordered on the way into X).
struct SvdGather {
  int64_t in_off;   // element offset of the block in the input tensor
  int64_t x_off;
  int32_t rows, cols;   // the block as a matrix: row-leg extent x column-leg extent
  int32_t row0, col0;   // its place in M_q
  int32_t rs, cs;
  int32_t scratch, pad;
};
struct SvdWork {
  int32_t job, start;   // 256 * 16 elements of one job per workgroup
};

// One sector matrix.  Element (row, col) of X is at x_off + row * x_rs + col *
// x_cs, of Vh at v_off + row * v_rs + col * v_cs (both in the X region; on the
// register path row is a sorted place, rowpos[p_off + row]).
struct SvdSec {
  int64_t x_off, v_off;
  int64_t s_off;    // r values in the sigma / sorted / perm regions
  int64_t log_off;  // register path: gathered X and reflections, then the rotation log
  int64_t p_off;    // register path: row order (p places, then their inverse), then column order (r)
  int32_t m, n;
  int32_t x_rs, x_cs, v_rs, v_cs;
  int32_t path;     // SvdPath
  int32_t ld;       // register path: padded column count N, the row stride
  int32_t nb;       // ... reflections per panel (r or more: all in one launch)
  int32_t pairs;    // ... column pairs per lane (U)
};

// One block of an output factor, written from its sector's X and Vh.
// kind 0: U block [row tuple..., k] (row-major as [ext x k]) from rows
// off0 .. off0 + ext of U_q; kind 1: V^dagger block [k, column tuple...]
// (row-major as [k x ext]) from rows off0 .. of V_q; kind 2: the k largest
// values of the sector into S (ext = k).
struct SvdWrite {
  int64_t out_off;
  int32_t sec, kind;
  int32_t off0, ext;
  int32_t k, pad;
};
struct SvdWriteWork {
  int32_t job, start;
};

constexpr int kSvdWaves = 16;             // waves of the Jacobi workgroup
constexpr int kSvdLdsBytes = 128 * 1024;  // X and Vh of a sector up to this size are rotated in LDS
constexpr int kSvdMaxSweeps = 60;

// Register path (kernels_svd_reg.hip): X in the registers of one workgroup of
// 8 waves, which may hold 256 registers per lane at that occupancy.  One
// column pair per lane (63 lanes at most) takes 32 rows per wave, two pairs 26.
constexpr int kSvdRegWaves = 8;
constexpr int kSvdRegMaxCols = 256;        // array sizes; 252 columns at most
constexpr int kSvdRegMaxRows = 256;
constexpr int kSvdRegCols1 = 126, kSvdRegRows1 = 256;   // one pair per lane
constexpr int kSvdRegRows2 = 208;                       // two
constexpr int kSvdPanelLds = 144 * 1024;   // rows of a Householder panel
constexpr int kSvdLogSweeps = 12;          // logged before V is updated in between (5 to 10 are usual)
constexpr int kSvdPanelRefl = 32;          // reflections of a panel of a sector that does not fit whole
constexpr int kSvdCtrl = 4;                // words of a sector's control record
constexpr int kSvdTrailRows = 32;          // rows of one workgroup after it
// row stride of a panel in LDS: whole groups of 16 lanes' pairs, a count that
// the kernels are built for
__host__ __device__ inline int svd_panel_ld(int64_t ld) { return ld <= 32 ? 32 : ld <= 64 ? 64 : ld <= 128 ? 128 : 224; }
// Lanes of a wave that the log stores: those with columns, the one before them,
// which hands a column back, and one that stands for the rest (zeros).
__host__ __device__ inline int svd_log_lanes(int64_t n, int64_t pairs) {
  const int64_t l = n / (2 * pairs) + 2;
  return (int)(l < 64 ? l : 64);
}
// doubles of one sweep's log: N steps of `pairs` x lanes pairs (beta, alpha), N factors
__host__ __device__ inline int64_t svd_log_sweep(int64_t n, int64_t pairs) {
  return n * pairs * svd_log_lanes(n, pairs) * 2 + n;
}
constexpr int kSvdGatherChunk = 256 * 16;

struct SvdLaunch {
  const SvdGather* gjobs;
  const SvdWork* gwork;
  int64_t ngwork;
  const SvdSec* secs;
  int32_t nsec;
  const double* in;
  double* X;          // X and Vh of every sector
  double* scratch;    // register path: gathered X and reflections, rotation logs
  int32_t* rowpos;    // register path: row and column orders
  // register path: its sectors, most panels and rows left after a panel (0:
  // every sector in one launch), most columns, logged sweeps, and per sector
  // [sweeps in the log, order reversed since, binary exponent taken out of X, -]
  const int32_t* reg;
  int32_t nreg, panels;
  int64_t trail_rows, reg_cols;
  int32_t logcap;
  int32_t* ctrl;
  int32_t nlds;       // sectors of the one-workgroup LDS path
  double* sig;        // |x_j| per column
  double* sorted;     // the same values in descending order
  int32_t* perm;      // column of X (or Vh) of the c-th largest value
  int32_t* sweeps;    // per sector: sweeps used (diagnostic)
  // sectors of the rounds path: rotated a round per launch by the whole
  // device before the per-sector kernel
  const int32_t* big;   // their sector indices
  int32_t nbig;
  int32_t rounds;       // most rounds per sweep over them (r + (r & 1) - 1)
  int32_t pairs;        // most pairs per round
  int64_t vmax;         // largest r * r
  int32_t* flags;       // per big sector: [rotated this sweep, converged]
};
// The gather, and the identity Vh and cleared flags of the big sectors.
hipError_t launch_svd_gather(const SvdLaunch& l, hipStream_t s);
// One sweep over the big sectors not yet converged: every round, then the
// sweep's count (a sector whose sweep rotated nothing is marked converged).
hipError_t launch_svd_sweep(const SvdLaunch& l, hipStream_t s);
// sigma and the sorted order of the sectors of one path, LDS (with their
// sweeps, one workgroup each) or rounds (after those).
hipError_t launch_svd_finish(const SvdLaunch& l, hipStream_t s, int path);
// Everything of the register path's sectors.
hipError_t launch_svd_reg(const SvdLaunch& l, hipStream_t s);

// Where sector (m, n)'s sweeps run: in one workgroup's registers where X fits
// them; else in one workgroup's LDS where it fits that (tall matrices of few
// columns); else a round per launch on the device.
enum SvdPath { kSvdPathReg = 0, kSvdPathLds = 1, kSvdPathRounds = 2 };
__host__ __device__ inline int svd_path(int64_t m, int64_t n) {
  const int64_t p = m >= n ? m : n, r = m >= n ? n : m;
  if ((r <= kSvdRegCols1 && p <= kSvdRegRows1) || p <= kSvdRegRows2) return kSvdPathReg;
  return r > 1 && p * r * 8 > kSvdLdsBytes ? kSvdPathRounds : kSvdPathLds;
}

struct SvdSelectLaunch {
  const SvdSec* secs;
  int32_t nsec;
  const double* sorted;        // per sector, descending
  const int64_t* min_blockdim; // nsec entries (device)
  int64_t keepdim;
  double err;
  int64_t* kept;               // nsec entries
  double* s_err;
};
hipError_t launch_svd_select(const SvdSelectLaunch& l, hipStream_t s);

struct SvdWriteLaunch {
  const SvdWrite* jobs;
  const SvdWriteWork* work;
  int64_t nwork;
  const SvdSec* secs;
  const double* X;
  const int32_t* rowpos;
  const double* sorted;
  const int32_t* perm;
  int32_t absorb;   // 0 none, 1 into U, 2 into V^dagger
  double* U;
  double* Vd;
  double* S;
};
hipError_t launch_svd_write(const SvdWriteLaunch& l, hipStream_t s);

}  // namespace bst

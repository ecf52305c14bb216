// Grouped sector GEMM for block-sparse contraction on CDNA4 (gfx950) MFMA.
//
// One launch covers every output block ("problem") of a contraction step.
// Each workgroup owns one BM x BN output tile of one problem and sums the
// problem's K-segments (one per matching contracted sector tuple) in a fixed
// order into registers, then writes the tile once: no atomics, so results
// are bitwise reproducible run to run.  Problems without segments produce
// zero tiles (output blocks that no sector pair reaches).
//
// Arithmetic forms (operands arrive as float64 or float32 and are converted
// on the way into LDS, so no separate conversion pass touches HBM):
//   FP64    v_mfma_f64_16x16x4f64,   double accumulate
//   FP32    v_mfma_f32_16x16x4f32,   operands rounded to float32 (RNE)
//   BF16X3  v_mfma_f32_16x16x32_bf16, a = a0 + a1 split, a0b0+a0b1+a1b0
//   BF16X6  same with a2: a0b0+a0b1+a1b0+a0b2+a1b1+a2b0
// Tiles: 4 waves (wave64) in a 2 x 2 arrangement, each wave a
// (BM/2) x (BN/2) patch of 16 x 16 MFMA sub-tiles.
#include "hcoef.h"

namespace bst {

typedef double dbl4 __attribute__((ext_vector_type(4)));
typedef double dbl2 __attribute__((ext_vector_type(2)));
typedef float flt4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short us8 __attribute__((ext_vector_type(8)));

// Direct (LDS-free) variants first.
static const std::vector<TileShape> kShapesF64 = {{64, 64, 1}, {128, 64, 1}, {64, 128, 1}, {32, 32, 1},
                                                  {32, 32, 0}, {64, 64, 0}, {64, 32, 0}, {32, 64, 0},
                                                  {32, 32, 4}};
static const std::vector<TileShape> kShapesF32 = {{64, 64, 1}, {128, 64, 1}, {64, 128, 1}, {32, 32, 1},
                                                  {32, 32, 0}, {64, 64, 0}, {128, 64, 0}, {64, 128, 0}};
static const std::vector<TileShape> kShapesBF3 = {{32, 32}, {64, 64}, {128, 64}, {64, 128}};
static const std::vector<TileShape> kShapesBF6 = {{32, 32}, {64, 64}};

const std::vector<TileShape>& gemm_tile_shapes(bst_precision form) {
  switch (form) {
    case BST_FP64: return kShapesF64;
    case BST_FP32: return kShapesF32;
    case BST_BF16X3: return kShapesBF3;
    default: return kShapesBF6;
  }
}

// float -> bfloat16 bits, round to nearest even (finite inputs)
__device__ __forceinline__ unsigned short bf16_rne(float x) {
  unsigned int u = __float_as_uint(x);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}
__device__ __forceinline__ float bf16_val(unsigned short h) { return __uint_as_float((unsigned int)h << 16); }

template <int NP>
__device__ __forceinline__ void split_bf16(double a, unsigned short* h) {
  float f = (float)a;
  h[0] = bf16_rne(f);
  if constexpr (NP > 1) {
    double r = a - (double)bf16_val(h[0]);
    h[1] = bf16_rne((float)r);
    if constexpr (NP > 2) {
      double r2 = r - (double)bf16_val(h[1]);
      h[2] = bf16_rne((float)r2);
    }
  }
}
template <int NP>
__device__ __forceinline__ void split_bf16(float a, unsigned short* h) {
  h[0] = bf16_rne(a);
  if constexpr (NP > 1) {
    float r = a - bf16_val(h[0]);  // exact: fewer than 24 significant bits
    h[1] = bf16_rne(r);
    if constexpr (NP > 2) {
      float r2 = r - bf16_val(h[1]);
      h[2] = bf16_rne(r2);
    }
  }
}

template <int FORM> struct FormTraits;
template <> struct FormTraits<BST_BF16X3> { static constexpr int BK = 32; static constexpr int NP = 2; };
template <> struct FormTraits<BST_BF16X6> { static constexpr int BK = 32; static constexpr int NP = 3; };

// Output element (row, col) of lane `lane`, register r of a 16x16 MFMA tile.
// float32 accumulators: row = 4*(lane/16) + r; float64: row = 4*r + lane/16.
template <bool F64ACC>
__device__ __forceinline__ int acc_row(int lane, int r) {
  return F64ACC ? (4 * r + lane / 16) : (4 * (lane / 16) + r);
}

// Split forms.
template <int FORM, typename TA, typename TC, bool TRANSB, int BM, int BN>
__global__ __launch_bounds__(256, kMfmaWaves) void gemm_grouped_kernel(const GemmTile* __restrict__ tiles,
                                                                       const GemmProb* __restrict__ probs,
                                                                       const GemmSeg* __restrict__ segs,
                                                                       void* const* __restrict__ ptrs) {
  constexpr int BK = FormTraits<FORM>::BK;
  constexpr int NP = FormTraits<FORM>::NP;
  constexpr int WM = BM / 2, WN = BN / 2;
  constexpr int SM = WM / 16, SN = WN / 16;
  constexpr int PADH = 8;   // LDS row pad (elements): keeps 16-byte alignment
  constexpr int EA = BM * BK / 256, EB = BN * BK / 256;   // tile elements per thread

  // LDS, double buffered: planes [NP][BM][BK+PADH], k contiguous, 16-byte lane reads
  __shared__ __attribute__((aligned(16))) unsigned short As[2][NP * BM * (BK + PADH)];
  __shared__ __attribute__((aligned(16))) unsigned short Bs[2][NP * BN * (BK + PADH)];

  const GemmTile t = tiles[blockIdx.x];
  if (t.prob < 0) return;   // padding of the per-XCD tile lists
  const GemmProb p = probs[t.prob];
  const int tid = threadIdx.x;
  const int wave = tid >> 6, lane = tid & 63;
  const int wm = wave >> 1, wn = wave & 1;
  const int m0 = t.m0, n0 = t.n0;

  flt4 acc[SM][SN];
#pragma unroll
  for (int i = 0; i < SM; ++i)
#pragma unroll
    for (int j = 0; j < SN; ++j) acc[i][j] = flt4{0, 0, 0, 0};

  // next k-step to fetch: segment ls, offset lk; values staged in registers
  int ls = 0, lk = 0;
  TA ra[EA];
  double rb[EB];
  auto fetch = [&]() {
    const GemmSeg g = segs[p.seg_begin + ls];
    const BST_G TA* __restrict__ A = (const BST_G TA*)(ptrs[g.a_buf]) + g.a_off;
    const BST_G double* __restrict__ B = (const BST_G double*)(ptrs[g.b_buf]) + g.b_off;
#pragma unroll
    for (int e = 0; e < EA; ++e) {
      const int idx = tid + e * 256;
      const int r = idx / BK, k = idx % BK;
      const int gr = m0 + r, gk = lk + k;
      ra[e] = (gr < p.M && gk < g.K) ? A[(int64_t)gr * g.lda + gk] : TA(0);
    }
#pragma unroll
    for (int e = 0; e < EB; ++e) {
      const int idx = tid + e * 256;
      int n, k;
      if constexpr (TRANSB) { n = idx / BK; k = idx % BK; }
      else { k = idx / BN; n = idx % BN; }
      const int gn = n0 + n, gk = lk + k;
      double v = 0.0;
      if (gn < p.N && gk < g.K) v = TRANSB ? B[(int64_t)gn * g.ldb + gk] : B[(int64_t)gk * g.ldb + gn];
      rb[e] = v;
    }
    lk += BK;
    if (lk >= g.K) {
      ls++;
      lk = 0;
    }
  };
  auto stage = [&](int buf) {
#pragma unroll
    for (int e = 0; e < EA; ++e) {
      const int idx = tid + e * 256;
      const int r = idx / BK, k = idx % BK;
      unsigned short h[3];
      split_bf16<NP>(ra[e], h);
#pragma unroll
      for (int q = 0; q < NP; ++q) As[buf][(q * BM + r) * (BK + PADH) + k] = h[q];
    }
#pragma unroll
    for (int e = 0; e < EB; ++e) {
      const int idx = tid + e * 256;
      int n, k;
      if constexpr (TRANSB) { n = idx / BK; k = idx % BK; }
      else { k = idx / BN; n = idx % BN; }
      unsigned short h[3];
      split_bf16<NP>(rb[e], h);
#pragma unroll
      for (int q = 0; q < NP; ++q) Bs[buf][(q * BN + n) * (BK + PADH) + k] = h[q];
    }
  };
  auto compute = [&](int buf) {
    bf16x8 a[NP][SM], b[NP][SN];
    const int kl = 8 * (lane >> 4);
#pragma unroll
    for (int q = 0; q < NP; ++q) {
#pragma unroll
      for (int i = 0; i < SM; ++i) {
        const int r = wm * WM + i * 16 + (lane & 15);
        us8 raw = *reinterpret_cast<const us8*>(&As[buf][(q * BM + r) * (BK + PADH) + kl]);
        a[q][i] = __builtin_bit_cast(bf16x8, raw);
      }
#pragma unroll
      for (int j = 0; j < SN; ++j) {
        const int c = wn * WN + j * 16 + (lane & 15);
        us8 raw = *reinterpret_cast<const us8*>(&Bs[buf][(q * BN + c) * (BK + PADH) + kl]);
        b[q][j] = __builtin_bit_cast(bf16x8, raw);
      }
    }
#pragma unroll
    for (int i = 0; i < SM; ++i)
#pragma unroll
      for (int j = 0; j < SN; ++j) {
        if constexpr (NP == 3) {
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[2][i], b[0][j], acc[i][j], 0, 0, 0);
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[1][i], b[1][j], acc[i][j], 0, 0, 0);
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0][i], b[2][j], acc[i][j], 0, 0, 0);
        }
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[1][i], b[0][j], acc[i][j], 0, 0, 0);
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0][i], b[1][j], acc[i][j], 0, 0, 0);
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0][i], b[0][j], acc[i][j], 0, 0, 0);
      }
  };

  // pipeline: the next k-step's global loads are in flight while the
  // current one runs on the MFMA units; one barrier per k-step
  if (p.seg_count > 0) {
    fetch();
    stage(0);
    __syncthreads();
    int buf = 0;
    while (true) {
      const bool more = ls < p.seg_count;
      if (more) fetch();
      compute(buf);
      if (more) stage(buf ^ 1);
      __syncthreads();
      buf ^= 1;
      if (!more) break;
    }
  }
  // ---- epilogue: each element written exactly once ----
  BST_G TC* __restrict__ C = (BST_G TC*)(ptrs[p.c_buf]) + p.c_off;
#pragma unroll
  for (int i = 0; i < SM; ++i)
#pragma unroll
    for (int j = 0; j < SN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = m0 + wm * WM + i * 16 + acc_row<false>(lane, r);
        const int col = n0 + wn * WN + j * 16 + (lane & 15);
        if (row < p.M && col < p.N) C[(int64_t)row * p.ldc + col] = (TC)acc[i][j][r];
      }
}

enum BLayout { kBPlain, kBTrans, kBComplex };   // [k][n], [n][k], complex [k / 2][n / 2]

// float64 / float32 forms.
//
// The sectors of a block-sparse operand are small and odd (a chi = 2048 spin-1/2
// H_eff has 372 block pairs of some 3 to 200 rows and K of 3 to 110).  Without
// its MFMAs this kernel takes nearly as long as with them, so what counts are
// the instructions that move operands, the L1's above all (it was busy nine
// cycles of ten with 8-byte loads):
//   - two neighbouring elements per load where the step and the tile lie inside
//     the segment and the block;
//   - a wave runs the MFMAs of its 16 x 16 sub-tiles that hold elements of the
//     block, and of a segment's last k-step those that reach into it;
//   - loads run D k-steps ahead, in registers, across segments; the record of
//     the next segment is read one segment ahead, the first with the problem's,
//     and the steps are counted while the first loads run (T3.R of chi = 512
//     13.4 -> 12.3 us).
// Rows and columns past the block read its last one (their results are not
// stored); k past the segment reads its last and is replaced by zero.
//
// LDS holds a row of A (and of a transposed B) as its 16 k in the order in which
// the four lane groups read them, each group its operands of the step's four
// MFMAs as one run.  float64: group g and MFMA q take k = 8 (q / 2) + 2 g + q % 2,
// so that a loaded pair stays one 16-byte store.  float32: k = 4 q + g, the plain
// order of the sum.  Rows are 18 doubles or 20 floats apart, so that the 16 rows
// of a read lie in different banks; k-rows of a plain B likewise.
//
// A complex B needs no copy: rows 2 k and 2 k + 1 of the real form of its row k
// are (re, im) pairs and (-im, re) pairs of the same elements (a chi = 1500
// contraction: 20.3 us with the expanded copy made first, now 11.4).
//
// L.psi / T3.R, with one-element loads, a zero for each element outside, every
// MFMA run and one register stage, then now: float64, spin-1/2 chi = 2048 (32 x 32)
// 28.5 / 32.8 -> 26.6 / 29.1 us, spin-1 chi = 4096 (64 x 32) 201 / 198 -> 174 / 161
// us; float32, chi = 4096 (64 x 64) 136 / 132 -> 109 / 102 us.  The MFMAs of the
// chi = 4096 steps alone take 104 (float64).
template <int FORM, typename TA, typename TC, int BL, int BM, int BN, int D>
__global__ __launch_bounds__(256, kMfmaWaves) void gemm_block_kernel(const GemmTile* __restrict__ tiles,
                                                                     const GemmProb* __restrict__ probs,
                                                                     const GemmSeg* __restrict__ segs,
                                                                     void* const* __restrict__ ptrs, int bslot,
                                                                     int hb, HCoefLaunch coef) {
  constexpr bool F64 = (FORM == BST_FP64), TRANSB = (BL == kBTrans), CPLX = (BL == kBComplex);
  constexpr int BK = 16, WM = BM / 2, WN = BN / 2, SM = WM / 16, SN = WN / 16;
  constexpr int EA = BM / 32, EB = BN / 32;               // pairs per lane and k-step
  constexpr int KB = 512 / BN;                            // k rows of B per load (not transposed)
  constexpr int LDK = F64 ? 18 : 20;                      // LDS row of A (and B if transposed)
  constexpr int LDN = F64 ? BN + 8 : BN + 16;             // LDS k-row of B if not
  using CT = typename std::conditional<F64, double, float>::type;
  using ACC = typename std::conditional<F64, dbl4, flt4>::type;
  typedef CT CT2 __attribute__((ext_vector_type(2)));
  typedef TA TA2 __attribute__((ext_vector_type(2)));
  typedef TA TA2u __attribute__((ext_vector_type(2), aligned(sizeof(TA))));
  typedef double dbl2u __attribute__((ext_vector_type(2), aligned(8)));
  __shared__ __attribute__((aligned(16))) CT As[2][BM * LDK];
  __shared__ __attribute__((aligned(16))) CT Bs[2][TRANSB ? BN * LDK : BK * LDN];

  static_assert(sizeof(As) >= 256 * sizeof(double), "coefficient rows");
  if ((int)blockIdx.x < hb) {   // the first hb workgroups: MPO coefficients
    if ((int64_t)blockIdx.x * 256 < coef.nentries)
      hcoef_block(coef, blockIdx.x, reinterpret_cast<double*>(&As[0][0]));
    return;
  }
  const GemmTile t = tiles[blockIdx.x - hb];
  if (t.prob < 0) return;   // padding of the per-XCD tile lists
  GemmSeg nxt = segs[t.seg];   // the first one, read beside the problem
  const GemmProb p = probs[t.prob];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int m0 = t.m0, n0 = t.n0;
  // sub-tiles of this wave that hold elements of the block
  const int mi = min(max((p.M - m0 - wm * WM + 15) / 16, 0), SM);
  const int nj = min(max((p.N - n0 - wn * WN + 15) / 16, 0), SN);
  const bool inner_n = TRANSB || n0 + BN <= p.N;   // pairs of columns lie inside the block

  ACC acc[SM][SN];
#pragma unroll
  for (int i = 0; i < SM; ++i)
#pragma unroll
    for (int j = 0; j < SN; ++j) acc[i][j] = ACC{0, 0, 0, 0};

  // load cursor: segment ls at k = lk
  int ls = 0, lk = 0, lK = 0;
  int64_t ldb = 0;
  const BST_G TA* pa[EA];
  const BST_G double* pb[EB];
  int a_buf = -1, b_buf = -1;
  const BST_G TA* A = nullptr;
  const BST_G double* B = nullptr;
  const int ak = 2 * (tid & 7), ar = tid >> 3;                           // A: first k of the pair, row
  const int bk = TRANSB ? ak : tid / (BN / 2), bn = TRANSB ? ar : 2 * (tid % (BN / 2));
  auto begin = [&]() {   // the segment in nxt becomes current
    const GemmSeg g = nxt;
    if (g.a_buf != a_buf) A = (const BST_G TA*)(ptrs[a_buf = g.a_buf]);
    const int gb = CPLX ? bslot : g.b_buf;
    const int64_t b_off = g.b_off >> CPLX;
    if (gb != b_buf) B = (const BST_G double*)(ptrs[b_buf = gb]);
    if (ls + 1 < p.seg_count) nxt = segs[p.seg_begin + ls + 1];
    lk = 0;
    lK = g.K;
    ldb = g.ldb;
#pragma unroll
    for (int e = 0; e < EA; ++e) pa[e] = A + g.a_off + (int64_t)min(m0 + ar + 32 * e, p.M - 1) * g.lda + ak;
#pragma unroll
    for (int e = 0; e < EB; ++e) {
      if constexpr (TRANSB)
        pb[e] = B + b_off + (int64_t)min(n0 + bn + 32 * e, p.N - 1) * g.ldb + bk;
      else
        pb[e] = B + b_off + (int64_t)((bk + KB * e) >> CPLX) * g.ldb + min(n0 + bn, p.N - 1);
    }
  };
  TA2 ra[D][EA];
  dbl2 rb[D][EB];
  int kv[D];   // k of a step inside its segment
  auto fetch = [&](TA2 (&a)[EA], dbl2 (&b)[EB], int& k) {
    k = min(BK, lK - lk);
    if (k == BK) {
#pragma unroll
      for (int e = 0; e < EA; ++e) a[e] = *reinterpret_cast<const BST_G TA2u*>(pa[e]);
    } else {
      const int o0 = min(k - 1 - ak, 0), o1 = min(k - 1 - ak, 1);   // element k or the last
#pragma unroll
      for (int e = 0; e < EA; ++e) a[e] = TA2{pa[e][o0], pa[e][o1]};
    }
    if (k == BK && inner_n) {
#pragma unroll
      for (int e = 0; e < EB; ++e) b[e] = *reinterpret_cast<const BST_G dbl2u*>(pb[e]);
    } else if constexpr (TRANSB) {
      const int o0 = min(k - 1 - bk, 0), o1 = min(k - 1 - bk, 1);
#pragma unroll
      for (int e = 0; e < EB; ++e) b[e] = dbl2{pb[e][o0], pb[e][o1]};
    } else {
      const int c1 = n0 + bn + 1 < p.N ? 1 : 0;   // the column's neighbour or itself
#pragma unroll
      for (int e = 0; e < EB; ++e) {
        const int kk = bk + KB * e;
        const BST_G double* const q = pb[e] + ((min(k - 1, kk) >> CPLX) - (kk >> CPLX)) * ldb;
        b[e] = dbl2{q[0], q[c1]};
      }
    }
    lk += BK;
    if (lk < lK) {
#pragma unroll
      for (int e = 0; e < EA; ++e) pa[e] += BK;
#pragma unroll
      for (int e = 0; e < EB; ++e) pb[e] += TRANSB ? BK : (BK >> CPLX) * ldb;
    } else if (++ls < p.seg_count) {
      begin();
    }
  };
  // a pair's place in its row
  auto put = [&](CT* row, CT x, CT y) {
    if constexpr (F64) {
      *reinterpret_cast<CT2*>(row + 2 * (ak & 6) + 2 * (ak >> 3)) = CT2{x, y};
    } else {
      row[4 * (ak & 3) + (ak >> 2)] = x;
      row[4 * (ak & 3) + (ak >> 2) + 4] = y;
    }
  };
  // (k past the segment is replaced here and not after the load, which would wait for it)
  auto stage = [&](int buf, TA2 (&a)[EA], dbl2 (&b)[EB], int k) {
    if constexpr (CPLX) {   // KB and BK are even, so a lane's k are all even or all odd
#pragma unroll
      for (int e = 0; e < EB; ++e) b[e] = bk & 1 ? dbl2{-b[e].y, b[e].x} : b[e];
    }
    if (k < BK) {
#pragma unroll
      for (int e = 0; e < EA; ++e) a[e] = TA2{ak < k ? a[e].x : (TA)0, ak + 1 < k ? a[e].y : (TA)0};
#pragma unroll
      for (int e = 0; e < EB; ++e) {
        if constexpr (TRANSB) b[e] = dbl2{bk < k ? b[e].x : 0.0, bk + 1 < k ? b[e].y : 0.0};
        else b[e] = bk + KB * e < k ? b[e] : dbl2{0.0, 0.0};
      }
    }
#pragma unroll
    for (int e = 0; e < EA; ++e) put(As[buf] + (ar + 32 * e) * LDK, (CT)a[e].x, (CT)a[e].y);
#pragma unroll
    for (int e = 0; e < EB; ++e) {
      if constexpr (TRANSB) put(Bs[buf] + (bn + 32 * e) * LDK, (CT)b[e].x, (CT)b[e].y);
      else *reinterpret_cast<CT2*>(Bs[buf] + (bk + KB * e) * LDN + bn) = CT2{(CT)b[e].x, (CT)b[e].y};
    }
  };
  auto mfma = [&](CT a, CT b, ACC c) -> ACC {
    if constexpr (F64) return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  };
  const bool full = mi == SM && nj == SN;
  const int l16 = lane & 15, lg = lane >> 4;
  auto compute = [&](int buf, int k) {
    const CT* const as = As[buf] + (wm * WM + l16) * LDK;
    const CT* const bs = Bs[buf] + (TRANSB ? (wn * WN + l16) * LDK : wn * WN + l16);
    // a lane's operands of MFMA q: element q of its run
    auto run = [&](const CT* row, CT (&v)[4]) {
      if constexpr (F64) {
        const dbl2 lo = *reinterpret_cast<const dbl2*>(row), hi = *reinterpret_cast<const dbl2*>(row + 2);
        v[0] = lo.x;
        v[1] = lo.y;
        v[2] = hi.x;
        v[3] = hi.y;
      } else {
        const flt4 w = *reinterpret_cast<const flt4*>(row);
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = w[q];
      }
    };
    CT a[SM][4], b[SN][4];
#pragma unroll
    for (int i = 0; i < SM; ++i) run(as + 16 * i * LDK + 4 * lg, a[i]);
#pragma unroll
    for (int j = 0; j < SN; ++j) {
      if constexpr (TRANSB) {
        run(bs + 16 * j * LDK + 4 * lg, b[j]);
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          b[j][q] = bs[(F64 ? 8 * (q >> 1) + 2 * lg + (q & 1) : 4 * q + lg) * LDN + 16 * j];
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if ((F64 ? 8 * (q >> 1) + (q & 1) : 4 * q) >= k) break;
#pragma unroll
      for (int i = 0; i < SM; ++i)
#pragma unroll
        for (int j = 0; j < SN; ++j)
          if (full || (i < mi && j < nj)) acc[i][j] = mfma(a[i][q], b[j][q], acc[i][j]);
    }
  };

  if (p.seg_count > 0) {
    begin();
#pragma unroll
    for (int d = 0; d < D; ++d)
      if (ls < p.seg_count) fetch(ra[d], rb[d], kv[d]);
    // k-steps of the tile, counted while the first of them load
    int steps = 0;
    for (int q = 0; q < p.seg_count; ++q) steps += (segs[p.seg_begin + q].K + BK - 1) / BK;
    stage(0, ra[0], rb[0], kv[0]);
    __syncthreads();
    // step u computes from LDS, step u + 1 is staged, step u + D is loaded
    for (int u0 = 0; u0 < steps; u0 += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        const int u = u0 + d;
        if (u >= steps) break;
        const int k = kv[d];
        if (u + D < steps) fetch(ra[d], rb[d], kv[d]);
        if (mi > 0 && nj > 0) compute(D % 2 ? u & 1 : d & 1, k);
        const int e = (d + 1) % D;
        if (u + 1 < steps) stage(D % 2 ? (u + 1) & 1 : (d + 1) & 1, ra[e], rb[e], kv[e]);
        __syncthreads();
      }
    }
  }
  // ---- epilogue: each element written exactly once ----
  BST_G TC* __restrict__ C = (BST_G TC*)(ptrs[p.c_buf]) + p.c_off;
#pragma unroll
  for (int i = 0; i < SM; ++i)
#pragma unroll
    for (int j = 0; j < SN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = m0 + wm * WM + i * 16 + acc_row<F64>(lane, r);
        const int col = n0 + wn * WN + j * 16 + (lane & 15);
        if (row < p.M && col < p.N) C[(int64_t)row * p.ldc + col] = (TC)acc[i][j][r];
      }
}

// float64 tiles of 32 x 32 whose k-steps are shared by the workgroup's four
// waves, a contiguous quarter each, and added at the end (waves 0 + 1, 2 + 3,
// then both).  A tile's k-steps are a serial chain, 0.33 us each in the staged
// kernel (stage, barrier, read, MFMA), and a step with few blocks of large K is
// as long as its longest chain; here a chain is a quarter, and a step of it has
// neither LDS nor barrier: a lane's loads are its MFMA operands, k = 4 g + q of
// MFMA q in lane group g.  T3.R of H_eff: chi = 64 7.5 -> 6.3 us,
// 256 10.8 -> 8.2, 512 13.4 -> 9.7, 1024 18.8 -> 15.1.  Loads two steps ahead; three
// take registers, that is waves (chi = 1024 16.2 us).
__device__ __forceinline__ int wave_scan(int v) {   // inclusive, all lanes active
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true);   // row_shr 1, 2, 4, 8
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // row_bcast 15 to rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // row_bcast 31 to rows 2 and 3
  return v;
}

template <int BL>
__global__ __launch_bounds__(256, kMfmaWaves) void gemm_ksplit_kernel(const GemmTile* __restrict__ tiles,
                                                                      const GemmProb* __restrict__ probs,
                                                                      const GemmSeg* __restrict__ segs,
                                                                      void* const* __restrict__ ptrs, int bslot) {
  constexpr int BK = 16, D = 2;
  typedef double dbl2u __attribute__((ext_vector_type(2), aligned(8)));
  __shared__ double sum[4][32 * 33];
  const GemmTile t = tiles[blockIdx.x];
  if (t.prob < 0) return;   // padding of the per-XCD tile lists
  const GemmProb p = probs[t.prob];
  const int lane = threadIdx.x & 63, l16 = lane & 15, lg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m0 = t.m0, n0 = t.n0;
  const bool m2 = m0 + 16 < p.M, n2 = n0 + 16 < p.N;   // the second 16 rows, columns hold elements

  // this wave's k-steps [t0, t1) of the tile's, and the segment they start in
  int total = 0, base = 0, scan = 0, own = 0;
  for (base = 0; base < p.seg_count; base += 64) {
    own = base + lane < p.seg_count ? (segs[p.seg_begin + base + lane].K + BK - 1) / BK : 0;
    scan = wave_scan(own);
    total += __builtin_amdgcn_readlane(scan, 63);
  }
  const int t0 = total * wave / 4, t1 = total * (wave + 1) / 4;
  int ls = 0, before = 0;   // segment, steps before it
  if (t0 < t1) {
    for (base = 0; base < p.seg_count; base += 64) {
      if (p.seg_count > 64) {
        own = base + lane < p.seg_count ? (segs[p.seg_begin + base + lane].K + BK - 1) / BK : 0;
        scan = wave_scan(own);
      }
      const int chunk = __builtin_amdgcn_readlane(scan, 63);
      if (before + chunk > t0) break;
      before += chunk;
    }
    const int l = __builtin_ctzll(__ballot(before + scan > t0));
    ls = base + l;
    before += __builtin_amdgcn_readlane(scan, l) - __builtin_amdgcn_readlane(own, l);
  }

  dbl4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = dbl4{0, 0, 0, 0};

  int lk = 0, lK = 0;
  int64_t ldb = 0;
  const BST_G double* pa[2];
  const BST_G double* pb[2];
  GemmSeg nxt{};
  auto begin = [&](int k0) {   // the segment in nxt becomes current, from k0 on
    const GemmSeg g = nxt;
    const BST_G double* A = (const BST_G double*)(ptrs[g.a_buf]) + g.a_off + k0 + 4 * lg;
    const BST_G double* B = BL == kBComplex ? (const BST_G double*)(ptrs[bslot]) + (g.b_off >> 1)
                                            : (const BST_G double*)(ptrs[g.b_buf]) + g.b_off;
    if (ls + 1 < p.seg_count) nxt = segs[p.seg_begin + ls + 1];
    lk = k0;
    lK = g.K;
    ldb = g.ldb;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      pa[i] = A + (int64_t)min(m0 + 16 * i + l16, p.M - 1) * g.lda;
      const int n = min(n0 + 16 * i + l16, p.N - 1);
      if constexpr (BL == kBTrans) pb[i] = B + (int64_t)n * g.ldb + k0 + 4 * lg;
      else if constexpr (BL == kBComplex) pb[i] = B + (int64_t)((k0 + 4 * lg) >> 1) * g.ldb + (n & ~1);
      else pb[i] = B + (int64_t)(k0 + 4 * lg) * g.ldb + n;
    }
  };
  dbl2 ra[D][2][2], rb[D][2][2];
  int kv[D];
  auto fetch = [&](dbl2 (&a)[2][2], dbl2 (&b)[2][2], int& k) {
    k = min(BK, lK - lk);
    if (k == BK) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          a[i][h] = *reinterpret_cast<const BST_G dbl2u*>(pa[i] + 2 * h);
          if constexpr (BL == kBTrans) b[i][h] = *reinterpret_cast<const BST_G dbl2u*>(pb[i] + 2 * h);
          else if constexpr (BL == kBComplex) b[i][h] = *reinterpret_cast<const BST_G dbl2u*>(pb[i] + h * ldb);
          else b[i][h] = dbl2{pb[i][2 * h * ldb], pb[i][(2 * h + 1) * ldb]};
        }
    } else {   // k past the segment reads its last
      const int d = k - 1 - 4 * lg;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int o0 = min(d, 2 * h), o1 = min(d, 2 * h + 1);
          a[i][h] = dbl2{pa[i][o0], pa[i][o1]};
          if constexpr (BL == kBTrans) b[i][h] = dbl2{pb[i][o0], pb[i][o1]};
          else if constexpr (BL == kBComplex)   // (K is even: a pair of k is one row)
            b[i][h] = *reinterpret_cast<const BST_G dbl2u*>(pb[i] + (o1 >> 1) * ldb);
          else b[i][h] = dbl2{pb[i][o0 * ldb], pb[i][o1 * ldb]};
        }
    }
    lk += BK;
    if (lk < lK) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        pa[i] += BK;
        pb[i] += BL == kBTrans ? BK : BL == kBComplex ? (BK / 2) * ldb : BK * ldb;
      }
    } else if (++ls < p.seg_count) {
      begin(0);
    }
  };
  auto compute = [&](const dbl2 (&ar)[2][2], const dbl2 (&br)[2][2], int k) {
    double a[2][4], b[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        a[i][q] = ar[i][q >> 1][q & 1];
        if constexpr (BL == kBComplex) {
          // (re, im) of one element: real columns (re, im) in row k even, (-im, re) in row k odd
          const dbl2 e = br[i][q >> 1];
          b[i][q] = q & 1 ? (l16 & 1 ? e.x : -e.y) : (l16 & 1 ? e.y : e.x);
        } else {
          b[i][q] = br[i][q >> 1][q & 1];
        }
      }
    if (k < BK) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          a[i][q] = 4 * lg + q < k ? a[i][q] : 0.0;
          b[i][q] = 4 * lg + q < k ? b[i][q] : 0.0;
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      acc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[0][q], b[0][q], acc[0][0], 0, 0, 0);
      if (n2) acc[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[0][q], b[1][q], acc[0][1], 0, 0, 0);
      if (m2) acc[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[1][q], b[0][q], acc[1][0], 0, 0, 0);
      if (m2 && n2) acc[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[1][q], b[1][q], acc[1][1], 0, 0, 0);
    }
  };
  const int steps = t1 - t0;
  if (steps > 0) {
    nxt = segs[p.seg_begin + ls];
    begin((t0 - before) * BK);
#pragma unroll
    for (int d = 0; d < D; ++d)
      if (d < steps) fetch(ra[d], rb[d], kv[d]);
    for (int u0 = 0; u0 < steps; u0 += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        const int u = u0 + d;
        if (u >= steps) break;
        compute(ra[d], rb[d], kv[d]);
        if (u + D < steps) fetch(ra[d], rb[d], kv[d]);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) sum[wave][(16 * i + acc_row<true>(lane, r)) * 33 + 16 * j + l16] = acc[i][j][r];
  __syncthreads();
  BST_G double* __restrict__ C = (BST_G double*)(ptrs[p.c_buf]) + p.c_off;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int row = (threadIdx.x >> 5) + 8 * e, col = threadIdx.x & 31, at = row * 33 + col;
    if (m0 + row < p.M && n0 + col < p.N)
      C[(int64_t)(m0 + row) * p.ldc + n0 + col] = (sum[0][at] + sum[1][at]) + (sum[2][at] + sum[3][at]);
  }
}

// k-steps that loads run ahead.  32 x 32 float64 at 1, 2, 3, 4: T3.R of chi =
// 512 14.3, 13.7, 13.3, 13.1 us, of chi = 2048 31.6, 28.4, 29.5, 29.4 us, L.psi of
// chi = 2048 26.1, 25.4, 27.7, 27.8 us: more depth costs registers, that is waves,
// which hide as much.  64 x 64 float32 (chi = 4096 L.psi) 120, 130, 131, 146 us.
template <int FORM, int BM, int BN>
constexpr int kBlockDepth = FORM == BST_FP64 || BM * BN <= 1024 ? 2 : 1;

template <int FORM, typename TA, typename TC, int BL>
static hipError_t launch_shape(int bm, int bn, const GemmLaunch& g, hipStream_t s) {
  // (a multiple of the XCD count, which keeps the tiles' place on the XCDs)
  const int64_t hb = (hcoef_blocks(g.coef) + 7) / 8 * 8;
  if (!hcoef_valid(g.coef) || g.ntiles + hb > 0x7FFFFFFF) return hipErrorInvalidValue;
  if (hb > 0 && FORM != BST_FP64 && FORM != BST_FP32) return hipErrorInvalidValue;
  dim3 grid((unsigned)(g.ntiles + hb)), block(256);
#define BST_SHAPE(BM_, BN_)                                                                      \
  if (bm == BM_ && bn == BN_) {                                                                  \
    if constexpr (FORM == BST_FP64 || FORM == BST_FP32)                                          \
      hipLaunchKernelGGL((gemm_block_kernel<FORM, TA, TC, BL, BM_, BN_, kBlockDepth<FORM, BM_, BN_>>), grid, block, 0, s, \
                         g.tiles, g.probs, g.segs, g.ptrs, g.b_complex, (int)hb, g.coef);                     \
    else                                                                                         \
      hipLaunchKernelGGL((gemm_grouped_kernel<FORM, TA, TC, BL == kBTrans, BM_, BN_>), grid, block, 0,   \
                         s, g.tiles, g.probs, g.segs, g.ptrs);                                   \
    return hipGetLastError();                                                                    \
  }
  if constexpr (FORM == BST_FP64) {
    BST_SHAPE(32, 32) BST_SHAPE(64, 64) BST_SHAPE(64, 32) BST_SHAPE(32, 64)
  } else if constexpr (FORM == BST_FP32) {
    BST_SHAPE(32, 32) BST_SHAPE(64, 64) BST_SHAPE(128, 64) BST_SHAPE(64, 128)
  } else {
    BST_SHAPE(32, 32) BST_SHAPE(64, 64)
    if constexpr (FORM == BST_BF16X3) { BST_SHAPE(128, 64) BST_SHAPE(64, 128) }
  }
#undef BST_SHAPE
  return hipErrorInvalidValue;
}

template <int FORM>
static hipError_t launch_form(const GemmLaunch& g, hipStream_t s) {
  const auto& shapes = gemm_tile_shapes((bst_precision)FORM);
  if (g.tile < 0 || g.tile >= (int)shapes.size()) return hipErrorInvalidValue;
  const int bm = shapes[g.tile].bm, bn = shapes[g.tile].bn;
  if constexpr (FORM == BST_FP64) {
    if (shapes[g.tile].direct == 4) {
      if (g.coef.nentries > 0 || g.ta != ElemType::F64 || g.tb != ElemType::F64 || g.tc != ElemType::F64)
        return hipErrorInvalidValue;
      const dim3 grid((unsigned)g.ntiles), block(256);
      if (g.b_complex >= 0)
        hipLaunchKernelGGL(gemm_ksplit_kernel<kBComplex>, grid, block, 0, s, g.tiles, g.probs, g.segs, g.ptrs,
                           g.b_complex);
      else if (g.transb)
        hipLaunchKernelGGL(gemm_ksplit_kernel<kBTrans>, grid, block, 0, s, g.tiles, g.probs, g.segs, g.ptrs, -1);
      else
        hipLaunchKernelGGL(gemm_ksplit_kernel<kBPlain>, grid, block, 0, s, g.tiles, g.probs, g.segs, g.ptrs, -1);
      return hipGetLastError();
    }
  }
  if (shapes[g.tile].direct)
    return g.coef.nentries > 0 || g.b_complex >= 0 ? hipErrorInvalidValue : launch_gemm_direct(g, bm, bn, s);
  const bool a64 = g.ta == ElemType::F64, c64 = g.tc == ElemType::F64;
  if (g.tb != ElemType::F64) return hipErrorInvalidValue;
  if (a64 && c64) {
    if constexpr (FORM == BST_FP64 || FORM == BST_FP32)
      if (g.b_complex >= 0) return launch_shape<FORM, double, double, kBComplex>(bm, bn, g, s);
    if (g.b_complex >= 0) return hipErrorInvalidValue;
    return g.transb ? launch_shape<FORM, double, double, kBTrans>(bm, bn, g, s)
                    : launch_shape<FORM, double, double, kBPlain>(bm, bn, g, s);
  }
  if constexpr (FORM != BST_FP64) {
    if (a64 && !c64 && !g.transb) return launch_shape<FORM, double, float, kBPlain>(bm, bn, g, s);
    if (!a64 && c64 && g.transb) return launch_shape<FORM, float, double, kBTrans>(bm, bn, g, s);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_gemm(const GemmLaunch& g, hipStream_t s) {
  if (g.ntiles <= 0) return hipSuccess;
  if (g.ntiles > 0x7FFFFFFF) return hipErrorInvalidValue;
  switch (g.form) {
    case BST_FP64: return launch_form<BST_FP64>(g, s);
    case BST_FP32: return launch_form<BST_FP32>(g, s);
    case BST_BF16X3: return launch_form<BST_BF16X3>(g, s);
    case BST_BF16X6: return launch_form<BST_BF16X6>(g, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace bst

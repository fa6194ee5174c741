// gp.hip -- Gaussian-process surrogate on the device, FP64 throughout
// (paper Sec. 2.2-2.3):
//   covariance   C = sigma_f^2 exp(-d^2 / 2 l^2) + sigma_n^2 I
//                (Eqs. quadraticKernelEq, d2Eq, covarianceEq)
//   factor       C = L L^T (blocked right-looking Cholesky, panels of 32)
//   weights      alpha = C^-1 y, carried through the factorisation
//   prediction   mean = K* alpha (Eq. predMeanEq),
//                var = sigma_f^2 - |L^-1 k*|^2 (diagonal of Eq. predVarEq), with
//                L^-1 formed once per factorisation so that a query is a
//                product on the matrix cores, not a sequential solve
//   evidence     -1/2 y^T alpha - sum log L_ii - n/2 log 2 pi (Eq. evidenceEq)
// Options: each point's own noise variance on the diagonal (heteroscedastic),
// the periodic kernel of App. B (Eq. periodicKernel) on a single input, and
// hyperparameters that maximise the evidence (gp_optimize).
// One elimination gives the factor, its inverse and the weights, a launch per
// panel; the evidence search factors many hyperparameter sets at once;
// prediction takes 32 queries a workgroup on the matrix cores, or, where
// queries are few and the database small, a workgroup per query
// (enqueue_predict).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "engine.h"

struct hmd_gp {
  hmd_ctx* ctx = nullptr;
  hmd_gp_hyper hyp{};
  int d = 0;
  int n = 0, cap = 0, ld = 0;  // points, columns reserved, leading dimension (cap + the tile row of y)
  std::vector<double> X, y, se;  // database (host copy)
  std::vector<double> stage;     // its upload
  double* slab = nullptr;        // the one allocation behind the pointers up to dnoise
  double scale[4] = {1, 1, 1, 1};
  double s_q = 1.0, sigma_n = 0.0;
  double* dX = nullptr;      // cap x 4, row-major
  double* dy = nullptr;      // scaled outputs
  double* dL = nullptr;      // ld x cap, column-major
  double* dLi = nullptr;     // L^-1, same layout (lower triangle)
  double* ddinv = nullptr;   // inverses of L's diagonal tiles
  double* dalpha = nullptr;  // C^-1 y
  double* dtmp = nullptr;    // cap
  double* dnoise = nullptr;  // cap: per-point noise variances (heteroscedastic)
  double* dq = nullptr;      // host queries and their results
  double* dpart = nullptr;   // sums of row groups (predictions on the matrix cores)
  size_t part_cap = 0;
  double* dout = nullptr;    // predictions / scalars
  int* dinfo = nullptr;
  size_t q_cap = 0;
};

namespace hmd {
namespace {

constexpr int GP_MAXD = 4;
constexpr int GP_MAXN = 6144;  // database points (the limit that gp_fit states; L and L^-1 then take 0.6 GB)

struct KParams {
  double inv_scale[GP_MAXD];
  double sf2, inv_2l2, sn2;
  double pi_over_T;  // periodic kernel: pi / T
  int d;
  int kind;          // 0 squared exponential (Eq. quadraticKernelEq), 1 periodic (Eq. periodicKernel)
};

// K(a, b): sigma_f^2 exp(-d^2 / 2 l^2) on the normalised distance of Eq.
// d2Eq, or sigma_f^2 exp(-2 sin^2(pi |t - t'| / T) / l^2) on the first input
__device__ __forceinline__ double sqexp(const double* a, const double* b, const KParams& P) {
  if (P.kind == 1) {
    const double sn = sin(P.pi_over_T * fabs(a[0] - b[0]));
    return P.sf2 * exp(-4.0 * sn * sn * P.inv_2l2);
  }
  double d2 = 0.0;
#pragma unroll
  for (int k = 0; k < GP_MAXD; ++k) {  // inputs past d are zero on both sides
    const double t = (a[k] - b[k]) * P.inv_scale[k];
    d2 += t * t;
  }
  return P.sf2 * exp(-d2 * P.inv_2l2);
}

// ---------------------------------------------------------------------------
// Factorisation.  The matrix is taken in tiles of 32 x 32 (rows and columns
// past n padded with the identity), the outputs y as one more tile row, and
// one launch eliminates one panel p from everything to its right and below:
//   S(i) = A(i,p) L_pp^-T                       (rows i > p: the factor's panel)
//   A(i,j) -= S(i) S(j)^T                       (j > p: trailing matrix)
//   W(i,j) -= S(i) Z(p,j), Z(p,j) = L_pp^-1 W(p,j), W(p,p) = I   (j <= p)
// W starts as the identity, so the same elimination leaves L, L^-1 (rows Z),
// L^-1 y (the y row of S) and -C^-1 y (the y row of W): no triangular solve
// follows.  The workgroup of tile (p+1, p+1) factors and inverts it at once
// for the next launch, so each panel costs one launch.  Up to ~1000 points
// what bounds it is the chain of that launch, a tile update and a 32 x 32
// factorisation: 12.8 us a panel, where a diagonal, a panel and an update
// launch took 52 us and the substitutions after them two barriers per row
// (one refit of 256 points: 840 -> 220 us).  At 3001 points it is the tiles'
// passes over the matrix (30 us a panel; factor, weights and inverse together
// 21 -> 2.9 ms).
//
// In place: A lives in L's array and W in L^-1's.  A panel's tiles are still
// read by the whole launch that eliminates it, so S(i) and Z(p,j) replace
// them one launch later (recomputed from the same inputs).
//
// All products are of the form F G^T with both factors column-major in LDS,
// 16 x 16 x 4 FP64 matrix instructions, four wavefronts a tile.  The result
// has rows along the lanes, so columns leave as contiguous 128-byte pieces.
// ---------------------------------------------------------------------------
constexpr int TB = 32;       // tile
constexpr int TP = TB + 1;   // pitch of a tile in LDS
constexpr int TILE_EL = TB * TP;

using f64x4 = __attribute__((ext_vector_type(4))) double;

// acc(r, c) += sum_k F(r, k) G(c, k) over 16 x 16 x K for one wavefront:
// F(r, k) = f[k fs + r], G(c, k) = g[k gk + c gc]; lane l holds r = l % 16,
// c = 4 t + l / 16 in element t.
template <int K>
__device__ __forceinline__ f64x4 tile_mma(const double* f, int fs, const double* g, int gk, int gc, double sign,
                                          f64x4 acc) {
  const int l = threadIdx.x & 63, m = l & 15, k = l >> 4;
#pragma unroll
  for (int k0 = 0; k0 < K; k0 += 4) {
    const double b = f[(k0 + k) * fs + m], a = sign * g[(k0 + k) * gk + m * gc];
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc, 0, 0, 0);
  }
  return acc;
}

__device__ __forceinline__ void tile_load(double* lds, const double* __restrict__ src, size_t ld) {
  for (int e = threadIdx.x; e < TB * TB; e += blockDim.x) lds[(e / TB) * TP + e % TB] = src[(e % TB) + (e / TB) * ld];
}

// A wavefront's quarter of a 32 x 32 result: rows 16 wr, columns 16 wc.
struct Quarter {
  int wr, wc, r, c;  // r: this lane's row, c: its first column (element t: column c + 4 t)
  __device__ Quarter() {
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    wr = w & 1;
    wc = w >> 1;
    r = 16 * wr + (l & 15);
    c = 16 * wc + (l >> 4);
  }
};

__device__ __forceinline__ double lane_value(double v, int lane) {
  const long long b = __double_as_longlong(v);
  const uint32_t lo = __builtin_amdgcn_readlane(uint32_t(b), lane);
  const uint32_t hi = __builtin_amdgcn_readlane(uint32_t(uint64_t(b) >> 32), lane);
  return __longlong_as_double(int64_t((uint64_t(hi) << 32) | lo));
}

// 1 / d to within rounding for normal d > 0 (the hardware estimate and two
// Newton steps).
__device__ __forceinline__ double reciprocal(double d) {
  double r = __builtin_amdgcn_rcp(d);
  r = fma(r, fma(-d, r, 1.0), r);
  return fma(r, fma(-d, r, 1.0), r);
}

// L D L^T of a 32 x 32 tile by one wavefront: t (lower triangle) becomes the
// unit factor U below the diagonal, inv U^-1 on and below it, piv the pivots.
//
// The quadrants (11, the transpose of 21, 22) stay in accumulators of the
// 16 x 16 x 4 matrix instruction, element b of lane 16 k + m being row 4 b + k,
// column m: by symmetry that is row m of column 4 b + k, so element b holds
// four columns just as the instruction takes an operand of K = 4.  Four
// columns at a time are eliminated among themselves (pivots and multipliers
// by readlane, reciprocals instead of roots) and from the rows of the inverse
// that starts as the identity; one instruction per quadrant then applies them
// to all that follows.  The eight steps are one loop: the code is read from
// memory once per launch, and unrolled it took longer to fetch than to run.
// Returns the first pivot that is not positive, or -1.
__device__ int tile_factor(double* t, double* inv, double* piv) {
  const int lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
  const bool g1 = (g & 1) != 0, g2 = (g & 2) != 0;
  auto mine = [&](double v0, double v1, double v2, double v3) {  // this lane group's of four
    const double lo = g1 ? v1 : v0, hi = g1 ? v3 : v2;
    return g2 ? hi : lo;
  };
  auto block = [](const f64x4& v, int b) { return b < 2 ? (b == 0 ? v[0] : v[1]) : (b == 2 ? v[2] : v[3]); };
  int bad = -1;
  double own = 1.0;  // lane c: pivot of column c
  f64x4 q, q12, q22, wd, w21;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const int c = 4 * b + g, lo = min(c, m), hi = max(c, m);
    q[b] = t[lo * TP + hi];
    q12[b] = t[c * TP + 16 + m];
    q22[b] = t[(16 + lo) * TP + 16 + hi];
    wd[b] = c == m ? 1.0 : 0.0;
    w21[b] = 0.0;
  }
#pragma unroll 1
  for (int step = 0; step < 8; ++step) {
    const int b = step & 3, half = step >> 2, r0 = 16 * half;
    if (step == 4) {
      q = q22;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        wd[k] = 4 * k + g == m ? 1.0 : 0.0;
        q12[k] = 0.0;
      }
    }
    const double qb = block(q, b), eb = block(q12, b), wb = block(wd, b), vb = block(w21, b);
    double c[4], e[4], w[4], v[4], lc[4], le[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      c[k] = __shfl(qb, 16 * k + m);  // row m (e: 16 + m) of the four columns
      e[k] = __shfl(eb, 16 * k + m);
      w[k] = __shfl(wb, 16 * k + m);  // column m of the inverse's four rows
      v[k] = __shfl(vb, 16 * k + m);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int col = r0 + 4 * b + k;
      double d = lane_value(c[k], 4 * b + k);
      if (!(d > 0.0)) {
        if (bad < 0) bad = col;
        d = 1.0;
      }
      own = lane == col ? d : own;
      const double ri = reciprocal(d);
      lc[k] = c[k] * ri;
      le[k] = e[k] * ri;
#pragma unroll
      for (int k2 = k + 1; k2 < 4; ++k2) {
        const double f = lane_value(c[k], 4 * b + k2), u = f * ri;  // U of row 4 b + k2
        c[k2] = fma(-lc[k], f, c[k2]);
        e[k2] = fma(-le[k], f, e[k2]);
        w[k2] = fma(-u, w[k], w[k2]);
        v[k2] = fma(-u, v[k], v[k2]);
      }
    }
    const double x1 = -mine(c[0], c[1], c[2], c[3]), y1 = mine(lc[0], lc[1], lc[2], lc[3]);
    const double x2 = -mine(e[0], e[1], e[2], e[3]), y2 = mine(le[0], le[1], le[2], le[3]);
    const double zd = mine(w[0], w[1], w[2], w[3]), z21 = mine(v[0], v[1], v[2], v[3]);
    const double below = m >= 4 * b + 4 ? -y1 : 0.0;  // rows after the four
    q = __builtin_amdgcn_mfma_f64_16x16x4f64(x1, y1, q, 0, 0, 0);
    q12 = __builtin_amdgcn_mfma_f64_16x16x4f64(x1, y2, q12, 0, 0, 0);
    q22 = __builtin_amdgcn_mfma_f64_16x16x4f64(x2, y2, q22, 0, 0, 0);
    wd = __builtin_amdgcn_mfma_f64_16x16x4f64(below, zd, wd, 0, 0, 0);
    w21 = __builtin_amdgcn_mfma_f64_16x16x4f64(half ? below : -y2, half ? z21 : zd, w21, 0, 0, 0);
    const int cc = 4 * b + g;  // this lane's column of U and row of U^-1
    t[(r0 + cc) * TP + r0 + m] = y1;
    inv[(r0 + m) * TP + r0 + cc] = zd;
    if (half) inv[m * TP + 16 + cc] = z21;
    else t[cc * TP + 16 + m] = y2;
  }
  if (lane < TB) piv[lane] = own;
  return bad;
}

// One problem of a batch of factorisations (gp_optimize): strides between
// problems; a single fit has one.
struct Chol {
  double* A;        // L (in place of C), tile rows up to the y row
  double* W;        // L^-1 (INV), same layout
  double* dinv;     // inverses of the diagonal tiles, TB x TB each
  int* info;        // 0, or k + 1 for the first pivot k that is not positive (see panel_failed)
  int ld, nt;       // leading dimension, column tiles
  size_t stride, dstride;
};

// After its tile is final: Cholesky factor and inverse of diagonal tile `p`
// (all threads; the tile is in t), scaled from L D L^T on the way out.
__device__ void finish_diag(const Chol& M, int z, int p, bool inv_out, double* t, double* inv) {
  __shared__ int bad;
  __shared__ double piv[TB], root[TB], iroot[TB];
  __syncthreads();
  if (threadIdx.x < 64) {
    const int b = tile_factor(t, inv, piv);
    if (threadIdx.x == 0) bad = b;
    if (threadIdx.x < TB) {
      const double r = sqrt(piv[threadIdx.x]);
      root[threadIdx.x] = r;
      iroot[threadIdx.x] = 1.0 / r;
    }
  }
  __syncthreads();
  double* const L = M.A + z * M.stride + size_t(p) * TB * (M.ld + 1);
  double* const V = M.dinv + z * M.dstride + size_t(p) * TB * TB;
  double* const Wd = M.W + (inv_out ? z * M.stride + size_t(p) * TB * (M.ld + 1) : 0);
  for (int e = threadIdx.x; e < TB * TB; e += blockDim.x) {
    const int r = e % TB, c = e / TB;
    const double u = r == c ? 1.0 : (r > c ? t[c * TP + r] : 0.0);
    const double ui = r >= c ? inv[c * TP + r] * iroot[r] : 0.0;
    L[r + size_t(c) * M.ld] = u * root[c];
    V[e] = ui;
    if (inv_out) Wd[r + size_t(c) * M.ld] = ui;
  }
  if (threadIdx.x == 0 && bad >= 0)
    __hip_atomic_store(M.info + z, p * TB + bad + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Covariance tiles (i >= j) of every problem, padded with the identity, the
// outputs y in tile row nt; the first diagonal tile is factored at once.
// par (nullable): sigma_f^2, 1 / 2 l^2 and sigma_n^2 of each problem.  The
// diagonal takes noise[i] when given (per-point variances), else sigma_n^2.
template <bool INV>
__global__ __launch_bounds__(256, 4) void k_gp_cov(int n, const double* __restrict__ X, const double* __restrict__ y,
                                                KParams P, const double* __restrict__ par,
                                                const double* __restrict__ noise, Chol M) {
  __shared__ double t[TILE_EL], inv[TILE_EL];
  const int z = blockIdx.y;
  int i = int((sqrt(8.0 * double(blockIdx.x) + 1.0) - 1.0) * 0.5);
  while ((i + 1) * (i + 2) / 2 <= int(blockIdx.x)) ++i;
  while (i * (i + 1) / 2 > int(blockIdx.x)) --i;
  const int j = int(blockIdx.x) - i * (i + 1) / 2;
  double* const A = M.A + z * M.stride;
  if (j >= M.nt) return;  // the y row has no diagonal tile
  if (i == M.nt) {
    if (threadIdx.x < TB) {
      const int c = j * TB + threadIdx.x;
      A[size_t(i) * TB + size_t(c) * M.ld] = c < n ? y[c] : 0.0;
    }
    return;
  }
  if (par) {
    P.sf2 = par[3 * z];
    P.inv_2l2 = par[3 * z + 1];
    P.sn2 = par[3 * z + 2];
  }
  const bool first = i == 0 && j == 0;
  for (int e = threadIdx.x; e < TB * TB; e += blockDim.x) {
    const int r = i * TB + e % TB, c = j * TB + e / TB;
    double v = r == c ? 1.0 : 0.0;
    if (r < n && c < n) {
      v = sqexp(X + GP_MAXD * r, X + GP_MAXD * c, P);
      if (r == c) v += noise ? noise[r] : P.sn2;
    }
    if (first) t[(e / TB) * TP + e % TB] = v;
    else A[r + size_t(c) * M.ld] = v;
  }
  if (first) {
    if (threadIdx.x == 0) M.info[z] = 0;
    finish_diag(M, z, 0, INV, t, inv);
  }
}

// Whether a diagonal tile up to that of panel p has failed.  Those were
// factored by earlier launches.  The launch that eliminates panel p may itself
// set info, for panel p + 1, while others of its workgroups ask: a failure
// there counts from the next launch on, so that all of them, and every thread
// of a workgroup, decide alike whichever value they read.
__device__ __forceinline__ bool panel_failed(int info, int p) { return info != 0 && (info - 1) / TB <= p; }

// Elimination of panel p (see above); launched for p = 0 .. nt with the tiles
// (i, j), i >= max(p - 1, 0), j <= min(i, nt - 1), numbered row by row.  The
// last launch only replaces panel nt - 1's tiles.  Without INV (the evidence
// alone) there is no W and only the y row of S is kept.  alpha (INV) receives
// C^-1 y.
template <bool INV>
__global__ __launch_bounds__(256, 4) void k_gp_panel(int p, Chol M, double* __restrict__ alpha) {
  __shared__ double f[TILE_EL], g[TILE_EL], v[TILE_EL];
  const int z = blockIdx.y;
  const int info = __hip_atomic_load(M.info + z, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const int i0 = INV ? max(p - 1, 0) : p, first = i0 * (i0 + 1) / 2;
  const int b = int(blockIdx.x) + first;
  int i = int((sqrt(8.0 * double(b) + 1.0) - 1.0) * 0.5);
  while ((i + 1) * (i + 2) / 2 <= b) ++i;
  while (i * (i + 1) / 2 > b) --i;
  const int j = b - i * (i + 1) / 2, nt = M.nt;
  if (j >= nt || i > nt) return;
  if (panel_failed(info, p)) return;  // (asked for first: its way is as long as the tile numbers')
  const size_t ld = M.ld;
  double* const A = M.A + z * M.stride;
  double* const W = M.W + z * M.stride;
  auto tile = [&](double* base, int ti, int tj) { return base + size_t(ti) * TB + size_t(tj) * TB * ld; };
  const Quarter Q;
  const f64x4 zero = {0.0, 0.0, 0.0, 0.0};
  // panel p - 1's tiles take their final values
  const bool late_s = p > 0 && j == p - 1 && i >= p && (INV || i == nt);
  const bool late_z = INV && p > 0 && i == p - 1 && j < p - 1;
  if (late_s || late_z) {
    const double* const dv = M.dinv + z * M.dstride + size_t(p - 1) * TB * TB;
    tile_load(v, dv, TB);
    double* const out = late_s ? tile(A, i, j) : tile(W, i, j);
    tile_load(f, out, ld);
    __syncthreads();
    const f64x4 s = late_s ? tile_mma<TB>(f + 16 * Q.wr, TP, v + 16 * Q.wc, TP, 1, 1.0, zero)
                           : tile_mma<TB>(v + 16 * Q.wr, TP, f + 16 * Q.wc * TP, 1, TP, 1.0, zero);
#pragma unroll
    for (int k = 0; k < 4; ++k) out[Q.r + size_t(Q.c + 4 * k) * ld] = s[k];
    __syncthreads();
  }
  if (INV && p == nt && i == nt) {  // the y row of W is complete
    if (threadIdx.x < TB) alpha[j * TB + threadIdx.x] = -tile(W, nt, j)[size_t(threadIdx.x) * ld];
    return;
  }
  if (p == nt || i <= p || (!INV && j <= p)) return;
  const double* const dp = M.dinv + z * M.dstride + size_t(p) * TB * TB;
  double* const out = j > p ? tile(A, i, j) : tile(W, i, j);
  f64x4 acc = zero;
  if (j != p) {
#pragma unroll
    for (int k = 0; k < 4; ++k) acc[k] = out[Q.r + size_t(Q.c + 4 * k) * ld];
  }
  tile_load(v, dp, TB);
  tile_load(f, tile(A, i, p), ld);
  if (j > p && j < i) tile_load(g, tile(A, j, p), ld);
  else if (j < p) tile_load(g, tile(W, p, j), ld);
  __syncthreads();
  // S(i), and S(j) or Z(p, j) kept as G(c, k) = [k][c]
  const f64x4 si = tile_mma<TB>(f + 16 * Q.wr, TP, v + 16 * Q.wc, TP, 1, 1.0, zero);
  f64x4 sj = zero;
  if (j > p && j < i) sj = tile_mma<TB>(g + 16 * Q.wr, TP, v + 16 * Q.wc, TP, 1, 1.0, zero);
  else if (j < p) sj = tile_mma<TB>(v + 16 * Q.wr, TP, g + 16 * Q.wc * TP, 1, TP, 1.0, zero);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    f[(Q.c + 4 * k) * TP + Q.r] = si[k];
    if (j > p && j < i) g[(Q.c + 4 * k) * TP + Q.r] = sj[k];
    else if (j < p) g[Q.r * TP + Q.c + 4 * k] = sj[k];
  }
  __syncthreads();
  if (j == p) acc = tile_mma<TB>(f + 16 * Q.wr, TP, v + 16 * Q.wc * TP, 1, TP, -1.0, acc);
  else acc = tile_mma<TB>(f + 16 * Q.wr, TP, (j == i ? f : g) + 16 * Q.wc, TP, 1, -1.0, acc);
  if (j > p && i == j && i == p + 1) {
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 4; ++k) g[(Q.c + 4 * k) * TP + Q.r] = acc[k];
    finish_diag(M, z, p + 1, INV, g, v);
    return;
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) out[Q.r + size_t(Q.c + 4 * k) * ld] = acc[k];
}

// x = L^-1 b (lower) then, if `both`, x = L^-T x: column-oriented
// substitution in one workgroup; b is overwritten by the result.
__global__ __launch_bounds__(1024) void k_gp_solve(int n, int ld, const double* __restrict__ L, double* __restrict__ b,
                                                   int both) {
  __shared__ double xk;
  const int tid = threadIdx.x, nt = blockDim.x;
  for (int k = 0; k < n; ++k) {
    if (tid == 0) {
      xk = b[k] / L[k + size_t(k) * ld];
      b[k] = xk;
    }
    __syncthreads();
    for (int i = k + 1 + tid; i < n; i += nt) b[i] -= L[i + size_t(k) * ld] * xk;
    __syncthreads();
  }
  if (!both) return;
  for (int k = n - 1; k >= 0; --k) {
    if (tid == 0) {
      xk = b[k] / L[k + size_t(k) * ld];
      b[k] = xk;
    }
    __syncthreads();
    for (int i = tid; i < k; i += nt) b[i] -= L[k + size_t(i) * ld] * xk;
    __syncthreads();
  }
}

// Prior at m queries (empty database).
__global__ void k_gp_prior(int m, double var0, double* __restrict__ mean, double* __restrict__ var) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= m) return;
  mean[q] = 0.0;
  var[q] = var0;
}

// L grew by row r (its leading rows unchanged): row r of L^-1 is
// -(1 / L_rr) sum_{j<=k<r} L_rk (L^-1)_kj for j < r, and 1 / L_rr on the
// diagonal. One wavefront per column j; row r of L staged in LDS.
__global__ __launch_bounds__(256) void k_gp_inv_append_row(int r, int ld, const double* __restrict__ L,
                                                           double* __restrict__ Li) {
  extern __shared__ double lr[];
  const int tid = threadIdx.x, lane = tid & 63;
  for (int k = tid; k < r; k += blockDim.x) lr[k] = L[r + size_t(k) * ld];
  __syncthreads();
  const double inv_d = 1.0 / L[r + size_t(r) * ld];
  const int j = blockIdx.x * (blockDim.x / 64) + (tid >> 6);
  if (j > r) return;
  if (j == r) {
    if (lane == 0) Li[r + size_t(r) * ld] = inv_d;
    return;
  }
  const double* col = Li + size_t(j) * ld;
  double t = 0.0;
  for (int k = j + lane; k < r; k += 64) t += lr[k] * col[k];
  for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o);
  if (lane == 0) Li[r + size_t(j) * ld] = -t * inv_d;
}

// Query q of an m x d row-major array, padded to GP_MAXD inputs.
struct Query {
  double x[GP_MAXD];
  __device__ Query(const double* Xq, int d, int q) {
#pragma unroll
    for (int k = 0; k < GP_MAXD; ++k) x[k] = k < d ? Xq[size_t(q) * d + k] : 0.0;
  }
};

// One query per workgroup of 256 x PARTS threads: k* in LDS (dynamic, n
// doubles), mean = k* . alpha, variance = sigma_f^2 - |L^-1 k*|^2 by block
// reduction, in output units.  Thread (i, part) sums every PARTS-th column of
// row i.  For few queries of a small database: what bounds it is the chain of
// dependent loads of a row, so rows are split (256 points, 200 queries: 21 us
// with one thread a row, 11 with four).
template <int PARTS>
__global__ __launch_bounds__(256 * PARTS) void k_gp_predict(int n, int ld, const double* __restrict__ X,
                                                            const double* __restrict__ Xq,
                                                            const double* __restrict__ Li,
                                                            const double* __restrict__ alpha, KParams P, double s_q,
                                                            double* __restrict__ mean, double* __restrict__ var) {
  extern __shared__ double ks[];
  __shared__ double rows[PARTS][256];
  __shared__ double red[2][4];
  const int q = blockIdx.x, tid = threadIdx.x, nt = 256 * PARTS, row = tid & 255, part = tid >> 8;
  const Query x(Xq, P.d, q);
  double sm = 0.0, sv = 0.0;
  for (int i = tid; i < n; i += nt) {
    const double k = sqexp(X + GP_MAXD * i, x.x, P);
    ks[i] = k;
  }
  __syncthreads();
  for (int i0 = 0; i0 < n; i0 += 256) {
    const int i = i0 + row;
    double w = 0.0;
    if (i < n) {
      if (part == 0) sm += ks[i] * alpha[i];
      double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
      const double* col = Li + i;
      int j = part;
      for (; j + 3 * PARTS <= i; j += 4 * PARTS) {  // column-major reads are coalesced over i
        a0 += col[size_t(j) * ld] * ks[j];
        a1 += col[size_t(j + PARTS) * ld] * ks[j + PARTS];
        a2 += col[size_t(j + 2 * PARTS) * ld] * ks[j + 2 * PARTS];
        a3 += col[size_t(j + 3 * PARTS) * ld] * ks[j + 3 * PARTS];
      }
      for (; j <= i; j += PARTS) a0 += col[size_t(j) * ld] * ks[j];
      w = (a0 + a1) + (a2 + a3);
    }
    rows[part][row] = w;
    __syncthreads();
    if (part == 0) {
#pragma unroll
      for (int p = 1; p < PARTS; ++p) w += rows[p][row];
      sv += w * w;
    }
    __syncthreads();
  }
  if (part == 0) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      sm += __shfl_xor(sm, o);
      sv += __shfl_xor(sv, o);
    }
    if ((tid & 63) == 0) {
      red[0][tid >> 6] = sm;
      red[1][tid >> 6] = sv;
    }
  }
  __syncthreads();
  if (tid == 0) {
    mean[q] = ((red[0][0] + red[0][1]) + (red[0][2] + red[0][3])) * s_q;
    var[q] = (P.sf2 - ((red[1][0] + red[1][1]) + (red[1][2] + red[1][3]))) * s_q * s_q;
  }
}

// 32 queries and 64 RB rows per workgroup: V = L^-1 K* on the FP64 matrix
// cores, k* formed 128 points at a time in LDS, L^-1 read as the operand (16
// rows of 4 columns a load); part[g m + q] receives the sum of V^2 over row
// group g, mean[q] (the last group, which passes every point) k* . alpha.
// A wavefront takes every fourth block of 16 rows, so that the triangle's
// work is shared evenly.  What bounds it is the matrix rate and the
// exponentials of k*, one per 256 rows and query: 20,000 queries of 1000
// points take 0.55 ms (36 TFLOP/s, half of what a large FP64 product
// reaches), 5.3 ms with a workgroup per query; 200 queries of 3001 points
// 0.34 ms, 2.8 before.
constexpr int PQ = 32, PK = 128, PQ_PITCH = 40;  // pitch: the four columns of an operand on different banks

template <int RB>
__global__ __launch_bounds__(256) void k_gp_predict_tiles(int n, int ld, const double* __restrict__ X, int m,
                                                          const double* __restrict__ Xq,
                                                          const double* __restrict__ Li,
                                                          const double* __restrict__ alpha, KParams P, double s_q,
                                                          double* __restrict__ part, double* __restrict__ mean) {
  __shared__ double ks[PK * PQ_PITCH];
  __shared__ double red[8][PQ];
  const int g = int(gridDim.y) - 1 - int(blockIdx.y);  // the longest rows first
  const int tid = threadIdx.x, l = tid & 63, w = tid >> 6, lr = l & 15, lk = l >> 4;
  const int qi = tid & (PQ - 1), kk = tid / PQ, q = blockIdx.x * PQ + qi;
  const bool tail = g == int(gridDim.y) - 1;
  const Query x(Xq, P.d, min(q, m - 1));
  const int row_g = g * 64 * RB + 16 * w;  // row block rb of this wavefront: row_g + 64 rb
  const int kend = min(n, (g + 1) * 64 * RB);
  f64x4 acc[RB][2];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) acc[rb][0] = acc[rb][1] = f64x4{0.0, 0.0, 0.0, 0.0};
  double sm = 0.0;
  for (int kc = 0; kc < kend; kc += PK) {
    __syncthreads();
    for (int i = kk; i < PK; i += 8) {
      const int k = kc + i;
      double v = 0.0;
      if (k < kend) {
        v = sqexp(X + GP_MAXD * k, x.x, P);
        if (tail) sm += v * alpha[k];
      }
      ks[i * PQ_PITCH + qi] = v;
    }
    __syncthreads();
    const int kn = min(PK, kend - kc);
    for (int kb = 0; kb < kn; kb += 16) {
      const int k0 = kc + kb;
      double a[RB][4], b[4][2];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        const int r0 = row_g + 64 * rb, r = r0 + lr;
        if (k0 > r0 || r0 >= n) continue;  // uniform
        const double* const src = Li + r + size_t(k0 + lk) * ld;
#pragma unroll
        for (int u = 0; u < 4; ++u) a[rb][u] = src[size_t(4 * u) * ld];
        if (k0 == r0 || r0 + 16 > n) {  // the diagonal, and rows past the last
#pragma unroll
          for (int u = 0; u < 4; ++u) a[rb][u] = k0 + lk + 4 * u <= r && r < n ? a[rb][u] : 0.0;
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        b[u][0] = ks[(kb + 4 * u + lk) * PQ_PITCH + lr];
        b[u][1] = ks[(kb + 4 * u + lk) * PQ_PITCH + 16 + lr];
      }
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        const int r0 = row_g + 64 * rb;
        if (k0 > r0 || r0 >= n) continue;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          acc[rb][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[rb][u], b[u][0], acc[rb][0], 0, 0, 0);
          acc[rb][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[rb][u], b[u][1], acc[rb][1], 0, 0, 0);
        }
      }
    }
  }
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    double s = 0.0;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int t = 0; t < 4; ++t) s += acc[rb][c][t] * acc[rb][c][t];
    s += __shfl_xor(s, 16);
    s += __shfl_xor(s, 32);
    if (lk == 0) red[w][16 * c + lr] = s;
  }
  __syncthreads();
  if (tid < PQ && q < m) part[size_t(g) * m + q] = (red[0][qi] + red[1][qi]) + (red[2][qi] + red[3][qi]);
  if (!tail) return;  // uniform
  __syncthreads();
  red[kk][qi] = sm;
  __syncthreads();
  if (tid < PQ && q < m) {
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < 8; ++k) s += red[k][qi];
    mean[q] = s * s_q;
  }
}

// Variances from the row groups' sums.
__global__ __launch_bounds__(256) void k_gp_predict_sum(int m, int groups, const double* __restrict__ part, double sf2,
                                                        double s_q, double* __restrict__ var) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= m) return;
  double s = 0.0;
  for (int g = 0; g < groups; ++g) s += part[size_t(g) * m + q];
  var[q] = (sf2 - s) * s_q * s_q;
}

// out[0] = y^T alpha, out[1] = sum log L_ii.
__global__ __launch_bounds__(256) void k_gp_lml(int n, int ld, const double* __restrict__ L,
                                                const double* __restrict__ y, const double* __restrict__ alpha,
                                                double* __restrict__ out) {
  __shared__ double r0[256], r1[256];
  double a = 0.0, b = 0.0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    a += y[i] * alpha[i];
    b += log(L[i + size_t(i) * ld]);
  }
  r0[threadIdx.x] = a;
  r1[threadIdx.x] = b;
  __syncthreads();
  for (int o = blockDim.x / 2; o > 0; o >>= 1) {
    if (threadIdx.x < o) {
      r0[threadIdx.x] += r0[threadIdx.x + o];
      r1[threadIdx.x] += r1[threadIdx.x + o];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[0] = r0[0];
    out[1] = r1[0];
  }
}

// ---------------------------------------------------------------------------
// Evidence of many hyperparameter sets at once (gp_optimize).
// ---------------------------------------------------------------------------
constexpr int EV_MAX = 256;   // sets of a launch: one per compute unit
constexpr int EV_LDS_N = 128; // points whose covariance one workgroup keeps in LDS

// State of the search on the device: logarithms of sigma_f, ell and sigma_n
// (scaled), the evidence there, and the bracket of the current line search.
struct EvState {
  double x[3], best, lo, hi;
};

// One round of a line search.  axis: parameter 0-2, -1 no line: set t is
// pts[t].  Round 0 opens the bracket at the current point +- width; a later
// round closes it around the best of the nb sets of the round before (between
// its neighbours); the last one takes that best where it beats the point the
// search started from.  Every wavefront that calls it computes the same.
struct EvLine {
  int axis, round, last, nb;
  double width;
  const double* pts;
  const EvState* in;
  EvState* out;
  const double* lml_in;
  double* lml_out;
};

__device__ __forceinline__ EvState ev_step(const EvLine& E) {
  EvState S = *E.in;
  if (E.round == 0) {
    S.lo = -E.width;
    S.hi = E.width;
    return S;
  }
  const int lane = threadIdx.x & 63;
  double f = -INFINITY;
  int at = 0;
  for (int t = lane; t < E.nb; t += 64) {  // largest, the first of equals
    const double v = E.lml_in[t];
    if (v > f) {
      f = v;
      at = t;
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const double v = __shfl_xor(f, o);
    const int w = __shfl_xor(at, o);
    if (v > f || (v == f && w < at)) {
      f = v;
      at = w;
    }
  }
  const double h = (S.hi - S.lo) / double(E.nb + 1), c = S.lo + double(at + 1) * h;
  if (E.last) {
    if (f >= S.best) {
#pragma unroll
      for (int k = 0; k < 3; ++k) S.x[k] += k == E.axis ? c : 0.0;
      S.best = f;
    }
  } else {
    S.lo = c - h;
    S.hi = c + h;
  }
  return S;
}

// sigma_f^2, 1 / 2 l^2 and sigma_n^2 of set t; block 0 of the launch keeps
// the state for the next one.
__device__ __forceinline__ void ev_set(const EvLine& E, int t, bool keep, double& sf2, double& i2l2, double& sn2) {
  double x[3];
  if (E.axis < 0) {
    for (int k = 0; k < 3; ++k) x[k] = E.pts[3 * t + k];
  } else {
    const EvState S = ev_step(E);
    if (keep) *E.out = S;
    const double c = S.lo + double(t + 1) * ((S.hi - S.lo) / double(E.nb + 1));
    for (int k = 0; k < 3; ++k) x[k] = S.x[k] + (k == E.axis ? c : 0.0);
  }
  sf2 = exp(2.0 * x[0]);
  i2l2 = 0.5 * exp(-2.0 * x[1]);
  sn2 = exp(2.0 * x[2]);
}

// Parameters of the sets of a round (panel elimination), or the end of a line
// search (E.last: the state only).
__global__ __launch_bounds__(EV_MAX) void k_gp_ev_line(EvLine E, double* __restrict__ par) {
  const int t = threadIdx.x;
  if (E.last) {
    const EvState S = ev_step(E);
    if (t == 0) *E.out = S;
    return;
  }
  double a, b, c;
  ev_set(E, t < E.nb ? t : 0, t == 0, a, b, c);
  if (t < E.nb) {
    par[3 * t] = a;
    par[3 * t + 1] = b;
    par[3 * t + 2] = c;
  }
}

// Evidence of set blockIdx.x by one workgroup (n <= EV_LDS_N): C with y as one
// more row, eliminated as L D L^T one column at a time -- only reciprocals of
// the pivots on the way, and
//   y^T C^-1 y = sum z_k^2 / d_k, log det C = sum log d_k
// need no back-substitution.  The matrix stays in registers: thread (tx, ty)
// of TX x 16 holds rows tx + TX a and columns ty + 16 b; LDS carries the
// current column (two buffers, one barrier a column).  What bounds it is the
// chain of a column (LDS, reciprocal, update, barrier): 22 us for 256 sets of
// 48 points, where one set took 82 us in eight launches and two read-backs.
template <int TX, int A, int B>
__global__ __launch_bounds__(TX * 16) void k_gp_ev_lds(int n, const double* __restrict__ X,
                                                       const double* __restrict__ y, KParams P,
                                                       const double* __restrict__ noise, EvLine E) {
  __shared__ double col[2][TX * A];
  __shared__ double piv[16 * B], zz[16 * B];
  const int tid = threadIdx.x, tx = tid % TX, ty = tid / TX;
  ev_set(E, blockIdx.x, blockIdx.x == 0 && tid == 0, P.sf2, P.inv_2l2, P.sn2);
  double v[A][B];
#pragma unroll
  for (int b = 0; b < B; ++b) {
    const int j = ty + 16 * b;
#pragma unroll
    for (int a = 0; a < A; ++a) {
      const int i = tx + TX * a;
      v[a][b] = 0.0;
      if (TX * (a + 1) <= 16 * b) continue;  // above the diagonal
      if (i >= j && j < n && i <= n) {
        if (i == n) {
          v[a][b] = y[j];
        } else {
          v[a][b] = sqexp(X + GP_MAXD * i, X + GP_MAXD * j, P);
          if (i == j) v[a][b] += noise ? noise[i] : P.sn2;
        }
      }
      if (b == 0 && ty == 0) col[0][i] = v[a][0];
    }
  }
  __syncthreads();
  bool ok = true;
#pragma unroll
  for (int kb = 0; kb < B; ++kb) {
    for (int kk = 0; kk < 16; ++kk) {
      const int k = 16 * kb + kk;
      if (k >= n) break;  // uniform
      const double* const c = col[k & 1];
      const double d = c[k];
      ok = ok && d > 0.0;
      const double ri = reciprocal(d);
      if (tid == 0) {
        piv[k] = d;
        zz[k] = c[n];
      }
      double ci[A];
#pragma unroll
      for (int a = 0; a < A; ++a) ci[a] = c[tx + TX * a];
      double* const nx = col[(k + 1) & 1];
#pragma unroll
      for (int b = kb; b < B; ++b) {
        const double fj = c[ty + 16 * b] * ri;  // columns up to k are not used again
#pragma unroll
        for (int a = 0; a < A; ++a) {
          if (TX * (a + 1) <= 16 * b) continue;
          v[a][b] = fma(-ci[a], fj, v[a][b]);
        }
        if (b <= kb + 1 && ty + 16 * b == k + 1) {
#pragma unroll
          for (int a = 0; a < A; ++a) nx[tx + TX * a] = v[a][b];
        }
      }
      __syncthreads();
    }
  }
  if (tid < 64) {
    double q = 0.0, lg = 0.0;
    for (int k = tid; k < n; k += 64) {
      q += zz[k] * zz[k] / piv[k];
      lg += log(piv[k]);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      q += __shfl_xor(q, o);
      lg += __shfl_xor(lg, o);
    }
    if (tid == 0) E.lml_out[blockIdx.x] = ok ? -0.5 * q - 0.5 * lg - 0.5 * double(n) * log(2.0 * M_PI) : -INFINITY;
  }
}

// Evidence of set blockIdx.x from its factor and the y row of S.
__global__ __launch_bounds__(256) void k_gp_ev_sum(int n, Chol M, double* __restrict__ lml) {
  __shared__ double red[2][4];
  const double* const A = M.A + blockIdx.x * M.stride;
  const int tid = threadIdx.x;
  double q = 0.0, lg = 0.0;
  for (int k = tid; k < n; k += blockDim.x) {
    const double z = A[size_t(M.nt) * TB + size_t(k) * M.ld];
    q += z * z;
    lg += log(A[k + size_t(k) * M.ld]);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    q += __shfl_xor(q, o);
    lg += __shfl_xor(lg, o);
  }
  if ((tid & 63) == 0) {
    red[0][tid >> 6] = q;
    red[1][tid >> 6] = lg;
  }
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < 4; ++w) {
      q += red[0][w];
      lg += red[1][w];
    }
    lml[blockIdx.x] = M.info[blockIdx.x] == 0 ? -0.5 * q - lg - 0.5 * double(n) * log(2.0 * M_PI) : -INFINITY;
  }
}

// New last row of L for the point at index n: row = L^-1 c, then the pivot.
__global__ __launch_bounds__(1024) void k_gp_append_row(int n, int ld, const double* __restrict__ X, KParams P,
                                                        double* __restrict__ L, double* __restrict__ row,
                                                        int* __restrict__ info) {
  __shared__ double xk;
  __shared__ double red[1024];
  const int tid = threadIdx.x, nt = blockDim.x;
  for (int i = tid; i < n; i += nt) row[i] = sqexp(X + GP_MAXD * i, X + GP_MAXD * n, P);
  __syncthreads();
  for (int k = 0; k < n; ++k) {
    if (tid == 0) {
      xk = row[k] / L[k + size_t(k) * ld];
      row[k] = xk;
    }
    __syncthreads();
    for (int i = k + 1 + tid; i < n; i += nt) row[i] -= L[i + size_t(k) * ld] * xk;
    __syncthreads();
  }
  double s = 0.0;
  for (int i = tid; i < n; i += nt) {
    s += row[i] * row[i];
    L[n + size_t(i) * ld] = row[i];
  }
  red[tid] = s;
  __syncthreads();
  for (int o = nt / 2; o > 0; o >>= 1) {
    if (tid < o) red[tid] += red[tid + o];
    __syncthreads();
  }
  if (tid == 0) {
    const double c = P.sf2 + P.sn2 - red[0];
    if (c > 0.0) {
      L[n + size_t(n) * ld] = sqrt(c);
      *info = 0;
    } else {
      *info = n + 1;
    }
  }
}

KParams kparams(const hmd_gp* g) {
  KParams P{};
  for (int k = 0; k < GP_MAXD; ++k) P.inv_scale[k] = k < g->d ? 1.0 / g->scale[k] : 0.0;
  P.sf2 = g->hyp.sigma_f * g->hyp.sigma_f;
  P.inv_2l2 = 1.0 / (2.0 * g->hyp.ell * g->hyp.ell);
  P.sn2 = g->sigma_n * g->sigma_n;
  P.d = g->d;
  P.kind = g->hyp.kernel;
  P.pi_over_T = g->hyp.kernel == 1 ? M_PI / g->hyp.period : 0.0;
  return P;
}

// Normalisation of Eq. d2Eq and the output scale (host, FP64).
void normalise(hmd_gp* g) {
  const int n = g->n, d = g->d;
  for (int k = 0; k < d; ++k) {
    const double fallback = 0.25 * g->hyp.range[k];
    double m = 0.0;
    if (g->hyp.scale_mode == 0 && n >= 2) {
      // sum of |x_i - x_j| over pairs: in ascending order, x_i is the larger
      // of i pairs; from the smallest value on, so that no part cancels
      std::vector<double> v(n);
      bool ordered = true;  // a NaN has no place in the order: its mean distance is none either
      for (int i = 0; i < n; ++i) {
        v[i] = g->X[size_t(i) * d + k];
        ordered = ordered && v[i] == v[i];
      }
      if (ordered) {
        std::sort(v.begin(), v.end());
        double s = 0.0;
        for (int i = 1; i < n; ++i) s += (v[i] - v[i - 1]) * (double(i) * double(n - i));
        m = s / (0.5 * double(n) * double(n - 1));
      }
    }
    g->scale[k] = m > 0.0 ? m : fallback;
  }
  g->s_q = 1.0;
  if (g->hyp.out_scale && n > 0) {
    double s = 0.0;
    for (double v : g->y) s += v * v;
    s = std::sqrt(s / double(n));
    if (s > 0.0) g->s_q = s;
  }
  if (g->hyp.sigma_n >= 0.0) {
    g->sigma_n = g->hyp.sigma_n / g->s_q;
  } else {
    double s = 0.0;
    for (double v : g->se) s += v;
    g->sigma_n = n > 0 ? (s / double(n)) / g->s_q : 0.0;
  }
}

// Device memory for `need` points: one allocation, grown by doubling.
int reserve(hmd_gp* g, int need) {
  hmd_ctx* ctx = g->ctx;
  if (need <= g->cap) return HMD_OK;
  int cap = g->cap > 0 ? g->cap : 64;
  while (cap < need) cap *= 2;
  if (g->slab) (void)hipFree(g->slab);
  g->slab = nullptr;
  g->cap = 0;
  const int ld = cap + TB;
  const size_t mat = size_t(ld) * cap;
  HMD_HIP(ctx, hipMalloc(&g->slab, sizeof(double) * (2 * mat + size_t(TB) * cap + size_t(GP_MAXD + 5) * cap)));
  g->dL = g->slab;
  g->dLi = g->dL + mat;
  g->ddinv = g->dLi + mat;
  g->dalpha = g->ddinv + size_t(TB) * cap;
  g->dtmp = g->dalpha + cap;
  g->dX = g->dtmp + 2 * cap;  // inputs, outputs and noise variances, packed by upload_db
  g->cap = cap;
  g->ld = ld;
  return HMD_OK;
}

// Database to the device as one copy: inputs (padded to GP_MAXD columns),
// scaled outputs, noise variances.  The host buffer lives as long as the GP,
// and every call that comes here waits for the stream before it returns.
int upload_db(hmd_gp* g) {
  hmd_ctx* ctx = g->ctx;
  const size_t n = size_t(g->n);
  g->stage.assign((GP_MAXD + 2) * n, 0.0);
  for (size_t i = 0; i < n; ++i) {
    for (int k = 0; k < g->d; ++k) g->stage[i * GP_MAXD + k] = g->X[i * g->d + k];
    g->stage[GP_MAXD * n + i] = g->y[i] / g->s_q;
    const double e = g->se[i] / g->s_q;
    g->stage[(GP_MAXD + 1) * n + i] = e * e;
  }
  g->dy = g->dX + GP_MAXD * n;
  g->dnoise = g->dy + n;
  HMD_HIP(ctx, hipMemcpyAsync(g->dX, g->stage.data(), 8 * g->stage.size(), hipMemcpyHostToDevice, ctx->stream));
  return HMD_OK;
}

// After a row was appended to L: the weights, and L^-1's new row.
int solve_alpha(hmd_gp* g) {
  hmd_ctx* ctx = g->ctx;
  hipStream_t s = ctx->stream;
  HMD_HIP(ctx, hipMemcpyAsync(g->dalpha, g->dy, 8 * size_t(g->n), hipMemcpyDeviceToDevice, s));
  hipLaunchKernelGGL(k_gp_solve, dim3(1), dim3(1024), 0, s, g->n, g->ld, g->dL, g->dalpha, 1);
  HMD_HIP(ctx, hipGetLastError());
  hipLaunchKernelGGL(k_gp_inv_append_row, dim3((g->n + 3) / 4), dim3(256), sizeof(double) * size_t(g->n), s, g->n - 1,
                     g->ld, g->dL, g->dLi);
  HMD_HIP(ctx, hipGetLastError());
  return HMD_OK;
}

// Queues covariance and elimination of M's problems (`nb` of them).
template <bool INV>
void enqueue_factor(const hmd_gp* g, const Chol& M, int nb, const double* par, double* alpha) {
  hipStream_t s = g->ctx->stream;
  const int nt = M.nt;
  hipLaunchKernelGGL(k_gp_cov<INV>, dim3((nt + 1) * (nt + 2) / 2, nb), dim3(256), 0, s, g->n, g->dX, g->dy, kparams(g),
                     par, g->hyp.noise_mode == 1 ? g->dnoise : nullptr, M);
  for (int p = 0; p <= nt; ++p) {
    const int i0 = INV ? std::max(p - 1, 0) : p;
    hipLaunchKernelGGL(k_gp_panel<INV>, dim3((nt + 1) * (nt + 2) / 2 - i0 * (i0 + 1) / 2, nb), dim3(256), 0, s, p, M,
                       alpha);
  }
}

// Full refit: normalisation, covariance, factorisation, weights and L^-1
// (upload false: the database and its scaling are already on the device).
int refit(hmd_gp* g, bool upload = true) {
  hmd_ctx* ctx = g->ctx;
  if (upload) normalise(g);
  if (g->n == 0) return HMD_OK;
  int rc = reserve(g, g->n);
  if (rc != HMD_OK) return rc;
  if (upload && (rc = upload_db(g)) != HMD_OK) return rc;
  const Chol M{g->dL, g->dLi, g->ddinv, g->dinfo, g->ld, (g->n + TB - 1) / TB, 0, 0};
  enqueue_factor<true>(g, M, 1, nullptr, g->dalpha);
  HMD_HIP(ctx, hipGetLastError());
  int info = 0;
  HMD_HIP(ctx, hipMemcpyAsync(&info, g->dinfo, sizeof(int), hipMemcpyDeviceToHost, ctx->stream));
  HMD_HIP(ctx, hipStreamSynchronize(ctx->stream));
  if (info != 0) {
    ctx->err = "gp: covariance not positive definite at pivot " + std::to_string(info - 1);
    return HMD_ENOTSPD;
  }
  return HMD_OK;
}

// Queues the predictions at m device queries (row-major, d columns).  Few
// queries of a small database: a workgroup each, the shortest chain (its work
// grows as m n^2, 13 us a call at 200 x 256, where the tiles' chain of barriers
// and exponentials alone is about 20 us), with four threads a row as far as
// two workgroups per compute unit go, with two up to twice that (513 queries of
// 256 points: 18 us, 24 with four, 26 by tiles; 1,024: 24, 32 and 27; 1,100:
// 28, 39 and 27).  Else the matrix cores (512 queries of 512 points: 45 us by
// workgroups, 48 by tiles; of 513: 59 and 52; 513 of 300: 26 with two threads a
// row and 33 by tiles, 800 of 300: 37 and 33), in row groups of 256 where that
// fills the chip, of 64 where it does not.
int enqueue_predict(hmd_gp* g, int m, const double* dXq, double* dmean, double* dvar, hipStream_t s) {
  hmd_ctx* ctx = g->ctx;
  const int n = g->n;
  const KParams P = kparams(g);
  if (n <= 512 && m <= 512) {
    hipLaunchKernelGGL(k_gp_predict<4>, dim3(m), dim3(1024), sizeof(double) * size_t(n), s, n, g->ld, g->dX, dXq,
                       g->dLi, g->dalpha, P, g->s_q, dmean, dvar);
    HMD_HIP(ctx, hipGetLastError());
    return HMD_OK;
  }
  if (n <= 256 && m <= 1024) {
    hipLaunchKernelGGL(k_gp_predict<2>, dim3(m), dim3(512), sizeof(double) * size_t(n), s, n, g->ld, g->dX, dXq,
                       g->dLi, g->dalpha, P, g->s_q, dmean, dvar);
    HMD_HIP(ctx, hipGetLastError());
    return HMD_OK;
  }
  const int qb = (m + PQ - 1) / PQ;
  const bool wide = int64_t(qb) * ((n + 255) / 256) >= 512;
  const int rows = wide ? 256 : 64, groups = (n + rows - 1) / rows;
  // scratch for any size of the database up to its reserved columns and for
  // any fewer queries (groups of 64 rows: fewer than 512 workgroups of 256 rows
  // by 32 queries): once a call of m queries has run, calls of up to m allocate
  // nothing until the database outgrows its columns, so that they can be
  // captured, and graphs that hold the scratch stay valid
  const size_t cols = size_t(g->cap);
  const size_t need = std::max((cols + 255) / 256 * m, std::min<size_t>((cols + 63) / 64 * m, 4 * 512 * PQ));
  if (need > g->part_cap) {
    HMD_HIP(ctx, hipStreamSynchronize(s));  // the old scratch may still be read
    if (g->dpart) (void)hipFree(g->dpart);
    g->dpart = nullptr;
    g->part_cap = 0;
    HMD_HIP(ctx, hipMalloc(&g->dpart, sizeof(double) * need));
    g->part_cap = need;
  }
  if (wide)
    hipLaunchKernelGGL(k_gp_predict_tiles<4>, dim3(qb, groups), dim3(256), 0, s, n, g->ld, g->dX, m, dXq, g->dLi,
                       g->dalpha, P, g->s_q, g->dpart, dmean);
  else
    hipLaunchKernelGGL(k_gp_predict_tiles<1>, dim3(qb, groups), dim3(256), 0, s, n, g->ld, g->dX, m, dXq, g->dLi,
                       g->dalpha, P, g->s_q, g->dpart, dmean);
  hipLaunchKernelGGL(k_gp_predict_sum, dim3((m + 255) / 256), dim3(256), 0, s, m, groups, g->dpart, P.sf2, g->s_q,
                     dvar);
  HMD_HIP(ctx, hipGetLastError());
  return HMD_OK;
}

}  // namespace
}  // namespace hmd

using namespace hmd;

extern "C" {

void hmd_gp_hyper_default(hmd_gp_hyper* h) {
  if (!h) return;
  h->sigma_f = 1.0;
  h->ell = 1.0;
  h->sigma_n = -1.0;
  h->scale_mode = 0;
  h->range[0] = 16.0;   // channel heights 4..20
  h->range[1] = 0.049;  // body forces 0.001..0.05
  h->range[2] = 1.0;
  h->range[3] = 1.0;
  h->out_scale = 1;
  h->noise_mode = 0;
  h->kernel = 0;
  h->period = 1.0;
}

int gp_fit(hmd_ctx* ctx, const double* X, const double* y, const double* y_se, int n, int d,
           const hmd_gp_hyper* hyper, hmd_gp** out) {
  if (!ctx || !out || n < 0 || n > GP_MAXN || d < 1 || d > GP_MAXD || (n > 0 && (!X || !y))) {
    if (ctx) ctx->err = "gp_fit: bad arguments (1 <= d <= 4, 0 <= n <= 6144)";
    return HMD_EINVAL;
  }
  HMD_HIP(ctx, hipSetDevice(ctx->device));
  auto* g = new hmd_gp();
  g->ctx = ctx;
  if (hyper) g->hyp = *hyper;
  else hmd_gp_hyper_default(&g->hyp);
  if (!(g->hyp.sigma_f > 0.0) || !(g->hyp.ell > 0.0) || g->hyp.noise_mode < 0 || g->hyp.noise_mode > 1 ||
      g->hyp.kernel < 0 || g->hyp.kernel > 1 || (g->hyp.kernel == 1 && (d != 1 || !(g->hyp.period > 0.0)))) {
    delete g;
    ctx->err = "gp_fit: sigma_f, ell positive; noise_mode 0/1; kernel 0, or 1 (periodic) with d = 1 and period > 0";
    return HMD_EINVAL;
  }
  g->d = d;
  g->n = n;
  g->X.assign(X, X + size_t(n) * d);
  g->y.assign(y, y + n);
  g->se.assign(n, 0.0);
  if (y_se) g->se.assign(y_se, y_se + n);
  if (hipMalloc(&g->dinfo, sizeof(int)) != hipSuccess || hipMalloc(&g->dout, sizeof(double) * 4) != hipSuccess) {
    gp_free(g);
    ctx->err = "gp_fit: device allocation failed";
    return HMD_ENOMEM;
  }
  const int rc = refit(g);
  if (rc != HMD_OK) {
    gp_free(g);
    return rc;
  }
  HMD_HIP(ctx, hipStreamSynchronize(ctx->stream));
  *out = g;
  return HMD_OK;
}

int gp_append(hmd_gp* g, const double* x, double y, double y_se) {
  if (!g || !x) return HMD_EINVAL;
  hmd_ctx* ctx = g->ctx;
  if (g->n >= GP_MAXN) {
    ctx->err = "gp_append: the database holds at most 6144 points";
    return HMD_EINVAL;
  }
  HMD_HIP(ctx, hipSetDevice(ctx->device));
  g->X.insert(g->X.end(), x, x + g->d);
  g->y.push_back(y);
  g->se.push_back(y_se);
  g->n += 1;
  // fixed normalisation, fixed noise and no output scaling: extend L by one
  // row; otherwise the normalisation moved and the factor is rebuilt
  const bool rank1 = (g->hyp.scale_mode == 1 || g->hyp.kernel == 1) && g->hyp.out_scale == 0 &&
                     (g->hyp.sigma_n >= 0.0 || g->hyp.noise_mode == 1) && g->n >= 2 && g->n <= g->cap;
  // returns with the factor, weights and L^-1 complete, so that a following
  // prediction on any stream sees them
  auto full_refit = [&]() -> int {
    const int r = refit(g);
    if (r != HMD_OK) return r;
    HMD_HIP(ctx, hipStreamSynchronize(ctx->stream));
    return HMD_OK;
  };
  if (!rank1) return full_refit();
  normalise(g);
  int rc = upload_db(g);
  if (rc != HMD_OK) return rc;
  hipStream_t s = ctx->stream;
  KParams P1 = kparams(g);
  if (g->hyp.noise_mode == 1) {
    const double e = y_se / g->s_q;
    P1.sn2 = e * e;
  }
  hipLaunchKernelGGL(k_gp_append_row, dim3(1), dim3(1024), 0, s, g->n - 1, g->ld, g->dX, P1, g->dL, g->dtmp,
                     g->dinfo);
  int info = 0;
  HMD_HIP(ctx, hipMemcpyAsync(&info, g->dinfo, sizeof(int), hipMemcpyDeviceToHost, s));
  HMD_HIP(ctx, hipStreamSynchronize(s));
  if (info != 0) return full_refit();
  rc = solve_alpha(g);
  if (rc != HMD_OK) return rc;
  HMD_HIP(ctx, hipStreamSynchronize(s));
  return HMD_OK;
}

int gp_predict(hmd_gp* g, const double* Xs, int m, double* mean, double* var) {
  if (!g || m < 0 || (m > 0 && (!Xs || !mean || !var))) return HMD_EINVAL;
  hmd_ctx* ctx = g->ctx;
  if (m == 0) return HMD_OK;
  const double sf2 = g->hyp.sigma_f * g->hyp.sigma_f;
  if (g->n == 0) {  // prior: zero mean, signal variance
    for (int q = 0; q < m; ++q) {
      mean[q] = 0.0;
      var[q] = sf2 * g->s_q * g->s_q;
    }
    return HMD_OK;
  }
  HMD_HIP(ctx, hipSetDevice(ctx->device));
  // queries, means and variances
  const size_t nq = size_t(g->d) * m, need = nq + 2 * size_t(m);
  if (need > g->q_cap) {
    if (g->dq) (void)hipFree(g->dq);
    g->dq = nullptr;
    g->q_cap = 0;
    HMD_HIP(ctx, hipMalloc(&g->dq, sizeof(double) * 2 * need));
    g->q_cap = 2 * need;
  }
  double* const dres = g->dq + nq;
  std::vector<double> res(2 * size_t(m));
  hipStream_t s = ctx->stream;
  HMD_HIP(ctx, hipMemcpyAsync(g->dq, Xs, 8 * nq, hipMemcpyHostToDevice, s));
  HMD_TRY(enqueue_predict(g, m, g->dq, dres, dres + m, s));
  HMD_HIP(ctx, hipMemcpyAsync(res.data(), dres, 8 * res.size(), hipMemcpyDeviceToHost, s));
  HMD_HIP(ctx, hipStreamSynchronize(s));
  std::copy(res.begin(), res.begin() + m, mean);
  std::copy(res.begin() + m, res.end(), var);
  return HMD_OK;
}

int gp_predict_dev(hmd_gp* g, const double* dXs, int m, double* dmean, double* dvar, void* stream) {
  if (!g || m < 0 || (m > 0 && (!dXs || !dmean || !dvar))) return HMD_EINVAL;
  hmd_ctx* ctx = g->ctx;
  if (m == 0) return HMD_OK;
  HMD_HIP(ctx, hipSetDevice(ctx->device));
  hipStream_t s = stream ? static_cast<hipStream_t>(stream) : ctx->stream;
  if (g->n > 0) return enqueue_predict(g, m, dXs, dmean, dvar, s);
  const double sf2 = g->hyp.sigma_f * g->hyp.sigma_f;
  hipLaunchKernelGGL(k_gp_prior, dim3((m + 255) / 256), dim3(256), 0, s, m, sf2 * g->s_q * g->s_q, dmean, dvar);
  HMD_HIP(ctx, hipGetLastError());
  return HMD_OK;
}

int gp_log_marginal(hmd_gp* g, double* lml) {
  if (!g || !lml) return HMD_EINVAL;
  hmd_ctx* ctx = g->ctx;
  if (g->n == 0) {
    *lml = 0.0;
    return HMD_OK;
  }
  HMD_HIP(ctx, hipSetDevice(ctx->device));
  hipStream_t s = ctx->stream;
  hipLaunchKernelGGL(k_gp_lml, dim3(1), dim3(256), 0, s, g->n, g->ld, g->dL, g->dy, g->dalpha, g->dout);
  double h[2];
  HMD_HIP(ctx, hipMemcpyAsync(h, g->dout, sizeof(h), hipMemcpyDeviceToHost, s));
  HMD_HIP(ctx, hipStreamSynchronize(s));
  *lml = -0.5 * h[0] - h[1] - 0.5 * double(g->n) * std::log(2.0 * M_PI);
  return HMD_OK;
}

// Hyperparameters that maximise Eq. evidenceEq (Sec. 2.3; App. B).  The
// evidence can have several local maxima (the periodic kernel's has in ell),
// so the search first evaluates it on a grid of 17 points per chosen
// parameter, a quarter decade apart over two decades either side of the
// start, then refines from the best grid point by cyclic line searches over
// the logarithm of each chosen parameter, bracketed at first by a factor 10
// around the current value and then by 32 times the last cycle's move, until
// a cycle gains less than 1e-12 relative (at most 30 cycles).
//
// Refits are independent of each other, so a whole grid, or a round of up to
// 256 points along a line, is one set of launches: a line search closes its
// bracket by (nb + 1) / 2 per round, three to five rounds where golden sections
// took 63 refits in turn.  (Searching along the way a cycle came as well
// converges in a third of the rounds, but where the cycles end at their limit
// on a flat ridge it ends elsewhere, by up to 1e-3 in sigma_f.)  The rounds of a
// cycle are queued without waiting for the host.  Up to EV_LDS_N points a set
// is one workgroup; beyond, the panel elimination runs on all sets at once, as
// many as a workspace of kEvBytes holds.
int gp_optimize(hmd_gp* g, int mask, double* lml) {
  if (!g || mask <= 0 || mask > 7) return HMD_EINVAL;
  hmd_ctx* ctx = g->ctx;
  if (g->n < 1 || ((mask & 4) && g->hyp.noise_mode == 1)) {
    ctx->err = "gp_optimize: needs data, and sigma_n only with uniform noise";
    return HMD_EINVAL;
  }
  HMD_HIP(ctx, hipSetDevice(ctx->device));
  hipStream_t s = ctx->stream;
  const int n = g->n, nt = (n + TB - 1) / TB, ld = (nt + 1) * TB;
  if (mask & 4) g->hyp.sigma_n = g->sigma_n * g->s_q;  // held explicitly from here on
  normalise(g);
  HMD_TRY(reserve(g, n));
  HMD_TRY(upload_db(g));
  // device buffers of the search, released on every return
  struct Work {
    double *A = nullptr, *dinv = nullptr, *small = nullptr;
    int* info = nullptr;
    ~Work() {
      for (void* p : {(void*)A, (void*)dinv, (void*)small, (void*)info})
        if (p) (void)hipFree(p);
    }
  } w;
  // parameters, points, two evidence buffers and two states
  HMD_HIP(ctx, hipMalloc(&w.small, sizeof(double) * 8 * EV_MAX + 2 * sizeof(EvState)));
  double* const par = w.small;
  double* const pts_dev = w.small + 3 * EV_MAX;
  double* const lml_dev[2] = {w.small + 6 * EV_MAX, w.small + 7 * EV_MAX};
  EvState* const st_dev = reinterpret_cast<EvState*>(w.small + 8 * EV_MAX);
  int nb = EV_MAX;
  Chol M{};
  if (n > EV_LDS_N) {
    constexpr double kEvBytes = 8.0 * 1024 * 1024 * 1024;
    M.ld = ld;
    M.nt = nt;
    M.stride = size_t(ld) * nt * TB;
    M.dstride = size_t(nt) * TB * TB;
    nb = int(std::min(double(EV_MAX), std::max(3.0, kEvBytes / (8.0 * double(M.stride + M.dstride)))));
    while (hipMalloc(&w.A, sizeof(double) * M.stride * nb) != hipSuccess) {
      w.A = nullptr;
      (void)hipGetLastError();
      if (nb == 3) {
        ctx->err = "gp_optimize: device allocation failed";
        return HMD_ENOMEM;
      }
      nb = std::max(3, nb / 2);
    }
    HMD_HIP(ctx, hipMalloc(&w.dinv, sizeof(double) * M.dstride * nb));
    HMD_HIP(ctx, hipMalloc(&w.info, sizeof(int) * nb));
    M.A = w.A;
    M.dinv = w.dinv;
    M.info = w.info;
  }
  int flip = 0;  // states and evidences alternate between launches
  auto line = [&](int axis, int round, int last, int m, double width) {
    return EvLine{axis, round, last, m, width, pts_dev, st_dev + flip, st_dev + 1 - flip, lml_dev[flip],
                  lml_dev[1 - flip]};
  };
  const double* const noise = g->hyp.noise_mode == 1 ? g->dnoise : nullptr;
  // one round: its sets' evidences
  auto evaluate = [&](const EvLine& E) {
    if (n <= 64) {
      hipLaunchKernelGGL((k_gp_ev_lds<16, 5, 4>), dim3(E.nb), dim3(256), 0, s, n, g->dX, g->dy, kparams(g), noise, E);
    } else if (n <= EV_LDS_N) {
      hipLaunchKernelGGL((k_gp_ev_lds<32, 5, 8>), dim3(E.nb), dim3(512), 0, s, n, g->dX, g->dy, kparams(g), noise, E);
    } else {
      hipLaunchKernelGGL(k_gp_ev_line, dim3(1), dim3(EV_MAX), 0, s, E, par);
      enqueue_factor<false>(g, M, E.nb, par, nullptr);
      hipLaunchKernelGGL(k_gp_ev_sum, dim3(E.nb), dim3(256), 0, s, n, M, E.lml_out);
    }
    flip = 1 - flip;
  };
  EvState st{};
  st.x[0] = std::log(g->hyp.sigma_f);
  st.x[1] = std::log(g->hyp.ell);
  st.x[2] = g->sigma_n > 0.0 ? std::log(g->sigma_n) : -INFINITY;
  int idx[3], m = 0, total = 1;
  for (int k = 0; k < 3; ++k)
    if (mask & (1 << k)) {
      idx[m++] = k;
      total *= 17;
    }
  st.best = -INFINITY;
  {
    EvState top = st;
    std::vector<double> pts, val(nb);
    for (int p0 = 0; p0 < total; p0 += nb) {
      const int c = std::min(nb, total - p0);
      pts.assign(3 * size_t(c), 0.0);
      for (int p = 0; p < c; ++p) {
        double* const x = &pts[3 * size_t(p)];
        std::copy(st.x, st.x + 3, x);
        int r = p0 + p;
        for (int j = 0; j < m; ++j, r /= 17) x[idx[j]] += std::log(10.0) * (-2.0 + 0.25 * (r % 17));
      }
      HMD_HIP(ctx, hipMemcpyAsync(pts_dev, pts.data(), 8 * pts.size(), hipMemcpyHostToDevice, s));
      const EvLine E = line(-1, 0, 0, c, 0.0);
      evaluate(E);
      HMD_HIP(ctx, hipGetLastError());
      HMD_HIP(ctx, hipMemcpyAsync(val.data(), E.lml_out, 8 * size_t(c), hipMemcpyDeviceToHost, s));
      HMD_HIP(ctx, hipStreamSynchronize(s));
      for (int p = 0; p < c; ++p)
        if (val[p] > top.best) {
          top.best = val[p];
          std::copy(&pts[3 * size_t(p)], &pts[3 * size_t(p)] + 3, top.x);
        }
    }
    st = top;
  }
  flip = 0;
  HMD_HIP(ctx, hipMemcpyAsync(st_dev, &st, sizeof(st), hipMemcpyHostToDevice, s));
  const double widest = std::log(10.0);
  double width = widest;
  for (int cycle = 0; cycle < 30; ++cycle) {
    const EvState before = st;
    // rounds that close the bracket below 1e-9
    const int rounds = std::max(1, int(std::ceil(std::log(2.0 * width / 1e-9) / std::log(0.5 * double(nb + 1)))));
    for (int j = 0; j < m; ++j) {
      for (int r = 0; r < rounds; ++r) evaluate(line(idx[j], r, 0, nb, width));
      hipLaunchKernelGGL(k_gp_ev_line, dim3(1), dim3(EV_MAX), 0, s, line(idx[j], rounds, 1, nb, width), par);
      flip = 1 - flip;
    }
    HMD_HIP(ctx, hipGetLastError());
    HMD_HIP(ctx, hipMemcpyAsync(&st, st_dev + flip, sizeof(st), hipMemcpyDeviceToHost, s));
    HMD_HIP(ctx, hipStreamSynchronize(s));
    if (std::fabs(st.best - before.best) <= 1e-12 * std::fabs(st.best)) break;
    double move = 0.0;
    for (int k = 0; k < m; ++k) move = std::max(move, std::fabs(st.x[idx[k]] - before.x[idx[k]]));
    width = std::min(widest, std::max(1e-6, 32.0 * move));
  }
  if (mask & 1) g->hyp.sigma_f = std::exp(st.x[0]);
  if (mask & 2) g->hyp.ell = std::exp(st.x[1]);
  if (mask & 4) {
    g->hyp.sigma_n = std::exp(st.x[2]) * g->s_q;
    g->sigma_n = g->hyp.sigma_n / g->s_q;
  }
  HMD_TRY(refit(g, false));  // at the kept values, with L^-1 for predictions
  if (lml) *lml = st.best;
  return HMD_OK;
}

int gp_hyper_get(const hmd_gp* g, hmd_gp_hyper* hyper) {
  if (!g || !hyper) return HMD_EINVAL;
  *hyper = g->hyp;
  return HMD_OK;
}

int gp_size(const hmd_gp* g) { return g ? g->n : 0; }

int gp_inputs(const hmd_gp* g, double* X, int* n, int* d) {
  if (!g) return HMD_EINVAL;
  if (n) *n = g->n;
  if (d) *d = g->d;
  if (X) std::copy(g->X.begin(), g->X.begin() + size_t(g->n) * g->d, X);
  return HMD_OK;
}

int gp_outputs(const hmd_gp* g, double* y, double* y_se) {
  if (!g) return HMD_EINVAL;
  if (y) std::copy(g->y.begin(), g->y.begin() + g->n, y);
  if (y_se) std::copy(g->se.begin(), g->se.begin() + g->n, y_se);
  return HMD_OK;
}

int gp_scales(const hmd_gp* g, double* scale, double* s_q, double* sigma_n) {
  if (!g) return HMD_EINVAL;
  if (scale)
    for (int k = 0; k < g->d; ++k) scale[k] = g->scale[k];
  if (s_q) *s_q = g->s_q;
  if (sigma_n) *sigma_n = g->sigma_n;
  return HMD_OK;
}

void gp_free(hmd_gp* g) {
  if (!g) return;
  for (void* p : {(void*)g->slab, (void*)g->dq, (void*)g->dpart, (void*)g->dout, (void*)g->dinfo})
    if (p) (void)hipFree(p);
  delete g;
}

}  // extern "C"

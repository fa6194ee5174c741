// series.hip -- mean and standard error of sampled time series on the device.
//
// The paper (Sec. 2.3, hyperparameters) takes the noise of an MD run as the
// standard deviation of its mean output computed from the raw
// time-instantaneous data.  The flux of a channel stays correlated for a
// viscous time ~h^2/nu (thousands of steps in wide channels), so the
// estimator must account for the correlation.  Default: the initial
// monotone sequence estimator of Geyer (Statistical Science 7 (1992) 473,
// Sec. 3.3) over the empirical autocovariances; alternative: the standard
// deviation of nb contiguous block means.
//
// Rows: S series of n samples each, row stride ld, every sample multiplied
// by `scale` (the MD series holds sums of B steps; scale = 1/B).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>

#include "engine.h"
#include "series.h"

namespace hmd {

namespace {

constexpr int SER_TPB = 256;

// Estimator state of a row between batches of lags, in lags 1-3 of its
// autocovariances (consumed by then; gamma_0 is still needed).
constexpr int kTotal = 1, kSmallest = 2, kDone = 3;

// Orders LDS accesses of a wavefront's lanes to each other's data.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace

// out[s*4 + 0] = mean, [2] = mean of the first n/2 samples, [3] = mean of
// the rest; [1] (the standard error) is left to the estimator kernels.  A long
// row is read by 16 wavefronts, four loads in flight each: latency bounds it
// (64 rows of 20,000: 23 us with four wavefronts, one load at a time).  Rows
// of fewer than four samples a thread take four wavefronts (65,535 rows of 16
// with the block rule: 126 us, 345 with sixteen).
constexpr int MOM_LONG = 4096;

template <int MOM_TPB>
__global__ __launch_bounds__(MOM_TPB) void k_series_moments(const double* __restrict__ x, int64_t ld, int64_t n,
                                                            double scale, double* __restrict__ out) {
  __shared__ double red[2][MOM_TPB / 64];
  const int s = blockIdx.x, tid = threadIdx.x;
  const double* row = x + int64_t(s) * ld;
  const int64_t half = n / 2;
  double sum[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int64_t end = h ? n : half;
    double a[4] = {0.0, 0.0, 0.0, 0.0};
    int64_t i = (h ? half : 0) + tid;
    for (; i + 3 * MOM_TPB < end; i += 4 * MOM_TPB) {
#pragma unroll
      for (int u = 0; u < 4; ++u) a[u] += row[i + u * MOM_TPB] * scale;
    }
    for (; i < end; i += MOM_TPB) a[0] += row[i] * scale;
    double v = (a[0] + a[1]) + (a[2] + a[3]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if ((tid & 63) == 0) red[h][tid >> 6] = v;
  }
  __syncthreads();
  if (tid == 0) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      sum[h] = 0.0;
      for (int w = 0; w < MOM_TPB / 64; ++w) sum[h] += red[h][w];
    }
    out[4 * s + 0] = (sum[0] + sum[1]) / double(n);
    out[4 * s + 2] = sum[0] / double(half);
    out[4 * s + 3] = sum[1] / double(n - half);
  }
}

// Everything of a short row by one wavefront: moments, then Geyer's estimator
// (see k_series_geyer) over 64 lags at a time, a lag per lane, each summed in
// ascending i from LDS, until the sequence ends.  The matrix form below works
// in pieces of 1024 samples and 304 lags, which rows of a few hundred samples
// leave empty (65,535 rows of 16: 57 us, 520 in matrix form).  What bounds it
// is the chain of a row's products and the LDS, two reads per product: for few
// rows it is the better one up to about 256 samples (a call with 64 random walks
// of 200: 14 against 23 us, of 384: 28 against 23), for many up to 512 (1,024
// white rows of 512 20 against 38 us, walks 45 against 39; 20,000 walks 297
// against 476).
constexpr int SHORT_N = 512;

bool short_rows(int S, int64_t n) { return n <= std::min(256 + S / 4, SHORT_N); }

__global__ __launch_bounds__(SER_TPB) void k_series_short(const double* __restrict__ x, int64_t ld, int n,
                                                         double scale, int S, double* __restrict__ out) {
  __shared__ double lds[SER_TPB / 64][SHORT_N + 64];
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6, s = blockIdx.x * (SER_TPB / 64) + w;
  if (s >= S) return;  // whole wavefronts
  double* const d = lds[w];
  const double* const row = x + int64_t(s) * ld;
  const int half = n / 2;
  double a = 0.0, b = 0.0;
  for (int i = l; i < n; i += 64) {
    const double v = row[i] * scale;
    d[i] = v;
    if (i < half) a += v;
    else b += v;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    a += __shfl_xor(a, o);
    b += __shfl_xor(b, o);
  }
  const double mean = (a + b) / double(n);
  for (int i = l; i < n; i += 64) d[i] -= mean;  // the lane's own
  d[n + l] = 0.0;
  wave_lds_fence();
  double total = 0.0, smallest = INFINITY, g0 = 0.0;
  bool any = false, stop = false;
  for (int t0 = 0; t0 < n && !stop; t0 += 64) {
    double g = 0.0;
#pragma unroll 8
    for (int i = 0; i < n - t0; ++i) g += d[i] * d[i + t0 + l];
    g /= double(n);
    if (t0 == 0) g0 = __shfl(g, 0);
    const double p = g + __shfl_down(g, 1);  // even lanes: a pair
    const bool even = (l & 1) == 0;
    const unsigned long long ends = __ballot(even && !(t0 + l + 1 < n && p > 0.0));
    const int c = ends ? __builtin_ctzll(ends) : 64;  // lanes of the sequence in this run
    stop = c < 64;
    any = any || c > 0;
    double m = even && l < c ? fmin(p, smallest) : INFINITY;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const double v = __shfl_up(m, o);
      if (l >= o) m = fmin(m, v);
    }
    double v = even && l < c ? m : 0.0;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    total += v;
    if (c > 0) smallest = __shfl(m, c - 1);
  }
  if (l != 0) return;
  double var = any ? -g0 + 2.0 * total : g0;
  if (!(var > 0.0)) var = g0;
  out[4 * s + 0] = mean;
  out[4 * s + 1] = sqrt(var / double(n));
  out[4 * s + 2] = a / double(half);
  out[4 * s + 3] = b / double(n - half);
}

// gamma_t = (1/n) sum_{i < n-t} d_i d_{i+t}, d = scale x - mean, on the FP64
// matrix cores.  With the series cut into pieces of 16 samples, X[m][r] =
// d_{16 m + r}, the products G_s = sum_m X[m][.]^T X[m + s][.] hold every lag:
// gamma_{16 s + u} n is the sum over r of G_s[r][r + u] (r + u < 16) and of
// G_{s+1}[r][r + u - 16].  Both operands of a 16 x 16 x 4 step are 64
// consecutive samples, read from LDS without conflict, and one read feeds
// 1024 products (a loop over lags made 64 of one, and the LDS bounded it at 13
// TFLOP/s).  64 rows of 20,000 samples correlated over 1000: 2.09 ms before,
// 0.2 ms with the batches below; what bounds a batch now is the matrix rate
// (2,432 lags of 64 rows in 0.125 ms, 50 TFLOP/s).
//
// A workgroup takes 4 NS shifts s, NS per wavefront, of one row: the lags
// 16 s0 .. 16 (s0 + 4 NS - 1) - 1, (the last shift only completes them).  NS =
// 5 wastes a twentieth of the products; 2 wastes an eighth and gives more
// workgroups where rows and lags are few.
//
// Rows that the estimator has finished with (see k_series_geyer) are skipped.
constexpr int AC_CH = 1024;  // samples per pass

template <int NS>
__global__ __launch_bounds__(SER_TPB, NS == 5 ? 4 : 6) void k_series_acov(const double* __restrict__ x, int64_t ld, int64_t n,
                                                        double scale, const double* __restrict__ mom,
                                                        double* __restrict__ gam, int64_t gld, int tile0) {
  using f64x4 = __attribute__((ext_vector_type(4))) double;
  constexpr int SH = 4 * NS, LAGS = 16 * (SH - 1);
  __shared__ double a[AC_CH], b[AC_CH + 16 * SH];
  const int s = blockIdx.y, tid = threadIdx.x, l = tid & 63, w = tid >> 6;
  double* const g = gam + int64_t(s) * gld;
  if (tile0 > 0 && g[kDone] != 0.0) return;
  const int64_t t0 = int64_t(tile0 + blockIdx.x) * LAGS;
  const double* row = x + int64_t(s) * ld;
  const double mean = mom[4 * s];
  f64x4 acc[NS];
#pragma unroll
  for (int k = 0; k < NS; ++k) acc[k] = f64x4{0.0, 0.0, 0.0, 0.0};
  for (int64_t i0 = 0; i0 + t0 < n; i0 += AC_CH) {
    __syncthreads();
#pragma unroll
    for (int e = tid; e < AC_CH; e += SER_TPB) a[e] = i0 + e < n ? row[i0 + e] * scale - mean : 0.0;
#pragma unroll
    for (int e = tid; e < AC_CH + 16 * SH; e += SER_TPB) {
      const int64_t i = i0 + t0 + e;
      b[e] = i < n ? row[i] * scale - mean : 0.0;
    }
    __syncthreads();
    auto products = [&](int end) {
      for (int c = 0; c < end; c += 64) {
        const double av = a[c + l];
#pragma unroll
        for (int k = 0; k < NS; ++k)
          acc[k] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, b[c + 16 * (w * NS + k) + l], acc[k], 0, 0, 0);
      }
    };
    // the last pass stops with the row (a call with 300 rows of 512: 38 -> 34 us)
    if (n - t0 - i0 >= AC_CH) products(AC_CH);
    else products(int(n - t0 - i0));
  }
  // lane l, element t holds G_s[4 t + l / 16][l % 16]: lag 16 s + r' - r.  Each
  // wavefront sums the 31 diagonals of its shifts (the samples are done with);
  // a lag has one of its shift and one of the next.  Shift after shift, with a
  // barrier each, this was most of a short row's time: 512 rows of 512 took 44 us,
  // 16 now
  __syncthreads();
  double* const st = a + 256 * w;  // a shift's 256 values
#pragma unroll
  for (int k = 0; k < NS; ++k) {
#pragma unroll
    for (int t = 0; t < 4; ++t) st[(4 * t + (l >> 4)) * 16 + (l & 15)] = acc[k][t];
    wave_lds_fence();
    const int u = l - 15;  // lag 16 (w NS + k) + u
    double v = 0.0;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const double x = st[r * 16 + min(max(r + u, 0), 15)];
      v += r + u >= 0 && r + u < 16 ? x : 0.0;
    }
    if (l < 31) b[(w * NS + k) * 32 + l] = v;
    wave_lds_fence();
  }
  __syncthreads();
  for (int e = tid; e < LAGS; e += SER_TPB) {
    const int u = e & 15;
    const double* const d = b + (e >> 4) * 32 + u;
    const double lag = d[15] + (u > 0 ? d[31] : 0.0);  // d[31]: the next shift's u - 16
    if (t0 + e < n) g[t0 + e] = lag / double(n);
  }
}

// Geyer's initial monotone sequence: Gamma_k = gamma_2k + gamma_2k+1 while
// positive, each replaced by the smallest so far; sigma^2 = -gamma_0 +
// 2 sum Gamma_k; SE = sqrt(sigma^2 / n).  An empty sequence, or a sigma^2
// that is not positive, falls back to the iid value gamma_0.  One wavefront
// per row, 64 pairs at a time (prefix minimum and sum across the lanes; one
// thread a row took 390 us over 20,000 samples).
//
// The lags come in batches (k0 .. k1 pairs); a row whose sequence ends in one
// is finished, and later batches of autocovariances skip it: the sequence of
// a flux ends after a few correlation times, and the lags past it are never
// formed.  Between batches the state stays in the row's own consumed lags.
__global__ __launch_bounds__(64) void k_series_geyer(double* __restrict__ gam, int64_t gld, int64_t n, int64_t k0,
                                                     int64_t k1, int last, double* __restrict__ out) {
  const int s = blockIdx.x, l = threadIdx.x;
  double* const g = gam + int64_t(s) * gld;
  if (k0 > 0 && g[kDone] != 0.0) return;
  double total = 0.0, smallest = INFINITY;
  if (k0 > 0) {
    total = g[kTotal];
    smallest = g[kSmallest];
  }
  bool stop = false;
  int64_t used = k0;
  auto pair = [&](int64_t k) { return k + l < k1 ? g[2 * (k + l)] + g[2 * (k + l) + 1] : -1.0; };
  double next = pair(k0);
  for (int64_t k = k0; k < k1 && !stop; k += 64) {
    const double p = next;
    next = pair(k + 64);
    const unsigned long long ends = __ballot(!(p > 0.0));
    const int c = ends ? __builtin_ctzll(ends) : 64;  // pairs of the sequence in this run
    double m = l < c ? fmin(p, smallest) : INFINITY;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const double v = __shfl_up(m, o);
      if (l >= o) m = fmin(m, v);
    }
    double v = l < c ? m : 0.0;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    total += v;
    if (c > 0) smallest = __shfl(m, c - 1);
    used += c;
    stop = c < 64 && k + c < k1;
  }
  if (l != 0) return;
  const double g0 = g[0];
  if (stop || last) {
    double var = used > 0 ? -g0 + 2.0 * total : g0;
    if (!(var > 0.0)) var = g0;
    out[4 * s + 1] = sqrt(var / double(n));
  }
  if (!last) {
    g[kTotal] = total;
    g[kSmallest] = smallest;
    g[kDone] = stop ? 1.0 : 0.0;
  }
}

// Block rule: nb contiguous blocks of floor(n / nb) samples (the remainder
// dropped from the front); mean and halves are those of the block means.
__global__ __launch_bounds__(SER_TPB) void k_series_blocks(const double* __restrict__ x, int64_t ld, int64_t n,
                                                          double scale, int nb, double* __restrict__ out) {
  __shared__ double bm[1024];
  const int s = blockIdx.x;
  const double* row = x + int64_t(s) * ld;
  const int64_t B = n / nb, r = n - int64_t(nb) * B;
  for (int j = threadIdx.x; j < nb; j += SER_TPB) {
    double acc = 0.0;
    for (int64_t k = 0; k < B; ++k) acc += row[r + int64_t(j) * B + k] * scale;
    bm[j] = acc / double(B);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double mean = 0.0;
    for (int j = 0; j < nb; ++j) mean += bm[j];
    mean /= double(nb);
    double var = 0.0;
    for (int j = 0; j < nb; ++j) var += (bm[j] - mean) * (bm[j] - mean);
    var /= double(nb - 1);
    const int h1 = nb / 2;
    double m1 = 0.0, m2 = 0.0;
    for (int j = 0; j < h1; ++j) m1 += bm[j];
    for (int j = h1; j < nb; ++j) m2 += bm[j];
    out[4 * s + 0] = mean;
    out[4 * s + 1] = sqrt(var / double(nb));
    out[4 * s + 2] = m1 / double(h1);
    out[4 * s + 3] = m2 / double(nb - h1);
  }
}

int series_stats_check(int S, int64_t n, int64_t ld, int n_blocks, std::string& err) {
  if (S < 1 || S > 65535 || n < 2 || ld < n || n_blocks < 0 || n_blocks == 1 || n_blocks > kSeriesMaxBlocks ||
      (n_blocks >= 2 && n < n_blocks)) {
    err = "series statistics: need 1..65535 rows of n >= 2 samples (row stride >= n) and n_blocks 0 or "
          "2..1024 with n >= n_blocks";
    return HMD_EINVAL;
  }
  return HMD_OK;
}

void series_stats_enqueue(hipStream_t st, const double* d_x, int S, int64_t n, int64_t ld, double scale,
                          int n_blocks, double* d_gam, double* d_out) {
  if (n_blocks == 0 && short_rows(S, n)) {
    constexpr int rows = SER_TPB / 64;
    hipLaunchKernelGGL(k_series_short, dim3((S + rows - 1) / rows), dim3(SER_TPB), 0, st, d_x, ld, int(n), scale, S,
                       d_out);
    return;
  }
  if (n >= MOM_LONG)
    hipLaunchKernelGGL(k_series_moments<1024>, dim3(S), dim3(1024), 0, st, d_x, ld, n, scale, d_out);
  else
    hipLaunchKernelGGL(k_series_moments<256>, dim3(S), dim3(256), 0, st, d_x, ld, n, scale, d_out);
  if (n_blocks >= 2) {
    hipLaunchKernelGGL(k_series_blocks, dim3(S), dim3(SER_TPB), 0, st, d_x, ld, n, scale, n_blocks, d_out);
    return;
  }
  // Batches of lag tiles: enough workgroups to fill the chip (narrow tiles four
  // per compute unit: a second batch's two launches cost more than the lags it
  // may save, 200 rows of 512 28 against 23 us a call), then twice as many lags
  // each time.  Where rows are few one batch holds every lag.
  const int64_t wide = 16 * (4 * 5 - 1), narrow = 16 * (4 * 2 - 1);
  const bool big = int64_t(S) * ((n + wide - 1) / wide) >= 512;
  const int64_t lags = big ? wide : narrow, tiles = (n + lags - 1) / lags, pairs = n / 2;
  int64_t step = std::max<int64_t>(2, ((big ? 512 : 1024) + S - 1) / S);
  for (int64_t t = 0; t < tiles; t += step, step = t) {
    // a last batch of a few tiles joins the one before (64 white rows of 1000:
    // 22.8 -> 19.5 us)
    if (tiles - t <= step + step / 4) step = tiles - t;
    const int64_t c = step;
    const dim3 grid{unsigned(c), unsigned(S), 1};
    if (big)
      hipLaunchKernelGGL(k_series_acov<5>, grid, dim3(SER_TPB), 0, st, d_x, ld, n, scale, d_out, d_gam, n, int(t));
    else
      hipLaunchKernelGGL(k_series_acov<2>, grid, dim3(SER_TPB), 0, st, d_x, ld, n, scale, d_out, d_gam, n, int(t));
    const bool last = t + c == tiles;
    hipLaunchKernelGGL(k_series_geyer, dim3(S), dim3(64), 0, st, d_gam, n, n, t * lags / 2,
                       last ? pairs : (t + c) * lags / 2, last ? 1 : 0, d_out);
  }
}

// ---------------------------------------------------------------------------
// Allocation-free form.  The autocovariance scratch lives in a fixed device
// array, one copy per GPU, held until the process ends.  Host code never
// passes the array's name to a kernel (on the host it is only a stand-in
// symbol): its device address is looked up once per device at context
// creation and that address is what the kernels receive.
// ---------------------------------------------------------------------------
namespace {

static __device__ __align__(256) double scratch[kNoAllocScratchDoubles];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[kMaxDevices] = {};

}  // namespace

int series_noalloc_init(int device, std::string& err) {
  if (device < 0 || device >= kMaxDevices) {
    err = "series scratch: device index out of range";
    return HMD_EINVAL;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[device]) return HMD_OK;
  int prev = 0;
  if (hipGetDevice(&prev) != hipSuccess) prev = device;
  hipError_t e = hipSetDevice(device);
  void* ptr = nullptr;
  if (e == hipSuccess) e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
  (void)hipSetDevice(prev);
  if (e != hipSuccess || !ptr) {
    err = std::string("series scratch: hipGetSymbolAddress: ") + hipGetErrorString(e);
    return HMD_EDEVICE;
  }
  g_scratch_ptr[device] = static_cast<double*>(ptr);
  return HMD_OK;
}

double* series_noalloc_scratch(int device) {
  if (device < 0 || device >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  return g_scratch_ptr[device];
}

}  // namespace hmd

extern "C" int md_series_stats_noalloc(hmd_ctx* ctx, const double* d_x, int S, int64_t n, int64_t ld, int n_blocks,
                                       double* d_out, void* stream) {
  if (!ctx || !d_x || !d_out) return HMD_EINVAL;
  HMD_TRY(hmd::series_stats_check(S, n, ld, n_blocks, ctx->err));
  const int64_t need = n_blocks == 0 ? int64_t(S) * n : 0;
  if (need > hmd::kNoAllocScratchDoubles) {
    ctx->err = "md_series_stats_noalloc: S * n = " + std::to_string(need) + " exceeds the fixed scratch of " +
               std::to_string(hmd::kNoAllocScratchDoubles) + " doubles";
    return HMD_EINVAL;
  }
  double* sc = hmd::series_noalloc_scratch(ctx->device);
  if (!sc) {
    ctx->err = "md_series_stats_noalloc: no scratch address for this device (context not set up)";
    return HMD_EDEVICE;
  }
  HMD_HIP(ctx, hipSetDevice(ctx->device));
  hipStream_t s = stream ? static_cast<hipStream_t>(stream) : ctx->stream;
  hmd::series_stats_enqueue(s, d_x, S, n, ld, 1.0, n_blocks, sc, d_out);
  HMD_HIP(ctx, hipGetLastError());
  return HMD_OK;
}

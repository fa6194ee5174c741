// ens.hip -- MLP deep ensemble on the device (a learned surrogate beside the
// paper's GP): members of 2 -> H -> H -> 1 tanh networks, FP32 weights and
// accumulation, trained full-batch on the mean squared error with Adam.
//
// Up to 256 points a member trains in one workgroup that keeps parameters,
// moments and activations on its compute unit for hundreds of iterations; larger
// sets are shared out over workgroups, two launches per iteration.  Either way
// the hidden layer's products run on the FP32 matrix cores.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <type_traits>
#include <vector>

#include "engine.h"

struct hmd_ens {
  hmd_ctx* ctx = nullptr;
  hmd_ens_cfg cfg{};
  int P = 0;                 // parameters per member
  double mu[2] = {0, 0}, sd[2] = {1, 1}, s_q = 1.0;
  float* dparams = nullptr;  // members x P
  std::vector<double> loss;  // final training loss per member
  std::vector<double> X, y;  // training set (host copy, for refits)
  // prediction buffers, grown on demand and kept for later calls
  double* dq = nullptr;      // queries, 2 per row
  float* dy = nullptr;       // members x queries outputs
  double* dout = nullptr;    // mean, std per query
  int qcap = 0;
};

namespace hmd {
namespace {

constexpr int ENS_TPB = 256;
constexpr int TRAIN_TPB = 512;
constexpr int CHUNK = 32;
constexpr int MAXH = 64;
constexpr int MAX_SHARES = 32;  // shared-out training: workgroups per member
constexpr int LOCAL_N = 256;    // points a member trains on within one workgroup (LDS: 2 x 256 x 68 floats)
constexpr int LOCAL_ITERS = 500;  // iterations per launch of that path

__host__ __device__ constexpr int nparams(int H) { return H * H + 5 * H + 1; }

using f32x4 = __attribute__((ext_vector_type(4))) float;

// One Adam step (Kingma & Ba 2015, beta = (0.9, 0.999), eps = 1e-8).
__device__ __forceinline__ void adam(float g, float c1, float c2, float lr, float& th, float& m, float& v) {
  m = 0.9f * m + 0.1f * g;
  v = 0.999f * v + 0.001f * g * g;
  th -= lr * (m * c1) / (sqrtf(v * c2) + 1e-8f);
}

// v + the value of lane ^ M within 16 lanes, M one of 1, 2, 7, 15 (which span all 16).
template <int M>
__device__ __forceinline__ float lane_xor(float v) {
  constexpr int ctrl = M == 1 ? 0xB1 : M == 2 ? 0x4E : M == 7 ? 0x141 : 0x140;
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, 0xf, 0xf, true));
}

// Sums of V values (4, 8 or 16) over 16 lanes: lane l receives the sum of
// value l % V.  Halving the set at each exchange takes 15 adds where V separate
// sums take 64.
template <int V>
__device__ __forceinline__ float sum_split(float (&v)[V], int l) {
  if constexpr (V < 16) {
#pragma unroll
    for (int i = 0; i < V; ++i) v[i] += lane_xor<15>(v[i]);
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = ((l & 8) ? v[i + 8] : v[i]) + lane_xor<15>((l & 8) ? v[i] : v[i + 8]);
  }
  if constexpr (V < 8) {
#pragma unroll
    for (int i = 0; i < V; ++i) v[i] += lane_xor<7>(v[i]);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = ((l & 4) ? v[i + 4] : v[i]) + lane_xor<7>((l & 4) ? v[i] : v[i + 4]);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) v[i] = ((l & 2) ? v[i + 2] : v[i]) + lane_xor<2>((l & 2) ? v[i] : v[i + 2]);
  return ((l & 1) ? v[1] : v[0]) + lane_xor<1>((l & 1) ? v[0] : v[1]);
}

// Iterations t0 + 1 .. t0 + iters of one member (a workgroup) on N <= LOCAL_N
// points; loss_out receives the loss at the parameters before the last step.
// With grad_out set the gradient is left there instead of being stepped along.
//
// Shared out over the chip, an iteration costs two launches and a trip of the
// gradient through memory (256 points, 64 units: 44 us on the VALU; fused into
// one launch and on the matrix cores 27 us, 15 of them the other workgroups'
// gradients arriving), far more than its arithmetic is worth on one compute
// unit.  Here a wavefront runs 16 points through both layers and back in
// registers: lane (point lane % 16, g = lane / 16) holds units 16 t + 4 g + u,
// which is how the 16 x 16 x 4 instructions leave a product transposed and
// also a layout they take the next operand in.  Only the hidden layer's
// gradient needs points as the contracted index; its operands pass through
// LDS, and the wavefront that forms one of its HT x HT tiles keeps that tile's
// parameters and moments.  19.7 us per iteration at 256 points and 64 units,
// bound by the matrix rate (10 us) and tanh of one compute unit; it falls with
// the points and units.
template <int HT>
__global__ __launch_bounds__(1024) void k_ens_local(int N, int H, const float* __restrict__ Xs,
                                                    const float* __restrict__ ys, const float* __restrict__ wts,
                                                    float* __restrict__ params, float* __restrict__ mom,
                                                    float* __restrict__ vel, int t0, int iters, float lr,
                                                    float* __restrict__ loss_out, float* __restrict__ grad_out) {
  constexpr int HP = 16 * HT, EP = HP + 4;  // row pitch: 16 rows' 4-float reads on different banks
  constexpr int V = HT == 3 ? 16 : 4 * HT;
  extern __shared__ float4 lds4[];
  float* const W2 = reinterpret_cast<float*>(lds4);  // HP rows
  float* const small = W2 + HP * EP;                 // W1 (x, y), b1, b2, W3: HP each; b3; two bias corrections
  float* const ha = small + 5 * HP + 4;              // first-layer activations, a row per point
  float* const da = ha + 16 * ((N + 15) / 16) * EP;  // second-layer residuals
  float* const part = ha;                            // per wavefront: sums for the small tensors
  constexpr int PART = 5 * HP + 4;
  const int P = nparams(H);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, g4 = 4 * (lane >> 4);
  const int member = blockIdx.x, nw = (N + 15) / 16;
  const size_t base = size_t(member) * P;
  const float invN = 1.0f / float(N);
  // this thread's parameters: four of W2 (owner wavefronts) and one of the small tensors
  const int to = wave / HT, ti = wave % HT;
  const bool owner = wave < HT * HT;
  float w_th[4], w_m[4], w_v[4], s_th = 0.f, s_m = 0.f, s_v = 0.f;
  int w_at[4], s_at = -1;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int o = 16 * to + g4 + u, i = 16 * ti + l16;
    w_at[u] = owner && o < H && i < H ? 3 * H + o * H + i : -1;
    const bool on = w_at[u] >= 0;
    w_th[u] = on ? params[base + w_at[u]] : 0.f;
    w_m[u] = on && t0 > 0 ? mom[base + w_at[u]] : 0.f;
    w_v[u] = on && t0 > 0 ? vel[base + w_at[u]] : 0.f;
    if (owner) W2[o * EP + i] = w_th[u];
  }
  if (tid <= 5 * HP) {
    const int what = tid / HP, o = tid % HP;
    if (what == 5) s_at = 5 * H + H * H;
    else if (o < H) s_at = what < 2 ? 2 * o + what : what == 2 ? 2 * H + o : (what - 3) * H + 3 * H + H * H + o;
    if (s_at >= 0) {
      s_th = params[base + s_at];
      if (t0 > 0) {
        s_m = mom[base + s_at];
        s_v = vel[base + s_at];
      }
    }
    small[tid] = s_th;
  }
  // this lane's point
  const int pt = 16 * wave + l16;
  const bool active = wave < nw, on = pt < N;
  const float x0 = on ? Xs[2 * pt] : 0.f, x1 = on ? Xs[2 * pt + 1] : 0.f, y = on ? ys[pt] : 0.f;
  // bootstrap: the point's count in this member's resample weights its squared
  // residual (the mean still over N)
  const float wt = !on ? 0.f : wts ? wts[size_t(member) * N + pt] : 1.0f;
  double p1 = 1.0, p2 = 1.0;  // beta^t
  if (tid == 0) {
    p1 = pow(0.9, double(t0));
    p2 = pow(0.999, double(t0));
  }
  float loss = 0.f;
  __syncthreads();
  for (int it = 0; it < iters; ++it) {
    float sums[5] = {}, gb3 = 0.f;
    if (active) {
      float h1[4 * HT];
      f32x4 z[HT];
#pragma unroll
      for (int t = 0; t < HT; ++t) {
        const int i = 16 * t + g4;
        const float4 wx = *reinterpret_cast<const float4*>(small + i);
        const float4 wy = *reinterpret_cast<const float4*>(small + HP + i);
        const float4 c = *reinterpret_cast<const float4*>(small + 2 * HP + i);
        const float4 d = *reinterpret_cast<const float4*>(small + 3 * HP + i);
        h1[4 * t] = tanhf(wx.x * x0 + wy.x * x1 + c.x);
        h1[4 * t + 1] = tanhf(wx.y * x0 + wy.y * x1 + c.y);
        h1[4 * t + 2] = tanhf(wx.z * x0 + wy.z * x1 + c.z);
        h1[4 * t + 3] = tanhf(wx.w * x0 + wy.w * x1 + c.w);
        *reinterpret_cast<float4*>(ha + pt * EP + i) =
            make_float4(h1[4 * t], h1[4 * t + 1], h1[4 * t + 2], h1[4 * t + 3]);
        z[t] = f32x4{d.x, d.y, d.z, d.w};
      }
#pragma unroll
      for (int t = 0; t < HT; ++t)
#pragma unroll
        for (int k = 0; k < HT; ++k) {
          const f32x4 a = *reinterpret_cast<const f32x4*>(W2 + (16 * t + l16) * EP + 16 * k + g4);
#pragma unroll
          for (int u = 0; u < 4; ++u) z[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u], h1[4 * k + u], z[t], 0, 0, 0);
        }
      float out = 0.f;
      f32x4 w3[HT];
#pragma unroll
      for (int t = 0; t < HT; ++t) {
        w3[t] = *reinterpret_cast<const f32x4*>(small + 4 * HP + 16 * t + g4);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          z[t][u] = tanhf(z[t][u]);
          out += w3[t][u] * z[t][u];
        }
      }
      out += __shfl_xor(out, 16);
      out += __shfl_xor(out, 32);
      const float r = out + small[5 * HP] - y;
      const float dout = on ? 2.0f * wt * r * invN : 0.f;
      loss = on ? wt * r * r : 0.f;
      gb3 = dout;
      gb3 += lane_xor<15>(gb3);
      gb3 += lane_xor<7>(gb3);
      gb3 += lane_xor<2>(gb3);
      gb3 += lane_xor<1>(gb3);
      float v[V];
      auto collect = [&](auto value) {
#pragma unroll
        for (int q = 0; q < V; ++q) v[q] = q < 4 * HT ? value(q) : 0.f;
        return sum_split<V>(v, l16);
      };
      sums[4] = collect([&](int q) { return dout * z[q / 4][q % 4]; });
#pragma unroll
      for (int t = 0; t < HT; ++t) {
#pragma unroll
        for (int u = 0; u < 4; ++u) z[t][u] = dout * w3[t][u] * (1.0f - z[t][u] * z[t][u]);
        *reinterpret_cast<f32x4*>(da + pt * EP + 16 * t + g4) = z[t];
      }
      sums[3] = collect([&](int q) { return z[q / 4][q % 4]; });
      f32x4 b[HT];
#pragma unroll
      for (int k = 0; k < HT; ++k) b[k] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < HT; ++t)
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int k = 0; k < HT; ++k)
            b[k] = __builtin_amdgcn_mfma_f32_16x16x4f32(W2[(16 * t + g4 + u) * EP + 16 * k + l16], z[t][u], b[k], 0, 0,
                                                        0);
#pragma unroll
      for (int q = 0; q < 4 * HT; ++q) h1[q] = b[q / 4][q % 4] * (1.0f - h1[q] * h1[q]);
      sums[0] = collect([&](int q) { return h1[q] * x0; });
      sums[1] = collect([&](int q) { return h1[q] * x1; });
      sums[2] = collect([&](int q) { return h1[q]; });
    }
    if (tid == 0) {
      p1 *= 0.9;
      p2 *= 0.999;
      small[5 * HP + 1] = float(1.0 / (1.0 - p1));
      small[5 * HP + 2] = float(1.0 / (1.0 - p2));
    }
    __syncthreads();
    const float a1 = small[5 * HP + 1], a2 = small[5 * HP + 2];
    if (owner) {
      f32x4 g = {0.f, 0.f, 0.f, 0.f};
      const float* dp = da + g4 * EP + 16 * to + l16;
      const float* hp = ha + g4 * EP + 16 * ti + l16;
      for (int c = 0; c < nw; ++c, dp += 16 * EP, hp += 16 * EP) {
#pragma unroll
        for (int u = 0; u < 4; ++u) g = __builtin_amdgcn_mfma_f32_16x16x4f32(dp[u * EP], hp[u * EP], g, 0, 0, 0);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (grad_out) {
          if (w_at[u] >= 0) grad_out[base + w_at[u]] = g[u];
        } else {
          adam(w_at[u] >= 0 ? g[u] : 0.f, a1, a2, lr, w_th[u], w_m[u], w_v[u]);
          W2[(16 * to + g4 + u) * EP + 16 * ti + l16] = w_th[u];
        }
      }
    }
    __syncthreads();
    if (active) {
      const int q = l16 % V, o = 16 * (q / 4) + g4 + q % 4;
      if (l16 < V && o < HP) {
#pragma unroll
        for (int j = 0; j < 5; ++j) part[wave * PART + j * HP + o] = sums[j];
      }
      if (lane == 0) part[wave * PART + 5 * HP] = gb3;
    }
    __syncthreads();
    if (s_at >= 0) {
      float g = 0.f;
#pragma unroll 4
      for (int w = 0; w < nw; ++w) g += part[w * PART + tid];
      if (grad_out) {
        grad_out[base + s_at] = g;
      } else {
        adam(g, a1, a2, lr, s_th, s_m, s_v);
        small[tid] = s_th;
      }
    }
    __syncthreads();
  }
  if (!grad_out) {
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (w_at[u] >= 0) {
        params[base + w_at[u]] = w_th[u];
        mom[base + w_at[u]] = w_m[u];
        vel[base + w_at[u]] = w_v[u];
      }
    if (s_at >= 0) {
      params[base + s_at] = s_th;
      mom[base + s_at] = s_m;
      vel[base + s_at] = s_v;
    }
  }
  if (lane < 16 && active) part[pt] = loss;
  __syncthreads();
  if (tid == 0) {
    float l = 0.f;
    for (int i = 0; i < N; ++i) l += part[i];
    loss_out[member] = l * invN;
  }
}

// Forward and backward pass of (share of the points, member), CHUNK points at a
// time, and its part of the gradient and loss (MSE over all N points: the 2/N
// and 1/N factors are applied here; wts as above).
//
// Hidden units are padded to HT tiles of 16 with zero weights, points to CHUNK
// with zero residuals.  The three products of the hidden layer (forward, back
// to the first layer, gradient) are 16 x 16 x 4 matrix instructions from LDS,
// a 16 x 16 tile per wavefront and turn.
template <int HT>
__global__ __launch_bounds__(TRAIN_TPB) void k_ens_share(int N, int H, const float* __restrict__ Xs,
                                                         const float* __restrict__ ys,
                                                         const float* __restrict__ wts,
                                                         const float* __restrict__ params, float* __restrict__ gout,
                                                         float* __restrict__ lout) {
  constexpr int HP = 16 * HT, EP = HP + 4;  // row pitch: a matrix operand's 16 rows x 4 columns on different banks
  constexpr int WAVES = TRAIN_TPB / 64;
  constexpr int GT = (HT * HT + WAVES - 1) / WAVES;  // gradient tiles per wavefront
  __shared__ float W2[HP * EP], h1[CHUNK * EP], h2[CHUNK * EP], dz1[CHUNK * EP];
  __shared__ float W1[2 * HP], b1[HP], b2[HP], W3[HP], b3[1];
  __shared__ float x[2 * CHUNK], dout[CHUNK], loss[CHUNK];
  const int P = nparams(H);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr16 = lane & 15, lk = lane >> 4;
  const int member = blockIdx.y, share = blockIdx.x, nshare = gridDim.x;
  // units H .. HP - 1 are zeros
  const float* const th = params + size_t(member) * P;
#pragma unroll 4
  for (int e = tid; e < HP * HP; e += TRAIN_TPB) {
    const int o = e / HP, i = e % HP;
    W2[o * EP + i] = o < H && i < H ? th[3 * H + o * H + i] : 0.f;
  }
  if (tid < HP) {
    const bool on = tid < H;
    W1[2 * tid] = on ? th[2 * tid] : 0.f;
    W1[2 * tid + 1] = on ? th[2 * tid + 1] : 0.f;
    b1[tid] = on ? th[2 * H + tid] : 0.f;
    b2[tid] = on ? th[3 * H + H * H + tid] : 0.f;
    W3[tid] = on ? th[4 * H + H * H + tid] : 0.f;
    if (tid == 0) b3[0] = th[5 * H + H * H];
  }
  // tile of a product over K with operands A(row, k) = a[row * as + k * ak],
  // B(k, col) = b[k * bk + col * bs], added to acc (element u: row 4 lk + u,
  // column lr16)
  auto product = [&](const float* a, int as, int ak, const float* b, int bk, int bs, int K, f32x4 acc) {
    const float* ap = a + lr16 * as + lk * ak;
    const float* bp = b + lk * bk + lr16 * bs;
#pragma unroll
    for (int q = 0; q < K; q += 4)
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(ap[q * ak], bp[q * bk], acc, 0, 0, 0);
    return acc;
  };
  const float invN = 1.0f / float(N);
  f32x4 gw2[GT];
#pragma unroll
  for (int j = 0; j < GT; ++j) gw2[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  float gw3 = 0.f, gsmall = 0.f, gb3 = 0.f, lsum = 0.f;
  for (int c0 = share * CHUNK; c0 < N; c0 += nshare * CHUNK) {
    const int nc = min(CHUNK, N - c0);
    if (tid < 2 * CHUNK) x[tid] = tid < 2 * nc ? Xs[2 * c0 + tid] : 0.f;
    __syncthreads();
#pragma unroll
    for (int e = tid; e < CHUNK * HP; e += TRAIN_TPB) {
      const int s = e / HP, o = e % HP;
      h1[s * EP + o] = tanhf(W1[2 * o] * x[2 * s] + W1[2 * o + 1] * x[2 * s + 1] + b1[o]);
    }
    __syncthreads();
    for (int q = wave; q < (CHUNK / 16) * HT; q += WAVES) {
      const int tr = q / HT, tc = q % HT, o = 16 * tc + lr16;
      const float bo = b2[o];
      const f32x4 z = product(h1 + 16 * tr * EP, EP, 1, W2 + 16 * tc * EP, 1, EP, HP, f32x4{bo, bo, bo, bo});
#pragma unroll
      for (int u = 0; u < 4; ++u) h2[(16 * tr + 4 * lk + u) * EP + o] = tanhf(z[u]);
    }
    __syncthreads();
    {  // output layer: 16 lanes per point
      const int s = tid / 16, part = tid & 15;
      float a = 0.f;
#pragma unroll
      for (int o = part; o < HP; o += 16) a += W3[o] * h2[s * EP + o];
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) a += __shfl_xor(a, o);
      if (part == 0) {
        float l = 0.f, d = 0.f;
        if (s < nc) {
          // bootstrap: the point's count in this member's resample weights its
          // squared residual (the mean still over N)
          const float w = wts ? wts[size_t(member) * N + c0 + s] : 1.0f;
          const float r = a + b3[0] - ys[c0 + s];
          l = w * r * r;
          d = 2.0f * w * r * invN;
        }
        loss[s] = l;
        dout[s] = d;
      }
    }
    __syncthreads();
    // W3, b3 and the loss, before h2 becomes the second layer's residuals
    if (tid < HP) {
#pragma unroll 8
      for (int s = 0; s < CHUNK; ++s) gw3 += dout[s] * h2[s * EP + tid];
    } else if (wave == WAVES - 1 && lane < CHUNK) {
      gb3 += dout[lane];
      lsum += loss[lane];
    }
    __syncthreads();
#pragma unroll
    for (int e = tid; e < CHUNK * HP; e += TRAIN_TPB) {
      const int s = e / HP, o = e % HP;
      const float v = h2[s * EP + o];
      h2[s * EP + o] = dout[s] * W3[o] * (1.0f - v * v);
    }
    __syncthreads();
    const float* const dz2 = h2;
    for (int q = wave; q < (CHUNK / 16) * HT; q += WAVES) {
      const int tr = q / HT, tc = q % HT, i = 16 * tc + lr16;
      const f32x4 a = product(dz2 + 16 * tr * EP, EP, 1, W2 + 16 * tc, EP, 1, HP, f32x4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int s = 16 * tr + 4 * lk + u;
        const float v = h1[s * EP + i];
        dz1[s * EP + i] = a[u] * (1.0f - v * v);
      }
    }
#pragma unroll
    for (int j = 0; j < GT; ++j) {
      const int q = wave + j * WAVES;
      if (q < HT * HT)
        gw2[j] = product(dz2 + 16 * (q / HT), 1, EP, h1 + 16 * (q % HT), EP, 1, CHUNK, gw2[j]);
    }
    __syncthreads();
    // W1, b1 (from dz1) and b2 (from dz2): four sums per unit
    if (tid < 4 * HP) {
      const int o = tid >> 2, what = tid & 3;
#pragma unroll 8
      for (int s = 0; s < CHUNK; ++s) {
        const float f = what < 2 ? x[2 * s + what] : 1.0f;
        gsmall += (what < 3 ? dz1[s * EP + o] : dz2[s * EP + o]) * f;
      }
    }
    __syncthreads();  // the next points' x and activations
  }
  float* const go = gout + (size_t(member) * nshare + share) * P;
#pragma unroll
  for (int j = 0; j < GT; ++j) {
    const int q = wave + j * WAVES, i = 16 * (q % HT) + lr16;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int o = 16 * (q / HT) + 4 * lk + u;
      if (o < H && i < H) go[3 * H + o * H + i] = gw2[j][u];
    }
  }
  if (tid < H) go[4 * H + H * H + tid] = gw3;
  if (tid < 4 * H) {
    const int o = tid >> 2, what = tid & 3;
    go[what < 2 ? 2 * o + what : (what == 2 ? 2 * H + o : 3 * H + H * H + o)] = gsmall;
  }
  if (wave == WAVES - 1) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      gb3 += __shfl_xor(gb3, o);
      lsum += __shfl_xor(lsum, o);
    }
    if (lane == 0) {
      go[5 * H + H * H] = gb3;
      lout[size_t(member) * nshare + share] = lsum * invN;
    }
  }
}

// Per member: the gradient summed over shares and one Adam step.  Grid:
// (parameter blocks, members); the step number is *tbase + k + 1.  loss_out
// receives the loss at the parameters before the step.
__global__ __launch_bounds__(ENS_TPB) void k_ens_adam(int P, int nshare, const float* __restrict__ gpart,
                                                      const float* __restrict__ lpart, float* __restrict__ params,
                                                      float* __restrict__ mom, float* __restrict__ vel,
                                                      const int* __restrict__ tbase, int k, float lr,
                                                      float* __restrict__ loss_out, float* __restrict__ grad_out) {
  const int member = blockIdx.y, p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p < P) {
    const float* gm = gpart + size_t(member) * nshare * P + p;
    const size_t at = size_t(member) * P + p;
    float g = 0.f;
#pragma unroll 8
    for (int c = 0; c < nshare; ++c) g += gm[size_t(c) * P];
    if (grad_out) {
      grad_out[at] = g;
    } else {
      const int t = *tbase + k + 1;
      const float c1 = float(1.0 / (1.0 - pow(0.9, double(t)))), c2 = float(1.0 / (1.0 - pow(0.999, double(t))));
      adam(g, c1, c2, lr, params[at], mom[at], vel[at]);
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    float l = 0.f;
    for (int c = 0; c < nshare; ++c) l += lpart[size_t(member) * nshare + c];
    loss_out[member] = l;
  }
}

__global__ void k_ens_tick(int* tbase, int k) { *tbase += k; }

// Prediction, member by member: a wavefront keeps its member's hidden layer in
// registers as matrix operands (the first layer's weights in LDS, which leaves
// room for three wavefronts a SIMD) and takes 16 queries at a time.  A lane
// forms the first-layer activations it feeds to the 16 x 16 x 4 instructions
// (query lane % 16, units 16 t + 4 (lane / 16) + u) itself, and the output
// layer is a sum over 16 lanes.  What bounds it is the tanh of two layers (128
// per query and member, about 40 instructions each) and the matrix rate:
// 50,000 queries of 5 members of 64 units: a whole call took 277 us with W2 in
// LDS and a lane per unit and takes 55 us now; this kernel took 65 us with all
// weights in registers and two wavefronts a SIMD, 50 us now.
template <int HT>
__global__ __launch_bounds__(256, 3) void k_ens_member_out(int m, int H, const float* __restrict__ params,
                                                        const double* __restrict__ Xq, double mu0, double mu1,
                                                        double sd0, double sd1, float* __restrict__ yout) {
  const int k = blockIdx.y, lane = threadIdx.x & 63, lr16 = lane & 15, lk = lane >> 4;
  const int P = nparams(H);
  const float* W1 = params + size_t(k) * P;
  const float* b1 = W1 + 2 * H;
  const float* W2 = b1 + H;
  const float* b2 = W2 + H * H;
  const float* W3 = b2 + H;
  const float b3 = W3[H];
  constexpr int HP = 16 * HT;
  __shared__ float4 first[3][HP / 4];  // W1 (x, y), b1
  for (int i = threadIdx.x; i < HP; i += blockDim.x) {
    float* const l = reinterpret_cast<float*>(first);
    l[i] = i < H ? W1[2 * i] : 0.f;
    l[HP + i] = i < H ? W1[2 * i + 1] : 0.f;
    l[2 * HP + i] = i < H ? b1[i] : 0.f;
  }
  float w2[HT][4 * HT], c2[HT], w3[HT];
#pragma unroll
  for (int q = 0; q < 4 * HT; ++q) {
    const int i = 16 * (q / 4) + 4 * lk + q % 4;
#pragma unroll
    for (int t = 0; t < HT; ++t) {
      const int o = 16 * t + lr16;
      w2[t][q] = i < H && o < H ? W2[o * H + i] : 0.f;
    }
  }
#pragma unroll
  for (int t = 0; t < HT; ++t) {
    const int o = 16 * t + lr16;
    c2[t] = o < H ? b2[o] : 0.f;
    w3[t] = o < H ? W3[o] : 0.f;
  }
  __syncthreads();
  const int tiles = (m + 15) / 16, nw = gridDim.x * (blockDim.x / 64);
  for (int tile = blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6); tile < tiles; tile += nw) {
    asm volatile("" ::: "memory");  // the first layer stays in LDS (held in registers, it spills others)
    const int qq = min(16 * tile + lr16, m - 1);
    const float x0 = float((Xq[2 * qq] - mu0) / sd0), x1 = float((Xq[2 * qq + 1] - mu1) / sd1);
    f32x4 z[HT];
#pragma unroll
    for (int t = 0; t < HT; ++t) z[t] = f32x4{c2[t], c2[t], c2[t], c2[t]};
#pragma unroll
    for (int k = 0; k < HT; ++k) {
      const float4 wx = first[0][4 * k + lk], wy = first[1][4 * k + lk], c = first[2][4 * k + lk];
      const float a[4] = {wx.x * x0 + wy.x * x1 + c.x, wx.y * x0 + wy.y * x1 + c.y, wx.z * x0 + wy.z * x1 + c.z,
                          wx.w * x0 + wy.w * x1 + c.w};
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        // (a padded unit's zero weights would make a NaN of an infinite query)
        const float h = 16 * k + 4 * lk + u < H ? tanhf(a[u]) : 0.f;
#pragma unroll
        for (int t = 0; t < HT; ++t)
          z[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(h, w2[t][4 * k + u], z[t], 0, 0, 0);
      }
    }
    // element u: query 4 lk + u, units 16 t + lr16
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      float v = 0.f;
#pragma unroll
      for (int t = 0; t < HT; ++t) v += w3[t] * tanhf(z[t][u]);
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) v += __shfl_xor(v, o);
      const int q = 16 * tile + 4 * lk + u;
      if (lr16 == 0 && q < m) yout[size_t(k) * m + q] = b3 + v;
    }
  }
}

// Ensemble mean and sample standard deviation (M - 1) per query, FP64.
__global__ __launch_bounds__(128) void k_ens_reduce(int m, int members, const float* __restrict__ yout,
                                                    double s_q, double* __restrict__ mean_out,
                                                    double* __restrict__ std_out) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= m) return;
  double sum = 0.0, sum2 = 0.0;
  for (int k = 0; k < members; ++k) {
    const double yo = double(yout[size_t(k) * m + q]) * s_q;
    sum += yo;
    sum2 += yo * yo;
  }
  const double mean = sum / members;
  const double var = members > 1 ? (sum2 - members * mean * mean) / (members - 1) : 0.0;
  mean_out[q] = mean;
  std_out[q] = sqrt(var > 0.0 ? var : 0.0);
}

// Calls f with the smallest number of 16-unit tiles that holds H units, as a type.
template <class F>
void with_tiles(int H, F f) {
  if (H <= 16) f(std::integral_constant<int, 1>{});
  else if (H <= 32) f(std::integral_constant<int, 2>{});
  else if (H <= 48) f(std::integral_constant<int, 3>{});
  else f(std::integral_constant<int, 4>{});
}

// Queues the members' outputs at m queries: 16 queries per wavefront and turn.
// One turn each up to a workgroup per compute unit (5 members of 64 units, 200
// to 3,000 queries: 16 us, 20 with two turns), then two, up to 512 workgroups
// per member, which share the loads of the hidden layer (5,000 queries: 20 us,
// 23 with one).
void enqueue_members(const hmd_ens* e, int m, const double* dXq, float* yout, hipStream_t s) {
  constexpr int kUnits = 256;
  const int H = e->cfg.hidden, tiles = (m + 15) / 16, one = (tiles + 3) / 4;
  const int blocks = one * e->cfg.members <= kUnits ? one : std::min(512, (tiles + 7) / 8);
  const dim3 grid{unsigned(blocks), unsigned(e->cfg.members), 1};
  with_tiles(H, [&](auto tiles) {
    hipLaunchKernelGGL(k_ens_member_out<decltype(tiles)::value>, grid, dim3(256), 0, s, m, H, e->dparams, dXq, e->mu[0],
                       e->mu[1], e->sd[0], e->sd[1], yout);
  });
}

// Glorot-uniform start of one member: Philox4x32-10 keyed by the seed, word
// p mod 4 of counter (p div 4, member, 2, 0); biases zero.
void glorot(int H, int member, uint64_t seed, float* out) {
  const int P = nparams(H);
  const uint32_t key[2] = {uint32_t(seed & 0xffffffffu), uint32_t(seed >> 32)};
  std::vector<double> u(P);
  for (int j = 0; 4 * j < P; ++j) {
    const uint32_t ctr[4] = {uint32_t(j), uint32_t(member), 2u, 0u};
    uint32_t r[4];
    philox4x32_10(ctr, key, r);
    for (int w = 0; w < 4 && 4 * j + w < P; ++w) u[4 * j + w] = (double(r[w]) + 0.5) / 4294967296.0;
  }
  for (int p = 0; p < P; ++p) out[p] = 0.f;
  const double l1 = std::sqrt(6.0 / (2.0 + H)), l2 = std::sqrt(6.0 / (2.0 * H)), l3 = std::sqrt(6.0 / (H + 1.0));
  for (int p = 0; p < 2 * H; ++p) out[p] = float(l1 * (2.0 * u[p] - 1.0));
  for (int p = 3 * H; p < 3 * H + H * H; ++p) out[p] = float(l2 * (2.0 * u[p] - 1.0));
  for (int p = 4 * H + H * H; p < 5 * H + H * H; ++p) out[p] = float(l3 * (2.0 * u[p] - 1.0));
}

// Bootstrap resample of member `member` (counts per point): draw j takes
// point (r n) >> 32 for the Philox word r of counter (j div 4, member, 3, 0),
// word j mod 4, keyed by the seed.
void bootstrap_counts(int n, int member, uint64_t seed, float* out) {
  const uint32_t key[2] = {uint32_t(seed & 0xffffffffu), uint32_t(seed >> 32)};
  for (int i = 0; i < n; ++i) out[i] = 0.f;
  for (int j = 0; 4 * j < n; ++j) {
    const uint32_t ctr[4] = {uint32_t(j), uint32_t(member), 3u, 0u};
    uint32_t r[4];
    philox4x32_10(ctr, key, r);
    for (int w = 0; w < 4 && 4 * j + w < n; ++w) out[(uint64_t(r[w]) * uint64_t(n)) >> 32] += 1.f;
  }
}

int check_cfg(hmd_ctx* ctx, const hmd_ens_cfg& c, int n) {
  if (c.members < 1 || c.members > 64 || c.hidden < 1 || c.hidden > MAXH || c.iters < 0 || !(c.lr > 0.0) || n < 1 ||
      c.bootstrap < 0 || c.bootstrap > 1) {
    ctx->err = "ens: 1..64 members, 1..64 hidden units, iters >= 0, lr > 0, n >= 1, bootstrap 0 or 1";
    return HMD_EINVAL;
  }
  return HMD_OK;
}

// Standardise inputs and scale outputs (host, FP64), upload as FP32; with
// the bootstrap option also each member's counts (*dw, members x n).
int stage_data(hmd_ens* e, const double* X, const double* y, int n, float** dX, float** dy, float** dw) {
  hmd_ctx* ctx = e->ctx;
  for (int k = 0; k < 2; ++k) {
    double s = 0.0;
    for (int i = 0; i < n; ++i) s += X[2 * i + k];
    e->mu[k] = s / n;
    double v = 0.0;
    for (int i = 0; i < n; ++i) v += (X[2 * i + k] - e->mu[k]) * (X[2 * i + k] - e->mu[k]);
    e->sd[k] = std::sqrt(v / n);
    if (!(e->sd[k] > 0.0)) e->sd[k] = 1.0;
  }
  double s2 = 0.0;
  for (int i = 0; i < n; ++i) s2 += y[i] * y[i];
  e->s_q = std::sqrt(s2 / n);
  if (!(e->s_q > 0.0)) e->s_q = 1.0;
  std::vector<float> xs(2 * size_t(n)), ys(n);
  for (int i = 0; i < n; ++i) {
    for (int k = 0; k < 2; ++k) xs[2 * i + k] = float((X[2 * i + k] - e->mu[k]) / e->sd[k]);
    ys[i] = float(y[i] / e->s_q);
  }
  HMD_HIP(ctx, hipMalloc(dX, sizeof(float) * xs.size()));
  HMD_HIP(ctx, hipMalloc(dy, sizeof(float) * ys.size()));
  HMD_HIP(ctx, hipMemcpyAsync(*dX, xs.data(), sizeof(float) * xs.size(), hipMemcpyHostToDevice, ctx->stream));
  HMD_HIP(ctx, hipMemcpyAsync(*dy, ys.data(), sizeof(float) * ys.size(), hipMemcpyHostToDevice, ctx->stream));
  *dw = nullptr;
  if (e->cfg.bootstrap) {
    const int M = e->cfg.members;
    std::vector<float> w(size_t(M) * n);
    for (int k = 0; k < M; ++k) bootstrap_counts(n, k, e->cfg.seed, w.data() + size_t(k) * n);
    HMD_HIP(ctx, hipMalloc(dw, sizeof(float) * w.size()));
    HMD_HIP(ctx, hipMemcpy(*dw, w.data(), sizeof(float) * w.size(), hipMemcpyHostToDevice));
  }
  return HMD_OK;
}

int run_train(hmd_ens* e, int n, const float* dX, const float* dy, const float* dw, int mode, float* dgrad) {
  hmd_ctx* ctx = e->ctx;
  const hmd_ens_cfg& c = e->cfg;
  const int P = e->P, M = c.members;
  const int iters = mode == 1 ? 1 : c.iters;
  // one workgroup per member as far as its LDS holds the points: 20 us per
  // iteration at its largest (256 points, 64 units) against 27 and more for
  // work shared out over the chip, which gains only on sets beyond that
  const bool local = n <= LOCAL_N;
  const int nshare = local ? 0 : std::min((n + CHUNK - 1) / CHUNK, MAX_SHARES);
  // one allocation: moments, gradient and loss shares, losses, step counter
  const size_t mp = size_t(M) * P;
  float* mom = nullptr;
  hipError_t err = hipMalloc(&mom, sizeof(float) * (2 * mp + nshare * (mp + M) + M + 1));
  float* const vel = mom + mp;
  float* const gpart = vel + mp;
  float* const lpart = gpart + nshare * mp;
  float* const dloss = lpart + size_t(nshare) * M;
  int* const tstep = reinterpret_cast<int*>(dloss + M);
  hipStream_t s = ctx->stream;
  if (local) {
    with_tiles(c.hidden, [&](auto tiles) {
      constexpr int HT = decltype(tiles)::value, HP = 16 * HT, EP = HP + 4;
      const int nw = (n + 15) / 16, waves = std::max({nw, HT * HT, (5 * HP + 64) / 64});
      // activations and residuals; the sums of the small tensors take their place
      const size_t act = std::max(2 * size_t(16 * nw) * EP, size_t(nw) * (5 * HP + 4));
      const size_t lds = sizeof(float) * (HP * EP + 5 * HP + 4 + act);
      if (err == hipSuccess)
        err = hipFuncSetAttribute(reinterpret_cast<const void*>(k_ens_local<HT>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
      for (int t = 0; t < iters && err == hipSuccess; t += LOCAL_ITERS) {
        hipLaunchKernelGGL(k_ens_local<HT>, dim3(M), dim3(64 * waves), lds, s, n, c.hidden, dX, dy, dw, e->dparams, mom,
                           vel, t, std::min(LOCAL_ITERS, iters - t), float(c.lr), dloss, mode == 1 ? dgrad : nullptr);
        err = hipGetLastError();
      }
    });
  } else {
    if (err == hipSuccess) err = hipMemsetAsync(mom, 0, sizeof(float) * 2 * mp, s);
    if (err == hipSuccess) err = hipMemsetAsync(tstep, 0, sizeof(int), s);
    const dim3 agrid((P + ENS_TPB - 1) / ENS_TPB, M);
    auto iteration = [&](int k) {
      with_tiles(c.hidden, [&](auto tiles) {
        hipLaunchKernelGGL(k_ens_share<decltype(tiles)::value>, dim3(nshare, M), dim3(TRAIN_TPB), 0, s, n, c.hidden, dX,
                           dy, dw, e->dparams, gpart, lpart);
      });
      hipLaunchKernelGGL(k_ens_adam, agrid, dim3(ENS_TPB), 0, s, P, nshare, gpart, lpart, e->dparams, mom, vel, tstep,
                         k, float(c.lr), dloss, mode == 1 ? dgrad : nullptr);
    };
    // iterations in captured blocks of kBlock (a graph replay per block), the
    // remainder as direct launches; the step counter advances once per block
    constexpr int kBlock = 100;
    const int nblock = iters / kBlock;
    if (err == hipSuccess && nblock > 0) {
      hipGraph_t g = nullptr;
      hipGraphExec_t ge = nullptr;
      err = hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal);
      if (err == hipSuccess) {
        for (int k = 0; k < kBlock; ++k) iteration(k);
        hipLaunchKernelGGL(k_ens_tick, dim3(1), dim3(1), 0, s, tstep, kBlock);
        err = hipStreamEndCapture(s, &g);
      }
      if (err == hipSuccess) err = hipGraphInstantiate(&ge, g, nullptr, nullptr, 0);
      for (int r = 0; r < nblock && err == hipSuccess; ++r) err = hipGraphLaunch(ge, s);
      if (ge) (void)hipGraphExecDestroy(ge);
      if (g) (void)hipGraphDestroy(g);
    }
    for (int k = 0; k < iters - nblock * kBlock && err == hipSuccess; ++k) {
      iteration(k);
      err = hipGetLastError();
    }
  }
  std::vector<float> loss(M, 0.f);
  if (err == hipSuccess && iters > 0)
    err = hipMemcpyAsync(loss.data(), dloss, sizeof(float) * M, hipMemcpyDeviceToHost, s);
  if (err == hipSuccess) err = hipStreamSynchronize(s);
  if (mom) (void)hipFree(mom);
  if (err != hipSuccess) {
    ctx->err = std::string("ens training: ") + hipGetErrorString(err);
    return HMD_EDEVICE;
  }
  e->loss.assign(loss.begin(), loss.end());
  return HMD_OK;
}

int init_params(hmd_ens* e) {
  hmd_ctx* ctx = e->ctx;
  const hmd_ens_cfg& c = e->cfg;
  e->P = nparams(c.hidden);
  std::vector<float> h(size_t(c.members) * e->P);
  for (int k = 0; k < c.members; ++k) glorot(c.hidden, k, c.seed, h.data() + size_t(k) * e->P);
  HMD_HIP(ctx, hipMalloc(&e->dparams, sizeof(float) * h.size()));
  HMD_HIP(ctx, hipMemcpyAsync(e->dparams, h.data(), sizeof(float) * h.size(), hipMemcpyHostToDevice, ctx->stream));
  return HMD_OK;
}

}  // namespace
}  // namespace hmd

using namespace hmd;

extern "C" {

void hmd_ens_cfg_default(hmd_ens_cfg* c) {
  if (!c) return;
  c->members = 5;
  c->hidden = 64;
  c->iters = 5000;
  c->lr = 1e-3;
  c->seed = 0;
  c->bootstrap = 0;
}

int ens_fit(hmd_ctx* ctx, const double* X, const double* y, int n, const hmd_ens_cfg* cfg, hmd_ens** out) {
  if (!ctx || !X || !y || !out) return HMD_EINVAL;
  hmd_ens_cfg c;
  if (cfg) c = *cfg;
  else hmd_ens_cfg_default(&c);
  int rc = check_cfg(ctx, c, n);
  if (rc != HMD_OK) return rc;
  HMD_HIP(ctx, hipSetDevice(ctx->device));
  auto* e = new hmd_ens();
  e->ctx = ctx;
  e->cfg = c;
  e->X.assign(X, X + 2 * size_t(n));
  e->y.assign(y, y + n);
  rc = ens_refit(e);
  if (rc != HMD_OK) {
    ens_free(e);
    return rc;
  }
  *out = e;
  return HMD_OK;
}

int ens_append(hmd_ens* e, const double* x, double y) {
  if (!e || !x) return HMD_EINVAL;
  e->X.push_back(x[0]);
  e->X.push_back(x[1]);
  e->y.push_back(y);
  return HMD_OK;
}

int ens_refit(hmd_ens* e) {
  if (!e) return HMD_EINVAL;
  hmd_ctx* ctx = e->ctx;
  const int n = int(e->y.size());
  int rc = check_cfg(ctx, e->cfg, n);
  if (rc != HMD_OK) return rc;
  HMD_HIP(ctx, hipSetDevice(ctx->device));
  if (e->dparams) {
    (void)hipFree(e->dparams);
    e->dparams = nullptr;
  }
  float *dX = nullptr, *dy = nullptr, *dw = nullptr;
  if ((rc = init_params(e)) == HMD_OK && (rc = stage_data(e, e->X.data(), e->y.data(), n, &dX, &dy, &dw)) == HMD_OK)
    rc = run_train(e, n, dX, dy, dw, 0, nullptr);
  for (void* p : {(void*)dX, (void*)dy, (void*)dw})
    if (p) (void)hipFree(p);
  return rc;
}

int ens_size(const hmd_ens* e) { return e ? int(e->y.size()) : 0; }

int ens_predict(hmd_ens* e, const double* Xs, int m, double* mean, double* std) {
  if (!e || m < 0 || (m > 0 && (!Xs || !mean || !std))) return HMD_EINVAL;
  if (m == 0) return HMD_OK;
  hmd_ctx* ctx = e->ctx;
  HMD_HIP(ctx, hipSetDevice(ctx->device));
  if (m > e->qcap) {
    if (e->dq) (void)hipFree(e->dq);
    if (e->dy) (void)hipFree(e->dy);
    if (e->dout) (void)hipFree(e->dout);
    e->dq = nullptr; e->dy = nullptr; e->dout = nullptr; e->qcap = 0;
    const int cap = std::max(m, 256);
    HMD_HIP(ctx, hipMalloc(&e->dq, sizeof(double) * 2 * cap));
    HMD_HIP(ctx, hipMalloc(&e->dy, sizeof(float) * size_t(e->cfg.members) * cap));
    HMD_HIP(ctx, hipMalloc(&e->dout, sizeof(double) * 2 * cap));
    e->qcap = cap;
  }
  std::vector<double> res(2 * size_t(m));  // means, then standard deviations
  HMD_HIP(ctx, hipMemcpyAsync(e->dq, Xs, sizeof(double) * 2 * m, hipMemcpyHostToDevice, ctx->stream));
  enqueue_members(e, m, e->dq, e->dy, ctx->stream);
  HMD_HIP(ctx, hipGetLastError());
  hipLaunchKernelGGL(k_ens_reduce, dim3((m + 127) / 128), dim3(128), 0, ctx->stream, m, e->cfg.members, e->dy,
                     e->s_q, e->dout, e->dout + m);
  HMD_HIP(ctx, hipGetLastError());
  HMD_HIP(ctx, hipMemcpyAsync(res.data(), e->dout, sizeof(double) * res.size(), hipMemcpyDeviceToHost,
                              ctx->stream));
  HMD_HIP(ctx, hipStreamSynchronize(ctx->stream));
  for (int q = 0; q < m; ++q) {
    mean[q] = res[q];
    std[q] = res[size_t(m) + q];
  }
  return HMD_OK;
}

int ens_predict_dev(hmd_ens* e, const double* dXs, int m, double* dmean, double* dstd, void* stream) {
  if (!e || m < 0 || (m > 0 && (!dXs || !dmean || !dstd))) return HMD_EINVAL;
  if (m == 0) return HMD_OK;
  hmd_ctx* ctx = e->ctx;
  HMD_HIP(ctx, hipSetDevice(ctx->device));
  hipStream_t s = stream ? static_cast<hipStream_t>(stream) : ctx->stream;
  if (m > e->qcap) {
    HMD_HIP(ctx, hipStreamSynchronize(s));  // the old scratch may still be read
    if (e->dq) (void)hipFree(e->dq);
    if (e->dy) (void)hipFree(e->dy);
    if (e->dout) (void)hipFree(e->dout);
    e->dq = nullptr; e->dy = nullptr; e->dout = nullptr; e->qcap = 0;
    const int cap = std::max(m, 256);
    HMD_HIP(ctx, hipMalloc(&e->dq, sizeof(double) * 2 * cap));
    HMD_HIP(ctx, hipMalloc(&e->dy, sizeof(float) * size_t(e->cfg.members) * cap));
    HMD_HIP(ctx, hipMalloc(&e->dout, sizeof(double) * 2 * cap));
    e->qcap = cap;
  }
  enqueue_members(e, m, dXs, e->dy, s);
  HMD_HIP(ctx, hipGetLastError());
  hipLaunchKernelGGL(k_ens_reduce, dim3((m + 127) / 128), dim3(128), 0, s, m, e->cfg.members, e->dy, e->s_q,
                     dmean, dstd);
  HMD_HIP(ctx, hipGetLastError());
  return HMD_OK;
}

int ens_loss(const hmd_ens* e, double* loss) {
  if (!e || !loss) return HMD_EINVAL;
  for (size_t k = 0; k < e->loss.size(); ++k) loss[k] = e->loss[k];
  return HMD_OK;
}

int ens_grad_init(hmd_ctx* ctx, const double* X, const double* y, int n, const hmd_ens_cfg* cfg, int member,
                  double* params, double* grad, int* n_params) {
  if (!ctx || !X || !y) return HMD_EINVAL;
  hmd_ens_cfg c;
  if (cfg) c = *cfg;
  else hmd_ens_cfg_default(&c);
  int rc = check_cfg(ctx, c, n);
  if (rc != HMD_OK) return rc;
  if (member < 0 || member >= c.members) return HMD_EINVAL;
  HMD_HIP(ctx, hipSetDevice(ctx->device));
  hmd_ens e;
  e.ctx = ctx;
  e.cfg = c;
  float *dX = nullptr, *dy = nullptr, *dg = nullptr, *dw = nullptr;
  if ((rc = init_params(&e)) == HMD_OK && (rc = stage_data(&e, X, y, n, &dX, &dy, &dw)) == HMD_OK) {
    if (hipMalloc(&dg, sizeof(float) * size_t(c.members) * e.P) != hipSuccess) rc = HMD_ENOMEM;
    else rc = run_train(&e, n, dX, dy, dw, 1, dg);
  }
  if (rc == HMD_OK) {
    std::vector<float> hp(e.P), hg(e.P);
    if (hipMemcpy(hp.data(), e.dparams + size_t(member) * e.P, sizeof(float) * e.P, hipMemcpyDeviceToHost) !=
            hipSuccess ||
        hipMemcpy(hg.data(), dg + size_t(member) * e.P, sizeof(float) * e.P, hipMemcpyDeviceToHost) != hipSuccess)
      rc = HMD_EDEVICE;
    for (int p = 0; p < e.P; ++p) {
      if (params) params[p] = hp[p];
      if (grad) grad[p] = hg[p];
    }
    if (n_params) *n_params = e.P;
  }
  for (void* p : {(void*)dX, (void*)dy, (void*)dg, (void*)dw, (void*)e.dparams})
    if (p) (void)hipFree(p);
  return rc;
}

int ens_members(const hmd_ens* e) { return e ? e->cfg.members : 0; }

void ens_free(hmd_ens* e) {
  if (!e) return;
  if (e->dparams) (void)hipFree(e->dparams);
  if (e->dq) (void)hipFree(e->dq);
  if (e->dy) (void)hipFree(e->dy);
  if (e->dout) (void)hipFree(e->dout);
  delete e;
}

}  // extern "C"

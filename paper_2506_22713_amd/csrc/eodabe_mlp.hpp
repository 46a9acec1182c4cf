// Learned rank predictor that warm-starts the basis size of Alg. 1: a GELU
// MLP 67 -> 256 -> 256 -> 256 -> 2 in FP32, trained and run by the kernels
// below.  Inputs: the first 64 values d_c = |T(c,c)| of the stopping test
// (the diagonal of the R factor of A Omega[:, :64], normalised by d_0 on a
// clamped log10 scale), log2 m, log2 n and log10(eps / d_0), the stopping
// threshold eps = tol ||A||_F on the scale of those values.  Head 0 regresses
// log(1 + rank); head 1 is the 0.9-quantile of the same quantity (pinball
// loss) and sizes the warm start.
#pragma once
#include "eodabe_kernels.hpp"

namespace eodabe {

constexpr int MLP_IN = 67, MLP_H = 256, MLP_OUT = 2;
constexpr double MLP_TAU = 0.9;
// flat parameter layout: W1 (H x IN, row-major), b1, W2 (H x H), b2, W3, b3, W4 (OUT x H), b4
constexpr int64_t MLP_W1 = 0, MLP_B1 = MLP_W1 + (int64_t)MLP_H * MLP_IN, MLP_W2 = MLP_B1 + MLP_H,
                  MLP_B2 = MLP_W2 + (int64_t)MLP_H * MLP_H, MLP_W3 = MLP_B2 + MLP_H,
                  MLP_B3 = MLP_W3 + (int64_t)MLP_H * MLP_H, MLP_W4 = MLP_B3 + MLP_H,
                  MLP_B4 = MLP_W4 + (int64_t)MLP_OUT * MLP_H, MLP_NPARAM = MLP_B4 + MLP_OUT;

// Input c of the network from the stopping-test values (c < 64), the
// geometry (c = 64, 65) or the threshold eps = tol ||A||_F of the test on
// the same scale as the d_c (c = 66).  Shared by the host (training sets)
// and the inference kernel.
__host__ __device__ inline float mlp_feature(const double* d, int c, int64_t m, int64_t n, double eps) {
  if (c < 64) {
    if (!(d[0] > 0.0) || !(d[c] > 0.0)) return -1.0f;
    const double l = log10(d[c] / d[0]);
    return (float)((l < -16.0 ? -16.0 : l) / 16.0);
  }
  if (c == 64) return (float)(log2((double)m) / 16.0);
  if (c == 65) return (float)(log2((double)n) / 16.0);
  if (!(d[0] > 0.0) || !(eps > 0.0)) return -1.0f;
  double l = log10(eps / d[0]);
  l = l < -16.0 ? -16.0 : (l > 16.0 ? 16.0 : l);
  return (float)(l / 16.0);
}

// Warm-start width from the quantile head: d0 = b ceil((rhat (1 + margin) + 1) / b),
// rhat = exp(y1) - 1, at least one block.
__host__ __device__ inline int64_t mlp_width(double y1, int b, double margin) {
  double rhat = exp(y1) - 1.0;
  if (!(rhat > 0.0)) rhat = 0.0;
  if (rhat > 1e9) rhat = 1e9;
  const double q = ceil((rhat * (1.0 + margin) + 1.0) / b);
  return (int64_t)b * (int64_t)(q < 1.0 ? 1.0 : q);
}

__device__ __forceinline__ float gelu_f(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_grad_f(float z) {
  const float cdf = 0.5f * (1.0f + erff(z * 0.70710678118654752f));
  const float pdf = 0.39894228040143268f * expf(-0.5f * z * z);
  return cdf + z * pdf;
}

constexpr int MLP_ROWS = 16;          // samples of one workgroup
constexpr int MLP_LDH = MLP_H + 4;    // row stride of a layer in LDS

// acc += (LDS rows of `h`) W^T for the 16 columns of this wave: W row-major
// (nout x MLP_H), lane (li, g) takes row li of the tile and four K at a time.
__device__ __forceinline__ f32x4 mlp_fwd_tile(const float (*h)[MLP_LDH], const float* __restrict__ Wr, int li, int g,
                                              bool vec) {
  typedef Mfma<float> MF;
  f32x4 a0 = MF::zero(), a1 = MF::zero();
#pragma unroll 8
  for (int t = 0; t < MLP_H / 16; ++t) {
    const f32x4 x = *reinterpret_cast<const f32x4*>(&h[li][16 * t + 4 * g]);
    f32x4 w;
    if (vec) {
      w = *reinterpret_cast<const f32x4*>(Wr + 16 * t + 4 * g);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = Wr[16 * t + 4 * g + e];
    }
    a0 = MF::op(x[0], w[0], a0);
    a1 = MF::op(x[1], w[1], a1);
    a0 = MF::op(x[2], w[2], a0);
    a1 = MF::op(x[3], w[3], a1);
  }
  return a0 + a1;
}
// acc += (LDS rows of `d`) W for the 16 columns of this wave (Wc = W + column).
__device__ __forceinline__ f32x4 mlp_bwd_tile(const float (*d)[MLP_LDH], const float* __restrict__ Wc, int li, int g) {
  typedef Mfma<float> MF;
  f32x4 a0 = MF::zero(), a1 = MF::zero();
#pragma unroll 8
  for (int t = 0; t < MLP_H / 16; ++t) {
    const f32x4 x = *reinterpret_cast<const f32x4*>(&d[li][16 * t + 4 * g]);
    float w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = Wc[(int64_t)(16 * t + 4 * g + e) * MLP_H];
    a0 = MF::op(x[0], w[0], a0);
    a1 = MF::op(x[1], w[1], a1);
    a0 = MF::op(x[2], w[2], a0);
    a1 = MF::op(x[3], w[3], a1);
  }
  return a0 + a1;
}

// What the weight gradients need of a batch, in the workspace (row-major):
// inputs h[l] of layers 2..4 and the gradients g[l] at the sums of layers
// 1..3 (B x H each), dy (B x 2) at the heads, and each sample's loss.
struct MlpTape {
  float *h[3], *g[3], *dy;
  double* loss_row;
};

// The whole network on 16 samples per workgroup, and with GRAD its backward
// pass down to the sums of layer 1.  The layers are too small to be worth a
// launch each (256 samples: eleven GEMM launches of 25-35 us on 4 to 16
// workgroups, and as many elementwise ones): here the activations of a strip
// stay in LDS, a wave owns 16 of the 256 columns of every layer, and the sums z
// stay in its registers until GELU'(z) needs them, since the forward and the
// backward tile of a column have the same lane layout.  What is left is the
// weights' way from L2 (256 KB a layer and workgroup) and 64 MFMAs in a row.
// A training step of 256 samples (both kernels, Adam, the loss on the host):
// 568 -> 77 us.
template <bool GRAD>
__global__ __launch_bounds__(64 * MLP_H / 16) void k_mlp_net(const float* __restrict__ P,
                                                             const float* __restrict__ X,
                                                             const float* __restrict__ T, int B,
                                                             float* __restrict__ Y, MlpTape tape, int vec) {
  typedef Mfma<float> MF;
  __shared__ float h[MLP_ROWS][MLP_LDH], x[MLP_ROWS][84], sdy[MLP_ROWS][2];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, li = lane & 15, g = lane >> 4;
  const int64_t b0 = blockIdx.x * (int64_t)MLP_ROWS;
  const int col = 16 * wv + li;
  for (int i = tid; i < MLP_ROWS * 80; i += 64 * MLP_H / 16) {
    const int r = i / 80, c = i % 80;
    x[r][c] = (c < MLP_IN && b0 + r < B) ? X[(b0 + r) * MLP_IN + c] : 0.f;
  }
  f32x4 z[3];
  {
    float w[20];
#pragma unroll
    for (int s = 0; s < 20; ++s) w[s] = 4 * s + g < MLP_IN ? P[MLP_W1 + (int64_t)col * MLP_IN + 4 * s + g] : 0.f;
    __syncthreads();
    f32x4 acc = MF::zero();
#pragma unroll
    for (int s = 0; s < 20; ++s) acc = MF::op(x[li][4 * s + g], w[s], acc);
    z[0] = acc + P[MLP_B1 + col];
  }
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    if (l) {
      const int64_t W = l == 1 ? MLP_W2 : MLP_W3, b = l == 1 ? MLP_B2 : MLP_B3;
      z[l] = mlp_fwd_tile(h, P + W + (int64_t)col * MLP_H, li, g, vec) + P[b + col];
    }
    __syncthreads();                                   // every wave has read the layer below
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = MF::row(g, e);
      const float a = gelu_f(z[l][e]);
      h[r][col] = a;
      if (GRAD && b0 + r < B) tape.h[l][(b0 + r) * MLP_H + col] = a;
    }
    __syncthreads();
  }
  // heads: wave r takes sample r
  {
    float y0 = 0.f, y1 = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float a = h[wv][64 * e + lane];
      y0 = fmaf(a, P[MLP_W4 + 64 * e + lane], y0);
      y1 = fmaf(a, P[MLP_W4 + MLP_H + 64 * e + lane], y1);
    }
    for (int o = 1; o < 64; o <<= 1) {
      y0 += __shfl_xor(y0, o);
      y1 += __shfl_xor(y1, o);
    }
    y0 += P[MLP_B4];
    y1 += P[MLP_B4 + 1];
    const int64_t b = b0 + wv;
    if (!GRAD) {
      if (lane == 0 && b < B) {
        Y[2 * b] = y0;
        Y[2 * b + 1] = y1;
      }
      return;
    }
    if (lane == 0) {
      float d0 = 0.f, d1 = 0.f;
      if (b < B) {
        const double invB = 1.0 / B, t = T[b], u = t - (double)y1, v = (double)y0 - t;
        tape.loss_row[b] = v * v + (u > 0 ? MLP_TAU * u : (MLP_TAU - 1.0) * u);
        d0 = (float)(2.0 * v * invB);
        d1 = (float)((u > 0 ? -MLP_TAU : 1.0 - MLP_TAU) * invB);
        tape.dy[2 * b] = d0;
        tape.dy[2 * b + 1] = d1;
      }
      sdy[wv][0] = d0;
      sdy[wv][1] = d1;
    }
  }
  __syncthreads();
#pragma unroll
  for (int l = 2; l >= 0; --l) {
    f32x4 d;
    if (l == 2) {
      const float w0 = P[MLP_W4 + col], w1 = P[MLP_W4 + MLP_H + col];
#pragma unroll
      for (int e = 0; e < 4; ++e) d[e] = fmaf(sdy[MF::row(g, e)][0], w0, sdy[MF::row(g, e)][1] * w1);
    } else {
      d = mlp_bwd_tile(h, P + (l == 1 ? MLP_W3 : MLP_W2) + col, li, g);
      __syncthreads();                                 // every wave has read the layer above
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = MF::row(g, e);
      const float v = d[e] * gelu_grad_f(z[l][e]);
      if (l) h[r][col] = v;
      if (b0 + r < B) tape.g[l][(b0 + r) * MLP_H + col] = v;
    }
    if (l) __syncthreads();
  }
}

// All weight and bias gradients in one launch: dW = g^T h and db = column
// sums of g, a 16 x 16 tile of one layer per workgroup, the batch split over
// its four waves and summed in wave order.  The last workgroup sums the loss
// (FP64, fixed order).  At 256 samples that is 608 workgroups of 16 MFMAs a
// wave; with a launch per product the chip was at most a quarter full.
constexpr int MLP_HT = MLP_H / 16, MLP_IT = (MLP_IN + 15) / 16;
constexpr int MLP_WG_TILES = 2 * MLP_HT * MLP_HT + MLP_HT * MLP_IT + MLP_HT;
__global__ __launch_bounds__(256) void k_mlp_wgrad(const float* __restrict__ X, MlpTape tape, int B,
                                                   float* __restrict__ G, double* __restrict__ loss) {
  typedef Mfma<float> MF;
  __shared__ f32x4 part[4][64];
  __shared__ float bpart[4][64];
  __shared__ double red[256];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, li = lane & 15, g = lane >> 4;
  int t = blockIdx.x;
  if (t == MLP_WG_TILES) {
    double s = 0.0;
    for (int b = tid; b < B; b += 256) s += tape.loss_row[b];
    red[tid] = s;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
      if (tid < off) red[tid] += red[tid + off];
      __syncthreads();
    }
    if (tid == 0) *loss = red[0] * (1.0 / B);
    return;
  }
  const float *a, *h;              // gradient (B x na) and layer input (B x nh)
  int na = MLP_H, nh = MLP_H, it, jt;
  int64_t ow, ob;
  if (t < 2 * MLP_HT * MLP_HT) {
    const int l = t / (MLP_HT * MLP_HT);
    t %= MLP_HT * MLP_HT;
    it = t / MLP_HT;
    jt = t % MLP_HT;
    a = l ? tape.g[2] : tape.g[1];
    h = l ? tape.h[1] : tape.h[0];
    ow = l ? MLP_W3 : MLP_W2;
    ob = l ? MLP_B3 : MLP_B2;
  } else if (t < 2 * MLP_HT * MLP_HT + MLP_HT * MLP_IT) {
    t -= 2 * MLP_HT * MLP_HT;
    it = t / MLP_IT;
    jt = t % MLP_IT;
    a = tape.g[0];
    h = X;
    nh = MLP_IN;
    ow = MLP_W1;
    ob = MLP_B1;
  } else {
    it = 0;
    jt = t - 2 * MLP_HT * MLP_HT - MLP_HT * MLP_IT;
    a = tape.dy;
    h = tape.h[2];
    na = MLP_OUT;
    ow = MLP_W4;
    ob = MLP_B4;
  }
  const int i = 16 * it + li, j = 16 * jt + li;
  const bool iok = i < na, jok = j < nh;
  const int kper = ((B + 3) / 4 + 3) / 4 * 4;          // samples of a wave, a multiple of 4
  const int k0 = wv * kper, k1 = k0 + kper < B ? k0 + kper : B;
  f32x4 acc = MF::zero();
  float bs = 0.f;
#pragma unroll 8
  for (int k = k0; k < k1; k += 4) {
    const bool ok = k + g < k1;
    const int64_t b = ok ? k + g : k;
    const float av = iok && ok ? a[b * na + i] : 0.f;
    const float hv = jok && ok ? h[b * nh + j] : 0.f;
    acc = MF::op(av, hv, acc);
    bs += av;
  }
  part[wv][lane] = acc;
  bpart[wv][lane] = bs;
  __syncthreads();
  if (wv) return;
  acc = part[0][lane] + part[1][lane] + part[2][lane] + part[3][lane];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int r = 16 * it + MF::row(g, e);
    if (r < na && jok) G[ow + (int64_t)r * nh + j] = acc[e];
  }
  if (jt == 0 && g == 0 && iok) {
    float s = 0.f;
    for (int w = 0; w < 4; ++w)
      for (int q = 0; q < 4; ++q) s += bpart[w][16 * q + li];
    G[ob + i] = s;
  }
}

// One Adam step with bias-corrected moments.  The coefficients come from
// the host, formed in FP64 and rounded once: beta, 1 - beta and the bias
// corrections c = 1 - beta^step.
struct AdamCoef {
  float lr, b1, omb1, b2, omb2, c1, c2, eps;
};
__global__ void k_adam(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, int64_t n, AdamCoef a) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const float gi = g[i];
    const float mi = a.b1 * m[i] + a.omb1 * gi;
    const float vi = a.b2 * v[i] + a.omb2 * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= a.lr * (mi / a.c1) / (sqrtf(vi / a.c2) + a.eps);
  }
}

// Result of one warm-start inference (device).
struct MlpPred {
  int64_t d0;       // warm-start width
  double y0, y1;    // both heads (log(1 + rank))
};

// Single-sample inference on one workgroup, straight from the stopping-test
// values on the device: features, three GELU layers (thread j computes
// unit j), the two heads, and the warm-start width.
__global__ __launch_bounds__(256) void k_mlp_infer1(const float* __restrict__ P, const double* __restrict__ diag,
                                                    int64_t m, int64_t n, const State* __restrict__ st, int b,
                                                    double margin, MlpPred* __restrict__ out) {
  __shared__ float x[MLP_IN], h[2][MLP_H];
  const int j = threadIdx.x;
  if (j < MLP_IN) x[j] = mlp_feature(diag, j, m, n, st->eps);
  __syncthreads();
  float z = P[MLP_B1 + j];
  for (int k = 0; k < MLP_IN; ++k) z += P[MLP_W1 + (int64_t)j * MLP_IN + k] * x[k];
  h[0][j] = gelu_f(z);
  __syncthreads();
  z = P[MLP_B2 + j];
  for (int k = 0; k < MLP_H; ++k) z += P[MLP_W2 + (int64_t)j * MLP_H + k] * h[0][k];
  h[1][j] = gelu_f(z);
  __syncthreads();
  z = P[MLP_B3 + j];
  for (int k = 0; k < MLP_H; ++k) z += P[MLP_W3 + (int64_t)j * MLP_H + k] * h[1][k];
  __syncthreads();
  h[0][j] = gelu_f(z);
  __syncthreads();
  if (j < MLP_OUT) {
    float y = P[MLP_B4 + j];
    for (int k = 0; k < MLP_H; ++k) y += P[MLP_W4 + (int64_t)j * MLP_H + k] * h[0][k];
    x[j] = y;
  }
  __syncthreads();
  if (j == 0) {
    MlpPred o;
    o.y0 = x[0];
    o.y1 = x[1];
    o.d0 = mlp_width(x[1], b, margin);
    *out = o;
  }
}

}  // namespace eodabe

// Device kernels of the two applications the paper evaluates EOD-ABE on:
//   * colour-image compression (introduction and section 4.1): each channel
//     is factored, reconstructed as U_hat D_hat V_hat^T, and the quality
//     criteria PSNR, global SSIM and RelErr are reduced in FP64 in a fixed
//     order, fused into the reconstruction pass;
//   * hyperspectral dimensionality reduction (section 4.2): pixel features
//     U_hat D_hat and KNN classification of every pixel by the pixels of the
//     other cross-validation folds.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "eodabe_kernels.hpp"

namespace eodabe {

constexpr int IMG_MAX_CH = 4;

// Per-channel factor locations of one image (passed by value).
struct ImgJob {
  const float* Ut[IMG_MAX_CH];   // r_cap x h row-major: row a is column a of U_hat
  const float* core[IMG_MAX_CH]; // r_cap x r_cap row-major: D_hat
  const float* Vt[IMG_MAX_CH];   // r_cap x w row-major: V_hat^T
  float* B[IMG_MAX_CH];          // scratch r x w: D_hat V_hat^T
  int r[IMG_MAX_CH];             // rank of the channel
  int rc;                        // r_cap of every channel
};

// B = D_hat V_hat^T for each channel (grid: w / 256 x r_max x channels);
// D_hat upper triangular, so B(a, j) = sum_{b >= a} D(a, b) Vt(b, j).
__global__ __launch_bounds__(256) void k_img_dvt(ImgJob job, int64_t w) {
  const int c = blockIdx.z, a = blockIdx.y;
  const int64_t j = blockIdx.x * (int64_t)256 + threadIdx.x;
  const int r = job.r[c];
  if (a >= r || j >= w) return;
  const float* D = job.core[c] + (int64_t)a * job.rc;
  const float* V = job.Vt[c];
  float acc = 0.f;
  for (int b = a; b < r; ++b) acc = fmaf(D[b], V[(int64_t)b * w + j], acc);
  job.B[c][(int64_t)a * w + j] = acc;
}

// Sums of one image pass: x = reconstruction, y = original.
struct ImgSums {
  double sx, sy, sxx, syy, sxy, sdd;
};

// A_hat = U_hat B for every channel (64 x 64 output tile per workgroup,
// 16 rows per wave on v_mfma_f32_16x16x4f32, the K loop over the rank),
// written to recon; the same pass accumulates the six FP64 sums of the
// criteria against the original image and writes one partial per
// workgroup (fixed tile order, so the fold is deterministic).
__global__ __launch_bounds__(256) void k_img_recon(ImgJob job, const float* __restrict__ img, int64_t h,
                                                   int64_t w, float* __restrict__ recon,
                                                   ImgSums* __restrict__ parts) {
  typedef Mfma<float> MF;
  __shared__ double red[6][4];
  const int c = blockIdx.z;
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63, lr = lane & 15, g = lane >> 4;
  const int64_t i0 = blockIdx.y * (int64_t)64 + 16 * wv, j0 = blockIdx.x * (int64_t)64;
  const int r = job.r[c];
  const float* U = job.Ut[c];
  const float* B = job.B[c];
  MF::acc_t acc[4] = {MF::zero(), MF::zero(), MF::zero(), MF::zero()};
  const int64_t ia = i0 + lr;
  for (int a0 = 0; a0 < r; a0 += 4) {
    const int a = a0 + g;
    const bool ka = a < r;
    const float av = (ka && ia < h) ? U[(int64_t)a * h + ia] : 0.f;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int64_t jb = j0 + 16 * t + lr;
      const float bv = (ka && jb < w) ? B[(int64_t)a * w + jb] : 0.f;
      acc[t] = MF::op(av, bv, acc[t]);
    }
  }
  const float* Y = img + (int64_t)c * h * w;
  float* X = recon + (int64_t)c * h * w;
  double s[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int64_t jj = j0 + 16 * t + lr;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int64_t ii = i0 + MF::row(g, e);
      if (ii < h && jj < w) {
        const float xv = acc[t][e];
        const double x = xv, y = Y[ii * w + jj], d = x - y;
        X[ii * w + jj] = xv;
        s[0] += x; s[1] += y; s[2] += x * x; s[3] += y * y; s[4] += x * y; s[5] += d * d;
      }
    }
  }
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    double v = s[q];
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if (lane == 0) red[q][wv] = v;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const int64_t pid = ((int64_t)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
    double* o = &parts[pid].sx;
#pragma unroll
    for (int q = 0; q < 6; ++q) o[q] = ((red[q][0] + red[q][1]) + red[q][2]) + red[q][3];
  }
}

// Criteria of section 4.1 over the whole image.
struct ImgMetrics {
  double relerr, psnr, ssim, sdd, syy, n;
};

// One workgroup: fold the partials in a fixed order, then the criteria:
// PSNR = 10 log10(255^2 N / sdd), SSIM of the vectorised images with
// c1 = (0.01 255)^2, c2 = (0.03 255)^2 and 1/(N-1) (co)variances,
// RelErr = sqrt(sdd / syy).
__global__ __launch_bounds__(256) void k_img_metrics(const ImgSums* __restrict__ parts, int64_t nparts,
                                                     double N, ImgMetrics* __restrict__ out) {
  __shared__ double red[6][256];
  double s[6] = {0, 0, 0, 0, 0, 0};
  for (int64_t p = threadIdx.x; p < nparts; p += 256) {
    const double* q = &parts[p].sx;
#pragma unroll
    for (int k = 0; k < 6; ++k) s[k] += q[k];
  }
#pragma unroll
  for (int k = 0; k < 6; ++k) red[k][threadIdx.x] = s[k];
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off)
#pragma unroll
      for (int k = 0; k < 6; ++k) red[k][threadIdx.x] += red[k][threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double sx = red[0][0], sy = red[1][0], sxx = red[2][0], syy = red[3][0], sxy = red[4][0],
                 sdd = red[5][0];
    const double mx = sx / N, my = sy / N;
    const double vx = (sxx - sx * mx) / (N - 1.0), vy = (syy - sy * my) / (N - 1.0);
    const double cxy = (sxy - sx * my) / (N - 1.0);
    const double c1 = (0.01 * 255.0) * (0.01 * 255.0), c2 = (0.03 * 255.0) * (0.03 * 255.0);
    ImgMetrics m;
    m.sdd = sdd;
    m.syy = syy;
    m.n = N;
    m.relerr = syy > 0.0 ? sqrt(sdd / syy) : 0.0;
    m.psnr = sdd > 0.0 ? 10.0 * log10(255.0 * 255.0 * N / sdd) : INFINITY;
    m.ssim = (2.0 * mx * my + c1) * (2.0 * cxy + c2) / ((mx * mx + my * my + c1) * (vx + vy + c2));
    *out = m;
  }
}

// Pixel features F = U_hat D_hat (m x r, row-major, ldf): F(i, a) =
// sum_{b <= a} U(i, b) D(b, a), b ascending, with D upper triangular.  A
// workgroup takes PX pixels and FEAT_W features at a time, a thread one pixel
// and PX / 16 of them; U's columns come UB chunks of FEAT_W at a time, a step
// ahead of their products, D's tiles with them through LDS, and the results
// leave through LDS as whole rows.  With many pixels it is bound by reading U
// and writing F, with few by the chain of steps of the last features: the rule
// of the launch (feat_split).  Grid: pixels / PX x features' chunks (blockIdx.y
// takes every gridDim.y-th, the longest first).
constexpr int FEAT_W = 16;
template <int PX, int UB>
__global__ __launch_bounds__(256) void k_features(const float* __restrict__ Ut, const float* __restrict__ core,
                                                  int64_t m, int r, int64_t rc, float* __restrict__ F,
                                                  int64_t ldf) {
  static_assert(FEAT_W * FEAT_W == 256, "one entry of a tile of D per thread");
  static_assert(PX % 64 == 0 && 256 % PX == 0, "whole waves per group of features");
  constexpr int G = 256 / PX, FW = FEAT_W / G;      // groups of features, features of a thread
  __shared__ float buf[PX][FEAT_W + 1];
  __shared__ __align__(16) float ds[UB][FEAT_W * FEAT_W];
  const int tid = threadIdx.x, dk = tid % FEAT_W, dq = tid / FEAT_W;
  const int px = tid % PX, k0 = G == 1 ? 0 : tid / PX * FW;
  const int64_t i0 = blockIdx.x * (int64_t)PX;
  const int rows = (int)(m - i0 < PX ? m - i0 : PX), pl = min(px, rows - 1);
  for (int c = (r - 1) / FEAT_W - (int)blockIdx.y; c >= 0; c -= gridDim.y) {
    const int a0 = FEAT_W * c;
    float acc[FW], u[UB][FEAT_W], un[UB][FEAT_W], d[UB], dn[UB];
    auto load = [&](float(&v)[UB][FEAT_W], float(&e)[UB], int b0) {   // entries past r are read at r - 1 and not used
#pragma unroll
      for (int s = 0; s < UB; ++s)
        if (b0 + FEAT_W * s <= a0) {
#pragma unroll
          for (int q = 0; q < FEAT_W; ++q) v[s][q] = (Ut + (int64_t)min(b0 + FEAT_W * s + q, r - 1) * m + i0)[pl];
          e[s] = core[(int64_t)min(b0 + FEAT_W * s + dq, r - 1) * rc + min(a0 + dk, r - 1)];
        }
    };
#pragma unroll
    for (int k = 0; k < FW; ++k) acc[k] = 0.f;
    load(u, d, 0);
    for (int b0 = 0; b0 <= a0; b0 += UB * FEAT_W) {
      load(un, dn, b0 + UB * FEAT_W);
      __syncthreads();
#pragma unroll
      for (int s = 0; s < UB; ++s) ds[s][tid] = d[s];
      __syncthreads();
#pragma unroll
      for (int s = 0; s < UB; ++s) {
        if (b0 + FEAT_W * s < a0) {
#pragma unroll
          for (int q = 0; q < FEAT_W; ++q)
#pragma unroll
            for (int k = 0; k < FW; ++k) acc[k] = fmaf(u[s][q], ds[s][q * FEAT_W + k0 + k], acc[k]);
        } else if (b0 + FEAT_W * s == a0) {          // D is upper triangular
#pragma unroll
          for (int q = 0; q < FEAT_W; ++q)
#pragma unroll
            for (int k = 0; k < FW; ++k) {
              const float v = fmaf(u[s][q], ds[s][q * FEAT_W + k0 + k], acc[k]);
              acc[k] = q <= k0 + k ? v : acc[k];
            }
        }
      }
#pragma unroll
      for (int s = 0; s < UB; ++s) {
#pragma unroll
        for (int q = 0; q < FEAT_W; ++q) u[s][q] = un[s][q];
        d[s] = dn[s];
      }
    }
#pragma unroll
    for (int k = 0; k < FW; ++k) buf[px][k0 + k] = acc[k];
    __syncthreads();
    if (a0 + dk < r)
      for (int row = dq; row < rows; row += 256 / FEAT_W) F[(i0 + row) * ldf + a0 + dk] = buf[row][dk];
  }
}
// Pixels of a workgroup, and workgroups that share the features of a strip.
// With fewer than FEAT_WG workgroups of 64 pixels and one chunk of features
// each, every chunk is a workgroup of 64 pixels; else a workgroup has 256
// pixels and the chunks are spread only until there are FEAT_WG (beyond,
// re-reading U from farther away costs more than the shorter chain gains).
// 4096 x 200: 13.7 us, all chunks of 256 pixels on one workgroup 180, a
// thread per pixel and feature 31; 1024 x 500: 28, 1028 and 50; 262144 x 15:
// 9, 9 and 38 (64 pixels 16); 262144 x 100: 133, 149 and 991.
constexpr int FEAT_WG = 1024;
struct FeatSplit {
  int px, parts;
};
inline FeatSplit feat_split(int64_t m, int64_t r) {
  const int64_t chunks = (r + FEAT_W - 1) / FEAT_W;
  const int px = (m + 63) / 64 * chunks < FEAT_WG ? 64 : 256;
  const int64_t strips = (m + px - 1) / px, parts = (FEAT_WG + strips - 1) / strips;
  return FeatSplit{px, (int)(parts < chunks ? parts : chunks)};
}

constexpr int KNN_KMAX = 16;
constexpr int KNN_DMAX = 32;
constexpr int KNN_CMAX = 64;

// KNN classification of every point by the points of the other folds
// (ten-fold cross-validation in one launch).  The answer is defined in FP64:
// squared distances summed feature by feature from the FP32 features with
// separate multiply and add (no contraction), the k nearest the smallest
// (distance, index) pairs, the vote to the most frequent label, ties to the
// smaller one.  pred[i] receives the class and conf[pred * nclass + label]
// counts it.
//
// Those FP64 sums for all m^2 pairs bound the direct form (one query per
// thread: 20.5 ms at m = 21025, d = 15, on 83 workgroups).  Here FP32 MFMA
// products find the few pairs that can matter, and only they are summed in
// FP64: 0.61 ms there, of which the products of the two passes are 0.23 ms at
// the FP32 MFMA rate.  A workgroup owns 32 queries; its waves stream 16-candidate tiles.
//   pass 1: |y|^2 - 2 x.y per pair as 4 S-deep MFMA products plus one for
//     |y|^2 (each lane's own partial norm against ones: no cross-lane sum),
//     padded upwards by the rounding bound, its minimum over each of 128
//     interleaved candidate classes kept per query.  The k-th smallest of
//     those minima bounds the k-th nearest distance from above (k <= 16
//     distinct candidates lie within it).
//   pass 2: the same products padded downwards; pairs below the bound go to
//     a per-wave queue and are summed in FP64 64 at a time, then kept in a
//     list per query, from which the k smallest pairs are taken.  The lists'
//     order varies between runs, the selection does not.
// A query whose list overflows (more than KNN_CAP pairs within the bound:
// duplicated or quantised points) is left to k_knn_rest.
//
// Rounding bound: with x', y' the features less a common centre, each off by
// a relative 2^-24, and K = 4 S + 4 products accumulated in FP32, the value
// differs from the FP64 distance by less than 8 (d + 8) 2^-24 (|x'|^2 +
// |y'|^2) (the pieces add to about half of that), plus 1e-36 for results
// below the normal range.  Norms past 1e37, where a product may overflow to
// either side, make the pair pass: a candidate's becomes -infinity, and a
// query's bound a NaN, which no comparison drops a pair against.
constexpr int KNN_WV = 8;       // waves of a workgroup
constexpr int KNN_QT = 2;       // 16-query tiles of a workgroup
constexpr int KNN_NQ = 16 * KNN_QT;
constexpr int KNN_CAP = 96;     // pairs kept per query
constexpr int32_t KNN_REST = -1;   // in pred between the two launches: not answered yet

__device__ __forceinline__ double knn_dist(const float* __restrict__ F, int64_t ldf, int d, int64_t i, int64_t j) {
  const float* x = F + i * ldf;
  const float* y = F + j * ldf;
  double dd = 0.0;
  {
#pragma clang fp contract(off)
    for (int a = 0; a < d; ++a) {
      const double u = (double)y[a] - (double)x[a];
      dd = dd + u * u;
    }
  }
  return dd;
}

// Class of query i from its nearest points (0x7fffffff: none), counted.
__device__ __forceinline__ void knn_vote(const int* sel, int k, const int32_t* __restrict__ label, int nclass, int64_t i,
                                         int32_t* __restrict__ pred, unsigned long long* __restrict__ conf) {
  int bl[KNN_KMAX];
#pragma unroll
  for (int s = 0; s < KNN_KMAX; ++s) bl[s] = (s < k && sel[s] != 0x7fffffff) ? label[sel[s]] : -1;
  int best = KNN_CMAX, bestc = -1;
#pragma unroll
  for (int s = 0; s < KNN_KMAX; ++s) {
    if (s >= k || bl[s] < 0) continue;
    int n = 0;
#pragma unroll
    for (int t = 0; t < KNN_KMAX; ++t) n += (t < k && bl[t] == bl[s]) ? 1 : 0;
    if (n > bestc || (n == bestc && bl[s] < best)) {
      bestc = n;
      best = bl[s];
    }
  }
  if (bestc < 0) best = 0;   // no candidate in other folds
  pred[i] = best;
  atomicAdd(&conf[(int64_t)best * nclass + label[i]], 1ull);
}

template <int S>
__global__ __launch_bounds__(64 * KNN_WV) void k_knn_cv(const float* __restrict__ F, int64_t m, int d, int64_t ldf,
                                                        const int32_t* __restrict__ label,
                                                        const int32_t* __restrict__ fold, int k, int nclass,
                                                        int32_t* __restrict__ pred,
                                                        unsigned long long* __restrict__ conf) {
  typedef Mfma<float> MF;
  constexpr int NB = KNN_WV * 16;                     // candidate classes of pass 1
  __shared__ union {
    float bmin[NB][KNN_NQ + 1];
    struct {
      double dd[KNN_NQ][KNN_CAP];
      int jj[KNN_NQ][KNN_CAP];
    } list;
  } sh;
  __shared__ int quej[KNN_WV][128];
  __shared__ unsigned char queq[KNN_WV][128];
  __shared__ float thr[KNN_NQ];
  __shared__ int cnt[KNN_NQ], sel[KNN_NQ][KNN_KMAX];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, li = lane & 15, g = lane >> 4;
  const int64_t q0 = blockIdx.x * (int64_t)KNN_NQ;
  const int64_t ntile = (m + 15) / 16;
  const float pad = 8.f * (float)(d + 8) * 5.9604645e-8f;

  // this lane's features are g S .. g S + S - 1 (zero past d), less the mean
  // of 16 rows spread over the points
  int off[S];
  bool in[S];
#pragma unroll
  for (int s = 0; s < S; ++s) {
    in[s] = s < S - 3 || g * S + s < d;
    off[s] = in[s] ? g * S + s : d - 1;
  }
  float c[S];
  {
    const float* p = F + (m * li / 16) * ldf;
#pragma unroll
    for (int s = 0; s < S; ++s) c[s] = p[off[s]];
#pragma unroll
    for (int s = 0; s < S; ++s) {
      for (int o = 1; o < 16; o <<= 1) c[s] += __shfl_xor(c[s], o);
      c[s] = fabsf(c[s]) < 1e18f ? c[s] * 0.0625f : 0.f;
    }
  }
  // query operands -2 x', norms and folds
  float b[KNN_QT][S], nx[KNN_QT];
  int qf[KNN_QT];
#pragma unroll
  for (int t = 0; t < KNN_QT; ++t) {
    const int64_t i = q0 + 16 * t + li < m ? q0 + 16 * t + li : m - 1;
    float n2 = 0.f;
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const float x = in[s] ? F[i * ldf + off[s]] - c[s] : 0.f;
      n2 = fmaf(x, x, n2);
      b[t][s] = -2.f * x;
    }
    n2 += __shfl_xor(n2, 16);
    n2 += __shfl_xor(n2, 32);
    nx[t] = n2;
    qf[t] = fold[i];
  }
  if (tid < KNN_NQ) cnt[tid] = 0;

  auto fetch = [&](int64_t tile, float(&x)[S]) {
    const int64_t j = tile * 16 + li < m ? tile * 16 + li : m - 1;
#pragma unroll
    for (int s = 0; s < S; ++s) x[s] = F[j * ldf + off[s]];
  };
  // centred candidate operand in place; its padded partial norm.  A norm out
  // of range becomes `big`; a row past m counts as infinitely far
  auto centre = [&](int64_t tile, float(&x)[S], float scale, float big) {
    float p = 0.f;
#pragma unroll
    for (int s = 0; s < S; ++s) {
      x[s] = in[s] ? x[s] - c[s] : 0.f;
      p = fmaf(x[s], x[s], p);
    }
    p = p > 1e37f ? big : p * scale;
    return tile * 16 + li < m ? p : INFINITY;
  };
  auto product = [&](const float(&x)[S], float p, int t) {
    typename MF::acc_t acc = MF::zero();
#pragma unroll
    for (int s = 0; s < S; ++s) acc = MF::op(x[s], b[t][s], acc);
    return MF::op(p, 1.f, acc);
  };

  // ---- pass 1
  {
    float mn[KNN_QT][4];
#pragma unroll
    for (int t = 0; t < KNN_QT; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) mn[t][e] = INFINITY;
    float x[S], xn[S];
    if (wv < ntile) fetch(wv, x);
    for (int64_t tile = wv; tile < ntile; tile += KNN_WV) {
      fetch(tile + KNN_WV < ntile ? tile + KNN_WV : tile, xn);
      int cf[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int64_t j = tile * 16 + MF::row(g, e);
        cf[e] = fold[j < m ? j : m - 1];
      }
      const float p = centre(tile, x, 1.f + pad, INFINITY);
#pragma unroll
      for (int t = 0; t < KNN_QT; ++t) {
        const typename MF::acc_t v = product(x, p, t);
#pragma unroll
        for (int e = 0; e < 4; ++e) mn[t][e] = (v[e] < mn[t][e] && cf[e] != qf[t]) ? v[e] : mn[t][e];
      }
#pragma unroll
      for (int s = 0; s < S; ++s) x[s] = xn[s];
    }
#pragma unroll
    for (int t = 0; t < KNN_QT; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) sh.bmin[wv * 16 + g * 4 + e][16 * t + li] = mn[t][e] + nx[t] * (1.f + pad);
  }
  __syncthreads();
  // the k-th smallest class minimum of each query (16 threads a query)
  {
    const int q = tid >> 4, sub = tid & 15;
    float v[NB / 16];
#pragma unroll
    for (int e = 0; e < NB / 16; ++e) v[e] = sh.bmin[sub * (NB / 16) + e][q];
    float last = INFINITY;
    for (int s = 0; s < k; ++s) {
      float best = v[0];
      int at = 0;
#pragma unroll
      for (int e = 1; e < NB / 16; ++e)
        if (v[e] < best) {
          best = v[e];
          at = e;
        }
      float gb = best;
      int who = sub;
      for (int o = 1; o < 16; o <<= 1) {
        const float ob = __shfl_xor(gb, o);
        const int ow = __shfl_xor(who, o);
        if (ob < gb || (ob == gb && ow < who)) {
          gb = ob;
          who = ow;
        }
      }
      last = gb;
#pragma unroll
      for (int e = 0; e < NB / 16; ++e)
        if (who == sub && e == at) v[e] = INFINITY;
    }
    if (sub == 0) thr[q] = last;
  }
  __syncthreads();

  // ---- pass 2
  {
    float tq[KNN_QT];
#pragma unroll
    for (int t = 0; t < KNN_QT; ++t) {
      tq[t] = thr[16 * t + li] - nx[t] * (1.f - pad) + 1e-36f;
      if (!(nx[t] < 1e37f)) tq[t] = __builtin_nanf("");
      if (q0 + 16 * t + li >= m) tq[t] = -INFINITY;
    }
    int qn = 0;                                       // queued pairs of this wave
    auto flush = [&](int n) {
      if (lane < n) {
        const int j = quej[wv][lane], q = queq[wv][lane];
        const double dd = knn_dist(F, ldf, d, q0 + q, j);
        if (dd < INFINITY) {
          const int at = atomicAdd(&cnt[q], 1);
          if (at < KNN_CAP) {
            sh.list.dd[q][at] = dd;
            sh.list.jj[q][at] = j;
          }
        }
      }
      const int left = qn - n;
      int j = 0, q = 0;
      if (lane < left) {
        j = quej[wv][n + lane];
        q = queq[wv][n + lane];
      }
      __builtin_amdgcn_wave_barrier();
      if (lane < left) {
        quej[wv][lane] = j;
        queq[wv][lane] = (unsigned char)q;
      }
      __builtin_amdgcn_wave_barrier();
      qn = left;
    };
    float x[S], xn[S];
    if (wv < ntile) fetch(wv, x);
    for (int64_t tile = wv; tile < ntile; tile += KNN_WV) {
      fetch(tile + KNN_WV < ntile ? tile + KNN_WV : tile, xn);
      const float p = centre(tile, x, 1.f - pad, -INFINITY);
      typename MF::acc_t v[KNN_QT];
      bool any = false;
#pragma unroll
      for (int t = 0; t < KNN_QT; ++t) {
        v[t] = product(x, p, t);
#pragma unroll
        for (int e = 0; e < 4; ++e) any |= !(v[t][e] >= tq[t]);
      }
      if (__any(any)) {
#pragma unroll
        for (int t = 0; t < KNN_QT; ++t)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            bool h = !(v[t][e] >= tq[t]);
            if (!__any(h)) continue;
            const int64_t j = tile * 16 + MF::row(g, e);
            h = h && j < m && q0 + 16 * t + li < m;
            h = h && fold[j] != qf[t] && cnt[16 * t + li] <= KNN_CAP;   // past that, k_knn_rest answers it
            const unsigned long long mk = __ballot(h);
            if (h) {
              const int at = qn + __popcll(mk & ((1ull << lane) - 1));
              quej[wv][at] = (int)j;
              queq[wv][at] = (unsigned char)(16 * t + li);
            }
            __builtin_amdgcn_wave_barrier();
            qn += __popcll(mk);
            if (qn >= 64) flush(64);
          }
      }
#pragma unroll
      for (int s = 0; s < S; ++s) x[s] = xn[s];
    }
    flush(qn);
  }
  __syncthreads();

  // ---- the k smallest (distance, index) pairs of each query's list
  {
    const int q = tid >> 4, sub = tid & 15;
    const int n = cnt[q] < KNN_CAP ? cnt[q] : KNN_CAP;
    double dv[KNN_CAP / 16];
    int jv[KNN_CAP / 16];
#pragma unroll
    for (int e = 0; e < KNN_CAP / 16; ++e) {
      const bool ok = sub + 16 * e < n;
      dv[e] = ok ? sh.list.dd[q][sub + 16 * e] : INFINITY;
      jv[e] = ok ? sh.list.jj[q][sub + 16 * e] : 0x7fffffff;
    }
    for (int s = 0; s < k; ++s) {
      double bd = dv[0];
      int bj = jv[0];
#pragma unroll
      for (int e = 1; e < KNN_CAP / 16; ++e)
        if (dv[e] < bd || (dv[e] == bd && jv[e] < bj)) {
          bd = dv[e];
          bj = jv[e];
        }
      for (int o = 1; o < 16; o <<= 1) {
        const double od = __shfl_xor(bd, o);
        const int oj = __shfl_xor(bj, o);
        if (od < bd || (od == bd && oj < bj)) {
          bd = od;
          bj = oj;
        }
      }
      if (sub == 0) sel[q][s] = bj;
#pragma unroll
      for (int e = 0; e < KNN_CAP / 16; ++e)
        if (jv[e] == bj) {
          dv[e] = INFINITY;
          jv[e] = 0x7fffffff;
        }
    }
  }
  __syncthreads();
  if (tid >= KNN_NQ || q0 + tid >= m) return;
  if (cnt[tid] > KNN_CAP) pred[q0 + tid] = KNN_REST;
  else knn_vote(sel[tid], k, label, nclass, q0 + tid, pred, conf);
}

// The queries that k_knn_cv left (pred = KNN_REST), by the definition: the
// FP64 distances to all points, which go through LDS KNN_RT rows at a time for
// all queries of the workgroup (the same 32 as there), 16 threads a query, or
// 64 where at most 8 are left; a thread keeps the k nearest of its points in
// registers, and the heads of the threads' lists are merged k times.  Bound by
// the FP64 sums.  21025 x 15 points of which half are the same take 2.6 / 2.7 /
// 2.9 ms at k = 1 / 5 / 16, all the same 2.7 / 2.8 / 2.9.  One query of the
// workgroup after the other, all points scanned k times with rows read from
// memory in lane-strided pieces, took 9.4 / 34 / 99 and 22 / 70 / 192, and one
// query per thread over all pairs 20.
constexpr int KNN_RT = 256;
template <int S>
__global__ __launch_bounds__(64 * KNN_WV) void k_knn_rest(const float* __restrict__ F, int64_t m, int d, int64_t ldf,
                                                          const int32_t* __restrict__ label,
                                                          const int32_t* __restrict__ fold, int k, int nclass,
                                                          int32_t* __restrict__ pred,
                                                          unsigned long long* __restrict__ conf) {
  constexpr int NF = 4 * S, P = NF + 1;               // features of a row in LDS (zeros past d), then its fold
  __shared__ float row[KNN_RT * P];
  __shared__ int left[KNN_NQ], sel[KNN_NQ][KNN_KMAX];
  const int tid = threadIdx.x, lane = tid & 63;
  const int64_t q0 = blockIdx.x * (int64_t)KNN_NQ;
  const int64_t ql = q0 + (lane & (KNN_NQ - 1));
  const unsigned mask = (unsigned)__ballot(lane < KNN_NQ && ql < m && pred[ql < m ? ql : m - 1] == KNN_REST);
  if (mask == 0u) return;                             // the same in every wave
  if (tid < KNN_NQ && ((mask >> tid) & 1u)) left[__popc(mask & ((1u << tid) - 1u))] = tid;
  __syncthreads();
  const int n = __popc(mask), tpq = n <= KNN_WV ? 64 : 16;
  const int slot = tid / tpq, sub = tid % tpq;
  const bool mine = slot < n;
  const int64_t i = q0 + left[mine ? slot : 0];
  const int fi = fold[i];
  double x[NF], bd[KNN_KMAX], worst = INFINITY;
  int bj[KNN_KMAX];
#pragma unroll
  for (int a = 0; a < NF; ++a) x[a] = a < d ? (double)F[i * ldf + (a < d ? a : 0)] : 0.0;
#pragma unroll
  for (int s = 0; s < KNN_KMAX; ++s) {
    bd[s] = INFINITY;
    bj[s] = 0x7fffffff;
  }
  for (int64_t j0 = 0; j0 < m; j0 += KNN_RT) {
    const int nr = (int)(m - j0 < KNN_RT ? m - j0 : KNN_RT);
    __syncthreads();
    for (int e = tid; e < nr * NF; e += 64 * KNN_WV) {
      const int t = e / NF, a = e % NF;
      row[t * P + a] = a < d ? F[(j0 + t) * ldf + a] : 0.f;
    }
    for (int t = tid; t < nr; t += 64 * KNN_WV) row[t * P + NF] = __int_as_float(fold[j0 + t]);
    __syncthreads();
    if (!mine) continue;
    for (int t = sub; t < nr; t += tpq) {             // ascending: an equal distance later is no nearer
      const float* y = row + t * P;
      double dd = 0.0;
      {
#pragma clang fp contract(off)
#pragma unroll
        for (int a = 0; a < NF; ++a) {
          const double u = (double)y[a] - x[a];
          dd = dd + u * u;
        }
      }
      if (__float_as_int(y[NF]) == fi || !(dd < worst)) continue;
      double v = dd;
      int vj = (int)j0 + t;
      bool in = false;
#pragma unroll
      for (int s = 0; s < KNN_KMAX; ++s) {            // in front of the first that is farther, the others one back
        in = in || v < bd[s];
        const double ov = bd[s];
        const int oj = bj[s];
        bd[s] = in ? v : ov;
        bj[s] = in ? vj : oj;
        v = in ? ov : v;
        vj = in ? oj : vj;
        if (s == k - 1) worst = bd[s];
      }
    }
  }
  for (int s = 0; s < k; ++s) {
    double hd = bd[0];
    int hj = bj[0];
    for (int o = 1; o < tpq; o <<= 1) {
      const double od = __shfl_xor(hd, o);
      const int oj = __shfl_xor(hj, o);
      if (od < hd || (od == hd && oj < hj)) {
        hd = od;
        hj = oj;
      }
    }
    if (mine && sub == 0) sel[slot][s] = hj;
    const bool take = bj[0] == hj;
#pragma unroll
    for (int e = 0; e < KNN_KMAX; ++e) {
      bd[e] = take ? (e + 1 < KNN_KMAX ? bd[e + 1 < KNN_KMAX ? e + 1 : e] : INFINITY) : bd[e];
      bj[e] = take ? (e + 1 < KNN_KMAX ? bj[e + 1 < KNN_KMAX ? e + 1 : e] : 0x7fffffff) : bj[e];
    }
  }
  if (mine && sub == 0) knn_vote(sel[slot], k, label, nclass, i, pred, conf);
}

}  // namespace eodabe

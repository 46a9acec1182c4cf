// Batched EOD-ABE for many small matrices (tiles): one workgroup factors a
// whole tile (Alg. 1 + Alg. 2, q = 0) with the same arithmetic as the
// single-matrix path (FP32 data, FP64 Grams, Cholesky with inverse), taking
// tiles from a device work queue until it is empty.  Tiles up to
// TILE_MAX x TILE_MAX; ranks up to TILE_RMAX are finished in the kernel
// (a tile whose rank goes above reports status TS_RANK and is left to the
// caller).  Ranks up to 64 close on LDS-resident FP64 matrices; wider ranks
// use the 2 x 2-blocked Cholesky with inverse on L2-resident ones.
#pragma once
#include "eodabe_kernels.hpp"

namespace eodabe {

constexpr int TILE_MAX = 1024;                 // largest tile side
constexpr int TILE_RMAX = 128;                 // rank finished inside the kernel
constexpr int TILE_BMAX = 64;                  // largest block width
constexpr int TILE_QW = TILE_RMAX + TILE_BMAX; // basis columns held (rank + one block)

// LDS operands of the routines kept out of line: a plain pointer would make
// every access a flat one.
typedef __attribute__((address_space(3))) double* lds_ptr;
typedef __attribute__((address_space(3))) const double* lds_cptr;

enum TileStatus : int32_t { TS_OK = 0, TS_RANK = 1, TS_NONFINITE = 2, TS_CAPACITY = 3 };

struct TileDesc {
  const float* A;        // row-major h x w, leading dimension lda
  int64_t h, w, lda;
  int64_t out_off;       // element offset of this tile's outputs in the pool
  int64_t r_cap;         // output capacity: Ut r_cap x h, core r_cap x r_cap, Vt r_cap x w
  int32_t b;             // block width (<= TILE_BMAX)
  int32_t index;         // position in the caller's arrays
};

struct TileResult {
  int64_t rank;
  int32_t blocks;
  int32_t status;
  double norm;
};

// Scratch of one workgroup (floats unless marked).
struct TileSlot {
  static constexpr int64_t LD = TILE_MAX;                // leading dimension of tall buffers
  static constexpr int64_t Y = 0;                        // block, LD x TILE_BMAX
  static constexpr int64_t Q = Y + LD * TILE_BMAX;       // basis, LD x TILE_QW
  static constexpr int64_t CT = Q + LD * TILE_QW;        // C^T, LD x TILE_RMAX
  static constexpr int64_t VP = CT + LD * TILE_RMAX;     // V' of a wide tile, LD x TILE_RMAX
  static constexpr int64_t FLOATS = VP + LD * TILE_RMAX;
  // FP64 matrices after the floats: ranks <= 64 (64 x 64, column-major)
  static constexpr int64_t SM = 64 * 64;
  static constexpr int64_t R1 = 0, R2 = SM, QH = 2 * SM, DH = 3 * SM, QH2 = 4 * SM, DH2 = 5 * SM;
  // ranks 65..128 (128 x 128, row-major, leading dimension LB)
  static constexpr int LB = 128;
  static constexpr int64_t B2 = (int64_t)LB * LB;
  static constexpr int64_t BIG = 6 * SM;                 // 16 buffers of B2
  static constexpr int64_t DOUBLES = BIG + 16 * B2;
  static constexpr int64_t BYTES = FLOATS * 4 + DOUBLES * 8;
};

// LDS arena (doubles): the closing QR's 4 small matrices, its work area and
// diagonal, then 72 scalars that live across phases (||A||^2, R1 diagonal).
constexpr int TILE_SQR = 4 * SmallCfg<64>::SIZE + 24 * 64 + 64;
constexpr int TILE_LDS = TILE_SQR + 72;
// basis-phase carve: Gram/R, R^{-1}, Cholesky work, diagonal; W = Q^T Y
// (TILE_QW x TILE_BMAX) from 0; the reductions' fold buffer after both.
constexpr int TL_GS = 0, TL_RI = SmallCfg<64>::SIZE, TL_WORK = 2 * SmallCfg<64>::SIZE,
              TL_DGS = TL_WORK + 24 * 64, TL_W = 0, TL_FOLD = TILE_QW * TILE_BMAX, TL_FOLD_N = 16 * 256;
static_assert(TL_DGS + 64 <= TL_FOLD, "Cholesky carve below the fold buffer");
static_assert(CHOL128_LDS <= TILE_SQR && 128 * 129 <= TILE_SQR, "wide-rank closing inside the arena");
static_assert(TL_FOLD + TL_FOLD_N <= TILE_SQR, "basis carve inside the arena");

// ---------------------------------------------------------------------------
// First launch of a batch: Omega^T (row c, TILE_MAX entries, is column c of
// the test matrix: a pure function of seed, row and column, so the tiles of a
// batch share it), and the reset of the work queue.  A block of a tile starts
// at a column <= TILE_RMAX and has at most TILE_BMAX columns: TILE_QW columns
// reach every one.  Made by each tile for itself it took 42 of a tile's 730 us
// (the Box-Muller pairs are evaluated in FP64).  Grid: TILE_QW x 256 threads.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_tile_begin(float* __restrict__ omt, uint32_t* __restrict__ queue,
                                                    uint32_t k0, uint32_t k1) {
  static_assert(TILE_MAX == 4 * 256, "one quad per thread");
  const int c = blockIdx.x, q = threadIdx.x;
  if (c == 0 && q < 64) queue[q] = 0u;
  V4<float> o;
  omega4(k0, k1, q, c, o.v);
  st4(omt + (int64_t)c * TILE_MAX + 4 * q, o);
}

// ---------------------------------------------------------------------------
// Y (m x nb, column-major ldy) = A B^T: A m x n row-major (lda), B given by
// its rows (row c at B + c*ldb, n entries, 16-byte aligned; rows >= nb read
// as zero), nb <= 64.  Wave w takes 64-row panels w, w+4, ...; each element
// of A is read once.  AL: rows of A 16-byte aligned (vector loads), else
// scalar loads.  ss (LDS, may be null): sum of squares of A.
// ---------------------------------------------------------------------------
template <bool AL>
__device__ __forceinline__ V4<float> tile_lda4(const float* p) {
  if constexpr (AL) {
    return ld4(p);
  } else {
    V4<float> v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v.v[e] = p[e];
    return v;
  }
}
// CTR = ceil(nb / 16) column tiles.  The loads of a full 16-column step are
// unconditional (rows of B past nb are read at row nb - 1 and zeroed by a
// select), and the steady state of the PF-deep ring has no branches, so
// each step waits only for its own loads.  Kept out of line, like the X^T Y
// routine below: the tile kernel is validated with these two as calls (an
// inlined build failed the batched parity test with an illegal address).
template <bool AL, int CTR>
__device__ __noinline__ void tile_rowprod_t(const float* A, int64_t lda, int64_t m, int64_t n, const float* B,
                                            int64_t ldb, int nb, float* Yb, int64_t ldy, double* ss,
                                            double* red) {
  typedef Mfma<float> MF;
  constexpr int RT = 4, PF = 4;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, r = lane & 15, g = lane >> 4;
  const int64_t nfull = n / 16;
  double sq = 0.0;
  const float* bp[CTR];
  bool bval[CTR];
#pragma unroll
  for (int u = 0; u < CTR; ++u) {
    const int bc = 16 * u + r;
    bval[u] = bc < nb;
    bp[u] = B + (int64_t)(bval[u] ? bc : (nb > 0 ? nb - 1 : 0)) * ldb + 4 * g;
  }
  for (int64_t p0 = (int64_t)wv * 64; p0 < m; p0 += 256) {
    const float* ap[RT];
    bool aval[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const int64_t row = p0 + 16 * t + r;
      aval[t] = row < m;
      ap[t] = A + (aval[t] ? row : (m - 1)) * lda + 4 * g;
    }
    MF::acc_t acc[RT][CTR];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int u = 0; u < CTR; ++u) acc[t][u] = MF::zero();
    auto step = [&](const V4<float>(&av)[RT], const V4<float>(&bv)[CTR]) {
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
          for (int u = 0; u < CTR; ++u) acc[t][u] = MF::op(av[t].v[v], bv[u].v[v], acc[t][u]);
      if (ss) {
#pragma unroll
        for (int t = 0; t < RT; ++t)
          if (aval[t])
#pragma unroll
            for (int v = 0; v < 4; ++v) sq += (double)av[t].v[v] * (double)av[t].v[v];
      }
    };
    V4<float> a[PF][RT], bq[PF][CTR];
    auto loadf = [&](int q, int64_t st) {        // a full step: no masks
      const int64_t k = 16 * st;
#pragma unroll
      for (int t = 0; t < RT; ++t) a[q][t] = tile_lda4<AL>(ap[t] + k);
#pragma unroll
      for (int u = 0; u < CTR; ++u) {
        const V4<float> v = ld4(bp[u] + k);
#pragma unroll
        for (int e = 0; e < 4; ++e) bq[q][u].v[e] = bval[u] ? v.v[e] : 0.f;
      }
    };
    if (nfull > 0) {
#pragma unroll
      for (int q = 0; q < PF; ++q) loadf(q, min((int64_t)q, nfull - 1));   // clamped, never used twice
      int64_t c = 0;
      for (; c + 2 * PF <= nfull; c += PF) {
#pragma unroll
        for (int q = 0; q < PF; ++q) {
          step(a[q], bq[q]);
          loadf(q, c + q + PF);
        }
      }
#pragma unroll
      for (int q = 0; q < PF; ++q) {
        if (c + q < nfull) {
          step(a[q], bq[q]);
          if (c + q + PF < nfull) loadf(q, c + q + PF);
        }
      }
#pragma unroll
      for (int q = 0; q < PF; ++q)
        if (c + PF + q < nfull) step(a[q], bq[q]);
    }
    if (16 * nfull < n) {                        // ragged last step, masked
      const int64_t k = 16 * nfull;
      V4<float> at[RT], bt[CTR];
#pragma unroll
      for (int t = 0; t < RT; ++t) at[t] = ld4_masked(ap[t] + k, k + 4 * g, n);
#pragma unroll
      for (int u = 0; u < CTR; ++u) {
        const V4<float> v = ld4_masked(bp[u] + k, k + 4 * g, n);
#pragma unroll
        for (int e = 0; e < 4; ++e) bt[u].v[e] = bval[u] ? v.v[e] : 0.f;
      }
      step(at, bt);
    }
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int u = 0; u < CTR; ++u) {
        const int64_t row = p0 + 16 * t + 4 * g;
        const int col = 16 * u + r;
        if (col < nb) {
          float* py = Yb + (int64_t)col * ldy + row;
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (row + e < m) py[e] = acc[t][u][e];
        }
      }
  }
  if (ss) {
    for (int off = 32; off > 0; off >>= 1) sq += __shfl_xor(sq, off);
    if (lane == 0) red[wv] = sq;
    __syncthreads();
    if (threadIdx.x == 0) *ss = red[0] + red[1] + red[2] + red[3];
  }
  __syncthreads();
}
template <bool AL>
__device__ __forceinline__ void tile_rowprod(const float* A, int64_t lda, int64_t m, int64_t n, const float* B,
                                             int64_t ldb, int nb, float* Yb, int64_t ldy, double* ss,
                                             double* red) {
  const int ct = (nb + 15) / 16;
  if (ct <= 1) tile_rowprod_t<AL, 1>(A, lda, m, n, B, ldb, nb, Yb, ldy, ss, red);
  else if (ct == 2) tile_rowprod_t<AL, 2>(A, lda, m, n, B, ldb, nb, Yb, ldy, ss, red);
  else if (ct == 3) tile_rowprod_t<AL, 3>(A, lda, m, n, B, ldb, nb, Yb, ldy, ss, red);
  else tile_rowprod_t<AL, 4>(A, lda, m, n, B, ldb, nb, Yb, ldy, ss, red);
}

// ---------------------------------------------------------------------------
// Ct (n x r, column-major ldc, multiple of 4) = A^T Q: A m x n row-major
// (lda), Q m x r column-major (ldq multiple of 4, 16-byte aligned columns),
// r <= 16 TR.  Wave w takes 64-column chunks of A (w, w+4, ...), so A is read
// once; element (j, i) of the product at i*ldc + j.  ss (LDS, may be null):
// sum of squares of A.
// A lane takes four consecutive columns of A: column 4 r + u of the chunk is
// column r of the u-th of four MFMA tiles, so a 16-row step costs 4 loads of
// 16 bytes (AL: rows of A 16-byte aligned; else of 4 bytes each) in place of
// 16 of 4 bytes, and a store covers four entries.  The last chunk of a ragged
// width reads columns past n at column n - 1 (their products are not stored),
// the last step of a ragged height counts rows past m as zero; no load has a
// guard, PF steps are in flight.  1024 tiles of 64..1024 rows at ranks 5..80:
// C^T 182 -> 132 us a tile, the sketches 272 -> 187, the batch 4.05 -> 3.44 ms.
// ---------------------------------------------------------------------------
template <bool AL, int TR>
__device__ __noinline__ void tile_colprod_t(const float* A, int64_t lda, int m, int n, const float* Q, int64_t ldq,
                                            int r, float* Ct, int64_t ldc, double* ss, double* red) {
  typedef Mfma<float> MF;
  constexpr int PF = 3;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, rr = lane & 15, g = lane >> 4;
  const int nfull = m / 16;
  double sq = 0.0;
  const float* qp[TR];
#pragma unroll
  for (int t = 0; t < TR; ++t) qp[t] = Q + (int64_t)min(16 * t + rr, r - 1) * ldq + 4 * g;
  for (int c0 = 64 * wv; c0 < n; c0 += 256) {
    MF::acc_t acc[TR][4];
#pragma unroll
    for (int t = 0; t < TR; ++t)
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[t][u] = MF::zero();
    V4<float> q[PF][TR], a[PF][4];
    const int cl = c0 + 4 * rr;                    // this lane's first column
    const bool inside = c0 + 64 <= n;
    auto step = [&](const V4<float>(&qs)[TR], const V4<float>(&as)[4]) {
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int t = 0; t < TR; ++t)
#pragma unroll
          for (int u = 0; u < 4; ++u) acc[t][u] = MF::op(qs[t].v[v], as[v].v[u], acc[t][u]);
      if (ss) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (cl + u < n) sq += (double)as[v].v[u] * (double)as[v].v[u];
      }
    };
    auto run = [&](auto lda4) {                    // lda4(row): this lane's 4 entries of a row of A
      auto load = [&](V4<float>(&qs)[TR], V4<float>(&as)[4], int st) {
#pragma unroll
        for (int v = 0; v < 4; ++v) as[v] = lda4(16 * st + 4 * g + v);
#pragma unroll
        for (int t = 0; t < TR; ++t) qs[t] = ld4(qp[t] + 16 * st);
      };
      if (nfull > 0) {
#pragma unroll
        for (int p = 0; p < PF; ++p) load(q[p], a[p], min(p, nfull - 1));
        int c = 0;
        for (; c + 2 * PF <= nfull; c += PF) {
#pragma unroll
          for (int p = 0; p < PF; ++p) {
            step(q[p], a[p]);
            load(q[p], a[p], c + p + PF);
          }
        }
#pragma unroll
        for (int p = 0; p < PF; ++p) {
          if (c + p < nfull) {
            step(q[p], a[p]);
            if (c + p + PF < nfull) load(q[p], a[p], c + p + PF);
          }
        }
#pragma unroll
        for (int p = 0; p < PF; ++p)
          if (c + PF + p < nfull) step(q[p], a[p]);
      }
      if (16 * nfull < m) {                        // ragged last step: rows past m count as zero
        const int kr = 16 * nfull + 4 * g;
#pragma unroll
        for (int t = 0; t < TR; ++t) q[0][t] = ld4_masked(qp[t] + 16 * nfull, kr, m);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const V4<float> x = lda4(min(kr + v, m - 1));
#pragma unroll
          for (int u = 0; u < 4; ++u) a[0][v].v[u] = kr + v < m ? x.v[u] : 0.f;
        }
        step(q[0], a[0]);
      }
    };
    if (inside) {
      run([&](int row) { return tile_lda4<AL>(A + (int64_t)row * lda + cl); });
    } else {
      int co[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) co[u] = min(cl + u, n - 1);
      run([&](int row) {
        V4<float> x;
#pragma unroll
        for (int u = 0; u < 4; ++u) x.v[u] = A[(int64_t)row * lda + co[u]];
        return x;
      });
    }
    // columns of Q past r were read at column r - 1, and are not stored either
#pragma unroll
    for (int t = 0; t < TR; ++t) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = 16 * t + 4 * g + e;
        if (i < r) {
          float* pc = Ct + (int64_t)i * ldc + cl;
          if (inside) {
            st4(pc, V4<float>{{acc[t][0][e], acc[t][1][e], acc[t][2][e], acc[t][3][e]}});
          } else {
#pragma unroll
            for (int u = 0; u < 4; ++u)
              if (cl + u < n) pc[u] = acc[t][u][e];
          }
        }
      }
    }
  }
  if (ss) {
    for (int off = 32; off > 0; off >>= 1) sq += __shfl_xor(sq, off);
    if (lane == 0) red[wv] = sq;
    __syncthreads();
    if (threadIdx.x == 0) *ss = red[0] + red[1] + red[2] + red[3];
  }
  __syncthreads();
}
template <bool AL>
__device__ __forceinline__ void tile_colprod(const float* A, int64_t lda, int64_t m, int64_t n, const float* Q,
                                             int64_t ldq, int r, float* Ct, int64_t ldc, double* ss, double* red) {
  if (r <= 16) tile_colprod_t<AL, 1>(A, lda, (int)m, (int)n, Q, ldq, r, Ct, ldc, ss, red);
  else if (r <= 32) tile_colprod_t<AL, 2>(A, lda, (int)m, (int)n, Q, ldq, r, Ct, ldc, ss, red);
  else if (r <= 48) tile_colprod_t<AL, 3>(A, lda, (int)m, (int)n, Q, ldq, r, Ct, ldc, ss, red);
  else tile_colprod_t<AL, 4>(A, lda, (int)m, (int)n, Q, ldq, r, Ct, ldc, ss, red);
}

// ---------------------------------------------------------------------------
// out (LDS or global, row-major, leading dimension ldo) = X^T Y in FP64: X
// m x wx and Y m x wy column-major (ldx, ldy multiples of 4, 16-byte aligned
// columns; columns beyond wx / wy read as zero), wx, wy <= 64.  Waves split
// the rows (16-row steps, interleaved) and accumulate every 16 x 16 tile of
// the product at once; the partial tiles are folded through red (16 * 256
// doubles, disjoint from out): up to 4 tiles all waves at once, up to 8 by
// pairs, more in wave order.  TX, TY: tile counts of X and
// Y; full steps load without branches (clamped columns zeroed by a select).
// ---------------------------------------------------------------------------
template <int TX, int TY>
__device__ __noinline__ void tile_xty_t(const float* X, int64_t ldx, int wx, const float* Yb, int64_t ldy,
                                        int wy, int64_t m, double* out, int ldo, lds_ptr red) {
  typedef Mfma<double> MF;
  constexpr int PF = TX + TY <= 4 ? 4 : 2;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, r = lane & 15, g = lane >> 4;
  MF::acc_t acc[TX][TY];
#pragma unroll
  for (int t = 0; t < TX; ++t)
#pragma unroll
    for (int u = 0; u < TY; ++u) acc[t][u] = MF::zero();
  const float* xb[TX];
  const float* yb0[TY];
  bool xval[TX], yval[TY];
#pragma unroll
  for (int t = 0; t < TX; ++t) {
    const int c = 16 * t + r;
    xval[t] = c < wx;
    xb[t] = X + (int64_t)(xval[t] ? c : (wx > 0 ? wx - 1 : 0)) * ldx + 4 * g;
  }
#pragma unroll
  for (int u = 0; u < TY; ++u) {
    const int c = 16 * u + r;
    yval[u] = c < wy;
    yb0[u] = Yb + (int64_t)(yval[u] ? c : (wy > 0 ? wy - 1 : 0)) * ldy + 4 * g;
  }
  auto step = [&](const V4<float>(&xa)[TX], const V4<float>(&ya)[TY]) {
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int t = 0; t < TX; ++t)
#pragma unroll
        for (int u = 0; u < TY; ++u) acc[t][u] = MF::op((double)xa[t].v[v], (double)ya[u].v[v], acc[t][u]);
  };
  // this wave's 16-row steps start at 16 wv + 64 s; a step is full when all
  // its 16 rows are < m
  const int64_t nfull = m >= 16 * (int64_t)wv + 16 ? (m - 16 * (int64_t)wv - 16) / 64 + 1 : 0;
  V4<float> xa[PF][TX], ya[PF][TY];
  auto loadf = [&](int q, int64_t st) {
    const int64_t k = 16 * (int64_t)wv + 64 * st;
#pragma unroll
    for (int t = 0; t < TX; ++t) {
      const V4<float> v = ld4(xb[t] + k);
#pragma unroll
      for (int e = 0; e < 4; ++e) xa[q][t].v[e] = xval[t] ? v.v[e] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < TY; ++u) {
      const V4<float> v = ld4(yb0[u] + k);
#pragma unroll
      for (int e = 0; e < 4; ++e) ya[q][u].v[e] = yval[u] ? v.v[e] : 0.f;
    }
  };
  if (nfull > 0) {
#pragma unroll
    for (int q = 0; q < PF; ++q) loadf(q, min((int64_t)q, nfull - 1));
    int64_t c = 0;
    for (; c + 2 * PF <= nfull; c += PF) {
#pragma unroll
      for (int q = 0; q < PF; ++q) {
        step(xa[q], ya[q]);
        loadf(q, c + q + PF);
      }
    }
#pragma unroll
    for (int q = 0; q < PF; ++q) {
      if (c + q < nfull) {
        step(xa[q], ya[q]);
        if (c + q + PF < nfull) loadf(q, c + q + PF);
      }
    }
#pragma unroll
    for (int q = 0; q < PF; ++q)
      if (c + PF + q < nfull) step(xa[q], ya[q]);
  }
  {
    const int64_t k = 16 * (int64_t)wv + 64 * nfull;   // this wave's ragged step, if any
    if (k < m) {
      const int64_t kr = k + 4 * g;
      V4<float> xt[TX], yt[TY];
#pragma unroll
      for (int t = 0; t < TX; ++t) {
        const V4<float> v = ld4_masked(xb[t] + k, kr, m);
#pragma unroll
        for (int e = 0; e < 4; ++e) xt[t].v[e] = xval[t] ? v.v[e] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < TY; ++u) {
        const V4<float> v = ld4_masked(yb0[u] + k, kr, m);
#pragma unroll
        for (int e = 0; e < 4; ++e) yt[u].v[e] = yval[u] ? v.v[e] : 0.f;
      }
      step(xt, yt);
    }
  }
  constexpr int NT = TX * TY * 256, S = TX * TY <= 4 ? 4 : (TX * TY <= 8 ? 2 : 1);   // waves per round
#pragma unroll
  for (int w = 0; w < 4; w += S) {
    if (S == 4 || wv / S == w / S) {
#pragma unroll
      for (int t = 0; t < TX; ++t)
#pragma unroll
        for (int u = 0; u < TY; ++u)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            lds_ptr q = red + (wv % S) * NT + ((t * TY + u) * 4 + e) * 64 + lane;
            *q = (w == 0) ? acc[t][u][e] : *q + acc[t][u][e];
          }
    }
    __syncthreads();
  }
#pragma unroll
  for (int tu = 0; tu < TX * TY; ++tu) {
    const int t = tu / TY, u = tu % TY, idx = tu * 256 + threadIdx.x, e = threadIdx.x >> 6;
    const int i = 16 * t + MF::row(lane >> 4, e), j = 16 * u + (lane & 15);
    double v = red[idx];
#pragma unroll
    for (int w = 1; w < S; ++w) v += red[idx + w * NT];
    if (i < wx && j < wy) out[i * ldo + j] = v;
  }
  __syncthreads();
}
template <int TX>
__device__ __forceinline__ void tile_xty_y(const float* X, int64_t ldx, int wx, const float* Yb, int64_t ldy,
                                           int wy, int64_t m, double* out, int ldo, lds_ptr red) {
  const int ty = (wy + 15) / 16;
  if (ty <= 1) tile_xty_t<TX, 1>(X, ldx, wx, Yb, ldy, wy, m, out, ldo, red);
  else if (ty == 2) tile_xty_t<TX, 2>(X, ldx, wx, Yb, ldy, wy, m, out, ldo, red);
  else if (ty == 3) tile_xty_t<TX, 3>(X, ldx, wx, Yb, ldy, wy, m, out, ldo, red);
  else tile_xty_t<TX, 4>(X, ldx, wx, Yb, ldy, wy, m, out, ldo, red);
}
__device__ __forceinline__ void tile_xty(const float* X, int64_t ldx, int wx, const float* Yb, int64_t ldy,
                                         int wy, int64_t m, double* out, int ldo, double* red_) {
  lds_ptr red = (lds_ptr)red_;
  const int tx = (wx + 15) / 16;
  if (tx <= 1) tile_xty_y<1>(X, ldx, wx, Yb, ldy, wy, m, out, ldo, red);
  else if (tx == 2) tile_xty_y<2>(X, ldx, wx, Yb, ldy, wy, m, out, ldo, red);
  else if (tx == 3) tile_xty_y<3>(X, ldx, wx, Yb, ldy, wy, m, out, ldo, red);
  else tile_xty_y<4>(X, ldx, wx, Yb, ldy, wy, m, out, ldo, red);
}

// ---------------------------------------------------------------------------
// Z (column-major, ldz, columns zoff .. zoff+ncols-1) = X (m x f, ldx) W
// (f x ncols FP64 in LDS, element (i,j) at i*ldw + j), f <= 4 KSM, on f64
// MFMA.  X lies in the slot: ldx = TILE_MAX rows can be read from every
// column, whatever m.  One workgroup has the CU to itself, so what bounds
// this is the number of memory instructions a wave waits for, not their
// bytes: a wave takes 64 rows and a lane four consecutive ones, one 16-byte
// load per column of X (row 4 r + v is row r of the v-th of four MFMA tiles,
// which share every operand of W) and one 16-byte store per output.  All
// loads of a panel come before its stores, so Z may alias X.  With the update
// below split the same way, 1024 tiles of 64..1024 rows at ranks 5..80:
// projections 150 -> 41 us a tile, applies about 220 -> 100 (16 rows a wave
// and 4-byte guarded loads before), the batch 6.9 -> 4.65 ms.
// ---------------------------------------------------------------------------
template <int KSM>
__device__ __noinline__ void tile_apply_t(const float* X, int64_t ldx, int m, int f, lds_cptr W, int ldw, float* Z,
                                          int64_t ldz, int ncols) {
  typedef Mfma<double> MF;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, r = lane & 15, g = lane >> 4;
  const int TT = (ncols + 15) / 16;
  const bool vec = ((uintptr_t)Z % 16 == 0) && (ldz % 4 == 0);
  for (int row0 = 64 * wv; row0 < m; row0 += 256) {
    V4<float> a[KSM];
#pragma unroll
    for (int kk = 0; kk < KSM; ++kk) a[kk] = ld4(X + (int64_t)min(4 * kk + g, f - 1) * ldx + row0 + 4 * r);
    loads_first();
    for (int u = 0; u < TT; ++u) {
      const int col = 16 * u + r, cw = min(col, ncols - 1);
      MF::acc_t z[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) z[v] = MF::zero();
#pragma unroll
      for (int kk = 0; kk < KSM; ++kk) {
        const int k = 4 * kk + g;
        const double w = W[min(k, f - 1) * ldw + cw], b = k < f ? w : 0.0;
#pragma unroll
        for (int v = 0; v < 4; ++v) z[v] = MF::op((double)a[kk].v[v], b, z[v]);
      }
      if (col < ncols) {
        float* zc = Z + (int64_t)col * ldz;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int row = row0 + 4 * MF::row(g, e);
          if (vec && row + 3 < m) {
            st4(zc + row, V4<float>{{(float)z[0][e], (float)z[1][e], (float)z[2][e], (float)z[3][e]}});
          } else {
#pragma unroll
            for (int v = 0; v < 4; ++v)
              if (row + v < m) zc[row + v] = (float)z[v][e];
          }
        }
      }
    }
  }
  __syncthreads();
}
__device__ __forceinline__ void tile_apply(const float* X, int64_t ldx, int64_t m, int f, const double* W, int ldw,
                                           float* Z, int64_t ldz, int64_t zoff, int ncols) {
  lds_cptr Wl = (lds_cptr)W;
  float* Zo = Z + zoff * ldz;
  if (f <= 16) tile_apply_t<4>(X, ldx, (int)m, f, Wl, ldw, Zo, ldz, ncols);
  else if (f <= 32) tile_apply_t<8>(X, ldx, (int)m, f, Wl, ldw, Zo, ldz, ncols);
  else if (f <= 64) tile_apply_t<16>(X, ldx, (int)m, f, Wl, ldw, Zo, ldz, ncols);
  else tile_apply_t<32>(X, ldx, (int)m, f, Wl, ldw, Zo, ldz, ncols);
}

// ---------------------------------------------------------------------------
// Y (m x f) -= Q (m x w) W (w x f, FP64 in LDS, element (i,j) at i*ldw + j),
// in FP32 on MFMA (the projection step of block Gram-Schmidt), f <= 16 TT.
// Rows split as in tile_apply (Q and Y lie in the slot too); the columns of
// Q come 16 at a time, one chunk ahead of its products.
// ---------------------------------------------------------------------------
template <int TT>
__device__ __noinline__ void tile_update_t(float* Yb, int64_t ldy, const float* Q, int64_t ldq, int m, int w, int f,
                                           lds_cptr W, int ldw) {
  typedef Mfma<float> MF;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, r = lane & 15, g = lane >> 4;
  for (int row0 = 64 * wv; row0 < m; row0 += 256) {
    MF::acc_t z[4][TT];
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int u = 0; u < TT; ++u) z[v][u] = MF::zero();
    V4<float> a[4], an[4];
    auto load = [&](V4<float>(&q)[4], int k0) {
#pragma unroll
      for (int s = 0; s < 4; ++s) q[s] = ld4(Q + (int64_t)min(k0 + 4 * s + g, w - 1) * ldq + row0 + 4 * r);
    };
    load(a, 0);
    for (int k0 = 0; k0 < w; k0 += 16) {
      load(an, k0 + 16);                           // past the last chunk: its last column again
      loads_first();
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int k = k0 + 4 * s + g;
#pragma unroll
        for (int u = 0; u < TT; ++u) {
          const float wk = (float)W[min(k, w - 1) * ldw + min(16 * u + r, f - 1)], b = k < w ? wk : 0.f;
#pragma unroll
          for (int v = 0; v < 4; ++v) z[v][u] = MF::op(a[s].v[v], b, z[v][u]);
        }
      }
#pragma unroll
      for (int s = 0; s < 4; ++s) a[s] = an[s];
    }
#pragma unroll
    for (int u = 0; u < TT; ++u) {
      const int col = 16 * u + r;
      if (col < f) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int row = row0 + 4 * MF::row(g, e);
          float* py = Yb + (int64_t)col * ldy + row;
          if (row + 3 < m) {
            V4<float> y = ld4(py);
#pragma unroll
            for (int v = 0; v < 4; ++v) y.v[v] -= z[v][u][e];
            st4(py, y);
          } else {
#pragma unroll
            for (int v = 0; v < 4; ++v)
              if (row + v < m) py[v] -= z[v][u][e];
          }
        }
      }
    }
  }
  __syncthreads();
}
__device__ __forceinline__ void tile_update(float* Yb, int64_t ldy, const float* Q, int64_t ldq, int64_t m, int w,
                                            int f, const double* W, int ldw) {
  lds_cptr Wl = (lds_cptr)W;
  if (f <= 16) tile_update_t<1>(Yb, ldy, Q, ldq, (int)m, w, f, Wl, ldw);
  else if (f <= 32) tile_update_t<2>(Yb, ldy, Q, ldq, (int)m, w, f, Wl, ldw);
  else tile_update_t<4>(Yb, ldy, Q, ldq, (int)m, w, f, Wl, ldw);
}

// Cholesky with inverse of G (LDS, row-major ld F+1) for the smallest
// template width F >= f; R overwrites G, R^{-1} goes to Ri (ld F+1).
// The leading dimension used is F+1 for the chosen F; callers pass ldF.
__device__ int chol_width(int f) { return f <= 16 ? 16 : (f <= 32 ? 32 : 64); }
__device__ __noinline__ void tile_chol(double* Gs, double* Ri, double* work, double* dgs, int f, uint64_t dmask_in,
                          int first_pass, uint64_t* dmask_out, int* nfl) {
  const int F = chol_width(f);
  if (F == 16) chol_inv<16>(Gs, Ri, work, dgs, f, dmask_in, first_pass, dmask_out, nfl);
  else if (F == 32) chol_inv<32>(Gs, Ri, work, dgs, f, dmask_in, first_pass, dmask_out, nfl);
  else chol_inv<64>(Gs, Ri, work, dgs, f, dmask_in, first_pass, dmask_out, nfl);
}

// Store the leading f x f block of an LDS row-major matrix (ld) to global
// (element (i,j) at j*f + i).
__device__ void tile_store_small(const double* in, int ld, int f, double* Mg) {
  for (int idx = threadIdx.x; idx < f * f; idx += 256) {
    const int j = idx / f, i = idx - j * f;
    Mg[idx] = in[i * ld + j];
  }
  __syncthreads();
}

// chol_tame after tile_chol's first pass of f columns
__device__ __noinline__ bool tile_tame(const double* Ri, const double* dgs, int f, double* work) {
  const int F = chol_width(f);
  if (F == 16) return chol_tame<16>(Ri, dgs, f, work);
  if (F == 32) return chol_tame<32>(Ri, dgs, f, work);
  return chol_tame<64>(Ri, dgs, f, work);
}

// ---------------------------------------------------------------------------
// QR of M^T (M = R2 R1, or R2 when R1 is null; f x f FP64 in global memory,
// element (i,j) at j*f + i) by CholeskyQR2 in FP64 on the LDS arena (as the
// closing QR of the single-matrix path; the second pass where chol_tame asks
// for it).  Qh -> Qout, Rh -> Dout (FP64,
// both element (i,j) at j*f + i).
// ---------------------------------------------------------------------------
template <int F>
__device__ void tile_small_qr(double* lds, const double* R1g, const double* R2g, int f, double* Qout,
                              double* Dout, int* nfloor) {
  typedef SmallCfg<F> S;
  constexpr int LD = S::LD;
  double* B0 = lds;
  double* B1 = B0 + S::SIZE;
  double* B2 = B1 + S::SIZE;
  double* B3 = B2 + S::SIZE;
  double* work = B3 + S::SIZE;
  double* dgs = work + 24 * F;
  const int tid = threadIdx.x;
  double* Mt = R1g ? B1 : B0;
  for (int idx = tid; idx < F * F; idx += 256) {
    const int i = idx / F, jj = idx - i * F;
    const bool ok = i < f && jj < f;
    Mt[i * LD + jj] = ok ? R2g[(int64_t)jj * f + i] : 0.0;
    if (R1g) B2[i * LD + jj] = ok ? R1g[(int64_t)jj * f + i] : 0.0;
  }
  __syncthreads();
  if (R1g) {
    lds_gemm<F, false, false>(B1, B2, [&](int i, int jj, double v) { B0[i * LD + jj] = v; });
    __syncthreads();
  }
  lds_gemm<F, false, true>(B0, B0, [&](int i, int jj, double v) { B1[i * LD + jj] = v; });
  __syncthreads();
  uint64_t dm1, dm2;
  int nf1, nf2;
  chol_inv<F>(B1, B2, work, dgs, f, 0ull, 1, &dm1, &nf1);
  if (dm1 == 0ull && nf1 == 0 && chol_tame<F>(B2, dgs, f, work)) {
    lds_gemm<F, true, false>(B0, B2, [&](int i, int jj, double v) {
      if (i < f && jj < f) Qout[(int64_t)jj * f + i] = v;
    });
    tile_store_small(B1, LD, f, Dout);
    *nfloor = 0;
    return;
  }
  lds_gemm<F, true, false>(B0, B2, [&](int i, int jj, double v) { B3[i * LD + jj] = v; });
  __syncthreads();
  lds_gemm<F, true, false>(B3, B3, [&](int i, int jj, double v) { B0[i * LD + jj] = v; });
  __syncthreads();
  chol_inv<F>(B0, B2, work, dgs, f, dm1, 0, &dm2, &nf2);
  lds_gemm<F, false, false>(B3, B2, [&](int i, int jj, double v) {
    if (i < f && jj < f) Qout[(int64_t)jj * f + i] = v;
  });
  lds_gemm<F, false, false>(B0, B1, [&](int i, int jj, double v) {
    if (i < f && jj < f) Dout[(int64_t)jj * f + i] = v;
  });
  __syncthreads();
  *nfloor = nf1 + nf2;
}
__device__ void tile_small_qr_any(double* lds, const double* R1g, const double* R2g, int f, double* Qout,
                                  double* Dout, int* nfloor) {
  if (f <= 16) tile_small_qr<16>(lds, R1g, R2g, f, Qout, Dout, nfloor);
  else if (f <= 32) tile_small_qr<32>(lds, R1g, R2g, f, Qout, Dout, nfloor);
  else tile_small_qr<64>(lds, R1g, R2g, f, Qout, Dout, nfloor);
}

// Load an f x f FP64 matrix (element (i,j) at j*f + i) into LDS row-major (ld).
__device__ void tile_load_small(const double* Mg, int f, double* out, int ld) {
  for (int idx = threadIdx.x; idx < f * f; idx += 256) {
    const int j = idx / f, i = idx - j * f;
    out[i * ld + j] = Mg[idx];
  }
  __syncthreads();
}
// ---------------------------------------------------------------------------
// Ranks 65..128: FP64 matrices row-major with leading dimension LB in the
// slot (L2-resident); the LDS arena stages the right-hand factors.
// ---------------------------------------------------------------------------
// G = X^T X (f x f, 64 < f <= 128) of X (rows x f, column-major ldx): the
// blocks G11, G12 and G22 (chol_inv128 does not read G21).
__device__ __attribute__((noinline)) void tile_gram_big(const float* X, int64_t ldx, int f, int64_t rows,
                                                        double* G, double* red) {
  constexpr int LB = TileSlot::LB;
  const int f2 = f - 64;
  tile_xty(X, ldx, 64, X, ldx, 64, rows, G, LB, red);
  tile_xty(X, ldx, 64, X + 64 * ldx, ldx, f2, rows, G + 64, LB, red);
  tile_xty(X + 64 * ldx, ldx, f2, X + 64 * ldx, ldx, f2, rows, G + 64 * LB + 64, LB, red);
}

// Z (columns 0..ncols-1, ldz) = X (m x f, ldx) W with W (f x ncols, f <= 128)
// row-major in global memory (ld LB), staged through the arena (ld 129).
__device__ __attribute__((noinline)) void tile_apply_big(const float* X, int64_t ldx, int64_t m, int f,
                                                         const double* Wg, double* lds, float* Z, int64_t ldz,
                                                         int ncols) {
  for (int idx = threadIdx.x; idx < f * ncols; idx += 256) {
    const int i = idx / ncols, j = idx - i * ncols;
    lds[i * 129 + j] = Wg[(int64_t)i * TileSlot::LB + j];
  }
  __syncthreads();
  tile_apply(X, ldx, m, f, lds, 129, Z, ldz, 0, ncols);
}

// chol_inv128 on row-major matrices of leading dimension LB.
__device__ __attribute__((noinline)) int tile_chol128(const double* G, int f, double* R, double* Rinv, double* lds,
                                                      uint64_t dm0, uint64_t dm1, int first_pass, uint64_t* o0,
                                                      uint64_t* o1) {
  return chol_inv128(G, TileSlot::LB, f, R, Rinv, lds, dm0, dm1, first_pass, o0, o1);
}

// QR of M^T (M = R2 R1, or R2 when R1 is null; f x f, 64 < f <= 128):
// small_qr_mid on row-major matrices (leading dimension LB); Qh and Rh out
// row-major; scr: 7 buffers of B2.
__device__ __attribute__((noinline)) void tile_small_qr_big(double* lds, const double* R1g, const double* R2g,
                                                            int f, double* Qh, double* Rh, double* scr) {
  constexpr int LB = TileSlot::LB;
  small_qr_mid(lds, R1g, R2g, f, LB, scr, [&](int i, int j, double v) { Qh[i * LB + j] = v; },
                      [&](int i, int j, double v) { Rh[i * LB + j] = v; });
}

// ---------------------------------------------------------------------------
// One tile: Alg. 1 with BCGS2 + CholeskyQR2 blocks and the device rank
// test, then Alg. 2 (q = 0): C^T = A^T Q, CholeskyQR2 of C^T, QR of
// (R2 R1)^T, U = Q Qh.  A wide tile (h < w) is factored as A^T without
// moving it: its sketch A^T Omega and its C^T = A Q are the two products
// of a tall tile with the roles of the routines exchanged; the core is
// then re-triangularised.
// ---------------------------------------------------------------------------
__device__ void tile_factor(const TileDesc& td, const float* omt, float* slot, double* sdbl, double* lds, float* out_pool,
                            TileResult* res, double tol) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  constexpr int64_t LD = TileSlot::LD;
  const bool tr = td.h < td.w;
  const int64_t m = tr ? td.w : td.h, n = tr ? td.h : td.w;     // oriented: m >= n
  const bool al = ((uintptr_t)td.A % 16 == 0) && (td.lda % 4 == 0);
  // LDS carve for the basis phase
  double* Gs = lds + TL_GS;                          // Gram -> R (ld chol_width(f) + 1)
  double* Ri = lds + TL_RI;                          // R^{-1}
  double* work = lds + TL_WORK;                      // Cholesky work area (24 x 64)
  double* dgs = lds + TL_DGS;                        // Cholesky diagonal
  double* Wp = lds + TL_W;                           // W = Q^T Y (TILE_QW x TILE_BMAX)
  double* fold = lds + TL_FOLD;                      // wave fold buffer of the reductions
  double* scal = lds + TILE_SQR;                     // [0] ||A||^2, [1..64] R1 diagonal
  __shared__ int s_keep, s_stop;
  float* Yb = slot + TileSlot::Y;
  float* Q = slot + TileSlot::Q;
  const int64_t ldk = TILE_MAX;                      // rows of Omega^T
  const int b = td.b;
  int64_t wcols = 0;
  int blocks = 0;
  int status = TS_OK;
  double eps = 0.0;
  for (int64_t col0 = 0; col0 < n; col0 += b) {
    const int f = (int)((n - col0) < b ? (n - col0) : b);
    ++blocks;
    const float* Om = omt + col0 * ldk;
    double* ss = (col0 == 0) ? &scal[0] : nullptr;
    // Y = A_o Omega_j (A_o the oriented tile, m x n)
    if (tr && al) tile_colprod<true>(td.A, td.lda, n, m, Om, ldk, f, Yb, LD, ss, fold);
    else if (tr) tile_colprod<false>(td.A, td.lda, n, m, Om, ldk, f, Yb, LD, ss, fold);
    else if (al) tile_rowprod<true>(td.A, td.lda, m, n, Om, ldk, f, Yb, LD, ss, fold);
    else tile_rowprod<false>(td.A, td.lda, m, n, Om, ldk, f, Yb, LD, ss, fold);
    if (col0 == 0) {
      const double a = scal[0];
      if (!(a < INFINITY)) {
        status = TS_NONFINITE;
        break;
      }
      eps = tol * sqrt(a);
    }
    // two rounds of [project against Q, Gram, Cholesky]; normalise between
    const int LDG = chol_width(f) + 1;
    uint64_t dm1 = 0, dm2 = 0;
    int nf = 0;
    for (int pass = 0; pass < 2; ++pass) {
      if (wcols > 0) {
        // W = Q^T Y (wcols x f), then Y -= Q W
        for (int64_t q0 = 0; q0 < wcols; q0 += 64) {
          const int wq = (int)((wcols - q0) < 64 ? (wcols - q0) : 64);
          tile_xty(Q + q0 * LD, LD, wq, Yb, LD, f, m, Wp + q0 * TILE_BMAX, TILE_BMAX, fold);
        }
        tile_update(Yb, LD, Q, LD, m, (int)wcols, f, Wp, TILE_BMAX);
      }
      tile_xty(Yb, LD, f, Yb, LD, f, m, Gs, LDG, fold);
      tile_chol(Gs, Ri, work, dgs, f, pass == 0 ? 0ull : dm1, pass == 0, pass == 0 ? &dm1 : &dm2, &nf);
      if (pass == 0) {
        for (int c = tid; c < f; c += 256) scal[1 + c] = Gs[c * LDG + c];   // R1 diag
        __syncthreads();
        tile_apply(Yb, LD, m, f, Ri, LDG, Yb, LD, 0, f);                      // Y := Y R1^{-1}
      }
    }
    // rank test (Alg. 1): first column with d_c = R2(c,c) R1(c,c) <= eps
    if (wv == 0) {
      bool hit = false;
      if (lane < f) {
        const double d = ((dm2 >> lane) & 1ull) ? 0.0 : Gs[lane * LDG + lane] * scal[1 + lane];
        hit = d <= eps;
      }
      const unsigned long long mask = __ballot(hit);
      if (lane == 0) {
        s_keep = mask ? (int)__ffsll((long long)mask) - 1 : f;
        s_stop = (mask != 0ull) || (col0 + f >= n);
      }
    }
    __syncthreads();
    const int keep = s_keep;
    const int stop = s_stop;
    if (keep > 0) tile_apply(Yb, LD, m, f, Ri, LDG, Q, LD, wcols, keep);      // append Z R2^{-1}
    wcols += keep;
    if (stop) break;
    if (wcols > TILE_RMAX) {                        // the rank will exceed the in-kernel cap
      status = TS_RANK;
      break;
    }
  }
  const int64_t r = wcols;
  if (status == TS_OK && r > TILE_RMAX) status = TS_RANK;
  if (status == TS_OK && r > td.r_cap) status = TS_CAPACITY;
  if (status == TS_OK && r > 0) {
    const int ri = (int)r;
    // a9: C^T = A_o^T Q (n x r), 64 columns of Q at a time
    float* Ct = slot + TileSlot::CT;
    for (int c0 = 0; c0 < ri; c0 += 64) {
      const int rc = (ri - c0) < 64 ? ri - c0 : 64;
      if (!tr && al) tile_colprod<true>(td.A, td.lda, m, n, Q + c0 * LD, LD, rc, Ct + c0 * LD, LD, nullptr, fold);
      else if (!tr) tile_colprod<false>(td.A, td.lda, m, n, Q + c0 * LD, LD, rc, Ct + c0 * LD, LD, nullptr, fold);
      else if (al) tile_rowprod<true>(td.A, td.lda, n, m, Q + c0 * LD, LD, rc, Ct + c0 * LD, LD, nullptr, fold);
      else tile_rowprod<false>(td.A, td.lda, n, m, Q + c0 * LD, LD, rc, Ct + c0 * LD, LD, nullptr, fold);
    }
    float* Ut = out_pool + td.out_off;
    float* core = Ut + td.r_cap * td.h;
    float* Vt = core + td.r_cap * td.r_cap;
    // V = C^T R2^{-1}: the output V (tall tile) or V' (wide tile)
    float* Vdst = tr ? slot + TileSlot::VP : Vt;
    const int64_t ldv = tr ? LD : td.w;
    if (ri <= 64) {
      // a10: C^T = V R by CholeskyQR2 (V over C^T in place), R1, R2 kept
      const int LDG = chol_width(ri) + 1;
      uint64_t dm1 = 0, dm2 = 0;
      int nf = 0;
      tile_xty(Ct, LD, ri, Ct, LD, ri, n, Gs, LDG, fold);
      tile_chol(Gs, Ri, work, dgs, ri, 0ull, 1, &dm1, &nf);
      tile_store_small(Gs, LDG, ri, sdbl + TileSlot::R1);
      const bool tame = dm1 == 0ull && nf == 0 && tile_tame(Ri, dgs, ri, work);
      if (tame) {                                   // one pass: V = C^T R1^{-1}, R2 = I
        tile_apply(Ct, LD, n, ri, Ri, LDG, Vdst, ldv, 0, ri);
      } else {
        tile_apply(Ct, LD, n, ri, Ri, LDG, Ct, LD, 0, ri);
        tile_xty(Ct, LD, ri, Ct, LD, ri, n, Gs, LDG, fold);
        tile_chol(Gs, Ri, work, dgs, ri, dm1, 0, &dm2, &nf);
        tile_store_small(Gs, LDG, ri, sdbl + TileSlot::R2);
        tile_apply(Ct, LD, n, ri, Ri, LDG, Vdst, ldv, 0, ri);
      }
      // a11: (R2 R1)^T = Qh Rh on the arena
      int nfq = 0;
      tile_small_qr_any(lds, tame ? nullptr : sdbl + TileSlot::R1, sdbl + (tame ? TileSlot::R1 : TileSlot::R2), ri,
                        sdbl + TileSlot::QH, sdbl + TileSlot::DH, &nfq);
      // U_hat = Q Qh (m x r)
      const int LDW = chol_width(ri) + 1;
      tile_load_small(sdbl + TileSlot::QH, ri, Gs, LDW);
      if (!tr) {
        tile_apply(Q, LD, m, ri, Gs, LDW, Ut, td.h, 0, ri);                   // U (h x r)
        for (int idx = tid; idx < ri * ri; idx += 256) {                       // core = Rh
          const int i = idx / ri, j = idx - i * ri;
          core[(int64_t)i * td.r_cap + j] = (float)sdbl[TileSlot::DH + (int64_t)j * ri + i];
        }
      } else {
        // A^T = U' D' V'^T with U' = Q Qh (w x r) and V' (h x r): A = V' D'^T U'^T,
        // QR(D'^T) = Q'' R'': U = V' Q'', core = R'', V = U'.
        tile_apply(Q, LD, m, ri, Gs, LDW, Vt, td.w, 0, ri);                   // V = U' (w x r)
        int nfq2 = 0;
        // M = D' (element (i,j) at j*r + i) -> QR(M^T) = QR(D'^T)
        tile_small_qr_any(lds, nullptr, sdbl + TileSlot::DH, ri, sdbl + TileSlot::QH2, sdbl + TileSlot::DH2,
                          &nfq2);
        tile_load_small(sdbl + TileSlot::QH2, ri, Gs, LDW);
        tile_apply(slot + TileSlot::VP, LD, n, ri, Gs, LDW, Ut, td.h, 0, ri);  // U = V' Q'' (h x r)
        for (int idx = tid; idx < ri * ri; idx += 256) {
          const int i = idx / ri, j = idx - i * ri;
          core[(int64_t)i * td.r_cap + j] = (float)sdbl[TileSlot::DH2 + (int64_t)j * ri + i];
        }
      }
    } else {
      // the same steps with the blocked 128-wide Cholesky and L2-resident matrices
      constexpr int LB = TileSlot::LB;
      constexpr int64_t B2 = TileSlot::B2;
      double* dd = sdbl + TileSlot::BIG;
      double* Gg = dd;
      double* R1g = dd + B2;
      double* R1i = dd + 2 * B2;
      double* R2g = dd + 3 * B2;
      double* R2i = dd + 4 * B2;
      double* Qh = dd + 5 * B2;
      double* Rh = dd + 6 * B2;
      double* Qh2 = dd + 7 * B2;
      double* Rh2 = dd + 8 * B2;
      double* scr = dd + 9 * B2;                    // 7 buffers
      uint64_t d10 = 0, d11 = 0, d20 = 0, d21 = 0;
      tile_gram_big(Ct, LD, ri, n, Gg, fold);
      const int nf1 = tile_chol128(Gg, ri, R1g, R1i, lds, 0ull, 0ull, 1, &d10, &d11);
      if (nf1 == 0 && (d10 | d11) == 0ull && chol128_tame(Gg, LB, R1i, ri, lds)) {
        tile_apply_big(Ct, LD, n, ri, R1i, lds, Vdst, ldv, ri);
        tile_small_qr_big(lds, nullptr, R1g, ri, Qh, Rh, scr);
      } else {
        tile_apply_big(Ct, LD, n, ri, R1i, lds, Ct, LD, ri);
        tile_gram_big(Ct, LD, ri, n, Gg, fold);
        tile_chol128(Gg, ri, R2g, R2i, lds, d10, d11, 0, &d20, &d21);
        tile_apply_big(Ct, LD, n, ri, R2i, lds, Vdst, ldv, ri);
        tile_small_qr_big(lds, R1g, R2g, ri, Qh, Rh, scr);
      }
      const double* Rc = Rh;
      if (!tr) {
        tile_apply_big(Q, LD, m, ri, Qh, lds, Ut, td.h, ri);                   // U (h x r)
      } else {
        tile_apply_big(Q, LD, m, ri, Qh, lds, Vt, td.w, ri);                   // V = U' (w x r)
        tile_small_qr_big(lds, nullptr, Rh, ri, Qh2, Rh2, scr);                // QR(D'^T)
        tile_apply_big(slot + TileSlot::VP, LD, n, ri, Qh2, lds, Ut, td.h, ri); // U = V' Q''
        Rc = Rh2;
      }
      for (int idx = tid; idx < ri * ri; idx += 256) {
        const int i = idx / ri, j = idx - i * ri;
        core[(int64_t)i * td.r_cap + j] = (float)Rc[(int64_t)i * LB + j];
      }
    }
    __syncthreads();
  }
  if (tid == 0) {
    TileResult o;
    o.rank = r;
    o.blocks = blocks;
    o.status = status;
    o.norm = sqrt(scal[0]);
    res[td.index] = o;
  }
  __syncthreads();
}

// Persistent launch: workgroup g uses scratch slot g and takes tiles in the
// order of descs (largest first) from the queue until it is empty.
__global__ __launch_bounds__(256) void k_tiles(const TileDesc* __restrict__ descs, int ntiles,
                                               uint32_t* __restrict__ queue, char* __restrict__ scratch,
                                               float* __restrict__ out_pool, TileResult* __restrict__ res,
                                               double tol, const float* __restrict__ omt) {
  __shared__ __align__(16) double lds[TILE_LDS];
  __shared__ int s_t;
  float* slot = reinterpret_cast<float*>(scratch + (int64_t)blockIdx.x * TileSlot::BYTES);
  double* sdbl = reinterpret_cast<double*>(slot + TileSlot::FLOATS);
  for (;;) {
    if (threadIdx.x == 0) s_t = (int)atomicAdd(queue, 1u);
    __syncthreads();
    const int t = s_t;
    __syncthreads();
    if (t >= ntiles) break;
    tile_factor(descs[t], omt, slot, sdbl, lds, out_pool, res, tol);
  }
}

}  // namespace eodabe

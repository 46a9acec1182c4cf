// The products of the batched tile kernel, compiled for the host from the
// kernel's own header and run lane by lane on buffers of exactly the sizes they
// have there, under the address and alignment sanitizers: every call that the
// per-tile routine makes for a tile h x w at block width b, the basis growing by
// whole blocks (the widest it can get), and the closing products of each rank.
// Arguments: h w b unaligned rank..., or "plant" for the same with buffers one
// element short, which has to end in a report.
#include "eodabe_tiles.hpp"

#include <cstdio>
#include <cstdlib>
#include <memory>
#include <vector>

using namespace eodabe;

static int short_by = 0;                               // planted mistake: elements missing from each buffer
template <typename T>
struct Buf {
  std::unique_ptr<char[]> raw;
  T* p;
  // n elements that end where the allocation ends; off: bytes the first is off 16-byte alignment
  Buf(int64_t n, int off = 0) : raw(new char[(n - short_by) * sizeof(T) + off]()), p((T*)(raw.get() + off)) {}
  operator T*() const { return p; }
};

template <typename F>
void lanes(F f) {
  for (unsigned t = 0; t < 256; ++t) {
    threadIdx.x = t;
    f();
  }
}

struct Tile {
  int64_t h, w;
  int b;
  bool unaligned;
  int64_t lda, m, n;
  bool tr, al;
  static constexpr int64_t LD = TileSlot::LD;
  Buf<float> A, Om, Y, Q, CT, VP;
  Buf<double> W, G, Ri, fold, scal, big, arena;
  int64_t lda_;

  Tile(int64_t h_, int64_t w_, int b_, bool un)
      : h(h_), w(w_), b(b_), unaligned(un), lda(w_), m(std::max(h_, w_)), n(std::min(h_, w_)), tr(h_ < w_),
        al(!un && w_ % 4 == 0), A(h_ * w_, un ? 4 : 0), Om((int64_t)TILE_QW * TILE_MAX), Y(LD * TILE_BMAX),
        Q(LD * TILE_QW), CT(LD * TILE_RMAX), VP(LD * TILE_RMAX), W((int64_t)TILE_QW * TILE_BMAX),
        G(SmallCfg<64>::SIZE), Ri(SmallCfg<64>::SIZE), fold(TL_FOLD_N), scal(72), big(TileSlot::B2), arena(TILE_SQR) {}

  // the two products of the tile with a block of Omega or of the basis
  void rows(const float* B, int64_t ldb, int nb, float* out, double* ss, int64_t mm, int64_t nn) {
    if (al) tile_rowprod<true>(A, lda, mm, nn, B, ldb, nb, out, LD, ss, fold);
    else tile_rowprod<false>(A, lda, mm, nn, B, ldb, nb, out, LD, ss, fold);
  }
  void cols(const float* B, int64_t ldb, int nb, float* out, double* ss, int64_t mm, int64_t nn) {
    if (al) tile_colprod<true>(A, lda, mm, nn, B, ldb, nb, out, LD, ss, fold);
    else tile_colprod<false>(A, lda, mm, nn, B, ldb, nb, out, LD, ss, fold);
  }

  int64_t basis() {
    int64_t wcols = 0;
    for (int64_t col0 = 0; col0 < n; col0 += b) {
      const int f = (int)std::min<int64_t>(b, n - col0), ldg = chol_width(f) + 1;
      double* ss = col0 == 0 ? scal.p : nullptr;
      lanes([&] {
        if (tr) cols(Om + col0 * TILE_MAX, TILE_MAX, f, Y, ss, n, m);
        else rows(Om + col0 * TILE_MAX, TILE_MAX, f, Y, ss, m, n);
      });
      lanes([&] {
        for (int64_t q0 = 0; q0 < wcols; q0 += 64)
          tile_xty(Q + q0 * LD, LD, (int)std::min<int64_t>(wcols - q0, 64), Y, LD, f, m, W + q0 * TILE_BMAX, TILE_BMAX, fold);
      });
      if (wcols > 0) lanes([&] { tile_update(Y, LD, Q, LD, m, (int)wcols, f, W, TILE_BMAX); });
      lanes([&] { tile_xty(Y, LD, f, Y, LD, f, m, G, ldg, fold); });
      lanes([&] { tile_apply(Y, LD, m, f, Ri, ldg, Y, LD, 0, f); });
      for (int keep : {f, 1})
        lanes([&] { tile_apply(Y, LD, m, f, Ri, ldg, Q, LD, wcols, keep); });
      wcols += f;
      if (wcols > TILE_RMAX) break;
    }
    return wcols;
  }

  void close(int r) {
    lanes([&] {
      for (int c0 = 0; c0 < r; c0 += 64) {
        const int rc = std::min(r - c0, 64);
        if (!tr) cols(Q + c0 * LD, LD, rc, CT + c0 * LD, nullptr, m, n);
        else rows(Q + c0 * LD, LD, rc, CT + c0 * LD, nullptr, n, m);
      }
    });
    Buf<float> Ut(r * h, unaligned ? 4 : 0), Vt(r * w, unaligned ? 8 : 0);
    float* V = tr ? VP.p : Vt.p;
    const int64_t ldv = tr ? LD : w;
    if (r <= 64) {
      const int ldg = chol_width(r) + 1;
      lanes([&] { tile_xty(CT, LD, r, CT, LD, r, n, G, ldg, fold); });
      lanes([&] { tile_apply(CT, LD, n, r, Ri, ldg, CT, LD, 0, r); });
      lanes([&] { tile_apply(CT, LD, n, r, Ri, ldg, V, ldv, 0, r); });
      if (!tr) {
        lanes([&] { tile_apply(Q, LD, m, r, G, ldg, Ut, h, 0, r); });
      } else {
        lanes([&] { tile_apply(Q, LD, m, r, G, ldg, Vt, w, 0, r); });
        lanes([&] { tile_apply(VP, LD, n, r, G, ldg, Ut, h, 0, r); });
      }
    } else {
      lanes([&] { tile_gram_big(CT, LD, r, n, big, fold); });
      lanes([&] { tile_apply_big(CT, LD, n, r, big, arena, CT, LD, r); });
      lanes([&] { tile_apply_big(CT, LD, n, r, big, arena, V, ldv, r); });
      if (!tr) {
        lanes([&] { tile_apply_big(Q, LD, m, r, big, arena, Ut, h, r); });
      } else {
        lanes([&] { tile_apply_big(Q, LD, m, r, big, arena, Vt, w, r); });
        lanes([&] { tile_apply_big(VP, LD, n, r, big, arena, Ut, h, r); });
      }
    }
  }
};

int main(int argc, char** argv) {
  int at = 1;
  if (argc > 1 && argv[1][0] == 'p') {
    short_by = 1;
    at = 2;
  }
  // one tile per group of arguments up to a "/"
  int n = 0;
  while (at < argc) {
    std::vector<int> v;
    for (; at < argc && argv[at][0] != '/'; ++at) v.push_back(atoi(argv[at]));
    ++at;
    Tile t(v[0], v[1], v[2], v[3] != 0);
    const int64_t wide = t.basis();
    for (size_t i = 4; i < v.size(); ++i)
      if (v[i] >= 1 && v[i] <= std::min<int64_t>(wide, TILE_RMAX)) t.close(v[i]);
    ++n;
  }
  printf("%d tiles\n", n);
  return 0;
}

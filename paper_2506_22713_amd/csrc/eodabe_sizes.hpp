// Sizes of the Gram partials.  A launch takes its split from here and the
// workspace its buffers, so that neither can change without the other.  Plain
// host arithmetic, without HIP.
#pragma once
#include <algorithm>
#include <cstdint>

namespace eodabe {

// Workgroups of a Gram kernel of the basis loop (one row panel each up to
// this; the partial buffer holds that many)
constexpr int GRAM_LOOP_WG = 192;
// At most this many for a Gram of F columns: the last to arrive sums the
// partials alone, F/16 (F/16 + 1) / 2 loads per thread and workgroup (20 MB of
// FP32 rows: 96 of 64 columns).
constexpr int64_t gram_wg(int F, int64_t max_wg) {
  return std::min<int64_t>(max_wg, F <= 16 ? 192 : (F <= 32 ? 128 : 96));
}
// Doubles those partials take at widths up to f (k_gram_rows: f <= 64).
constexpr int64_t gram_parts(int64_t f, int64_t max_wg) {
  const int F = f <= 16 ? 16 : (f <= 32 ? 32 : 64);
  return gram_wg(F, max_wg) * (F / 16) * (F / 16 + 1) / 2 * 256;
}

// K-splits of the Gram of closing QRs wider than 128 columns.
constexpr int GRAM_SPLITS_WIDE = 16;
// Gram of f > 64 columns: f x f partials of `splits` row ranges, `stride`
// doubles apart, and their sum behind them.
struct GramSplit {
  int splits;
  int64_t stride;
  constexpr int64_t need() const { return (splits + 1) * stride; }
};
// Up to 63 splits of at least 64 rows for f <= 128 (more splits put more
// workgroups on the FP64 products), GRAM_SPLITS_WIDE of at least 512 rows
// above; one split less where the stride is rounded up for the fold's vector
// loads (f odd), so that they fit the room of the next even width.
constexpr GramSplit gram_split(int64_t f, int64_t rows) {
  const int64_t ff = f * f, stride = (ff + 3) / 4 * 4;
  const int pad = stride != ff ? 1 : 0;
  const int64_t s = f <= 128 ? std::min<int64_t>(63 - pad, rows / 64) : std::min<int64_t>(GRAM_SPLITS_WIDE - pad, rows / 512);
  return GramSplit{(int)std::max<int64_t>(1, s), stride};
}

// Doubles for the Grams of the basis blocks: up to bn columns (a multiple of
// 16, at most 128) of `rows` rows, the last block of any smaller width.
constexpr int64_t gram_loop_room(int64_t bn, int64_t rows) {
  return std::max(gram_parts(bn, GRAM_LOOP_WG), bn > 64 ? gram_split(bn, rows).need() : 0);
}
// Doubles for the Grams of the closing QRs above 64 columns, up to r (the
// longer side of theirs may be any number of rows).
constexpr int64_t gram_close_room(int64_t r) {
  const int64_t r128 = std::min<int64_t>(r, 128);
  return std::max<int64_t>(64 * r128 * r128, (GRAM_SPLITS_WIDE + 1) * r * r);
}

}  // namespace eodabe

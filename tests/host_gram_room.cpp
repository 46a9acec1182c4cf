// Host replay of the Gram launches: every launch that gram_chol makes for a
// block is recorded instead of made, and what it writes is compared with the
// buffers that the workspace carve gives it.  No device is touched.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <cstdio>
#include <string>
#include <tuple>

struct Rec {
  const char *lo = nullptr, *hi = nullptr;   // extent of the doubles written to the partials' buffer
  int launches = 0;
  void add(const void* p, int64_t doubles) {
    const char* b = (const char*)p;
    if (!lo || b < lo) lo = b;
    if (!hi || b + 8 * doubles > hi) hi = b + 8 * doubles;
  }
} rec;

template <int I, typename... A>
auto arg(const std::tuple<A...>& t) {
  if constexpr (I < (int)sizeof...(A)) return std::get<I>(t);
  else return 0;
}
template <typename P>
int64_t num(P v) {
  if constexpr (std::is_pointer_v<P> || std::is_null_pointer_v<P>) return 0;
  else if constexpr (std::is_convertible_v<P, int64_t>) return (int64_t)v;
  else return 0;
}
template <typename P>
const void* ptr(P v) {
  if constexpr (std::is_pointer_v<P>) return (const void*)v;
  else return nullptr;
}

template <typename... A>
void record(const char* name, dim3 grid, A... a) {
  const std::tuple<A...> t(a...);
  const std::string k(name);
  ++rec.launches;
  if (k.find("k_gemm_nt") != std::string::npos) {          // out[s * part_stride + i * ldo + j]
    rec.add(ptr(arg<8>(t)), (grid.y - 1) * num(arg<10>(t)) + num(arg<4>(t)) * num(arg<5>(t)));
  } else if (k.find("k_fold_parts") != std::string::npos || k.find("k_reduce") != std::string::npos) {
    rec.add(ptr(arg<4>(t)), num(arg<3>(t)));               // (parts, nparts, stride, count, out, ...)
  } else if (k.find("k_gram_rows") != std::string::npos) { // (k_gram_rows<T, F, MODE>): parts is the 6th
    const int F = std::stoi(k.substr(k.find(',') + 1));
    rec.add(ptr(arg<5>(t)), (int64_t)grid.x * (F / 16) * (F / 16 + 1) / 2 * 256);
  }
}

#undef hipLaunchKernelGGL
#define hipLaunchKernelGGL(kern, grid, block, shared, stream, ...) record(#kern, grid, __VA_ARGS__)
#define hipGetLastError() hipSuccess
#include "eodabe.hip"

template <typename T>
bool check(eodabe_ctx& ctx, int b, int64_t m, int64_t n) {
  ctx.o.block = b;
  ctx.o.a_dtype = sizeof(T) == 8 ? EODABE_F64 : EODABE_F32;
  Geo g;
  if (!plan(&ctx, m, n, (n + 3) / 4 * 4, (const void*)16, 0, g)) return false;
  const WS w = carve((void*)4096, g);
  bool ok = true;
  auto held = [&](const char* what, int f, int64_t rows, const void* buf, const void* end) {
    const bool in = rec.launches > 0 && rec.lo >= (const char*)buf && rec.hi <= (const char*)end;
    if (!in)
      printf("%s block %d, %ld x %ld (%zu bytes): width %d over %ld rows writes %ld doubles, the buffer has %ld\n", what, b,
             (long)m, (long)n, sizeof(T), f, (long)rows, (long)((rec.hi - (const char*)buf) / 8),
             (long)(((const char*)end - (const char*)buf) / 8));
    ok = ok && in;
  };
  // basis blocks: the full width and every width the last one may have
  for (int f : {b, b - 1, (b + 64) / 2, 65, 64, 33, 17, 1}) {
    if (f > b || f < 1) continue;
    rec = Rec();
    const CholArgs ca = chol_args(w, w.r1, w.dead, 1, 0, 0);
    CholArgs c = ca;
    c.Rinv = w.r1inv;
    if (gram_chol<T>(&ctx, nullptr, w, (T*)w.y, g.ldy, g.mm, f, w.gpart, c, nullptr, 0, nullptr, GRAM_LOOP_WG) != 0) {
      printf("block %d, %ld x %ld: refused\n", b, (long)m, (long)n);
      return false;
    }
    held("loop", f, g.mm, w.gpart, w.wfp);
  }
  // closing QRs of every rank class the capacity allows
  for (int64_t f : {(int64_t)1, (int64_t)20, (int64_t)64, (int64_t)65, (int64_t)101, (int64_t)128, (int64_t)129, (int64_t)195, g.r_cap}) {
    if (f > g.r_cap) continue;
    for (int64_t rows : {g.nn, g.mm, f}) {
      rec = Rec();
      CholArgs c = chol_args(w, w.rb1, w.deadbig, 1, 1, 1);
      c.Rinv = w.rb3;
      if (gram_chol<T>(&ctx, nullptr, w, (T*)w.cbuf, g.ldk, rows, (int)f, w.gbig, c) != 0) {
        printf("closing %ld of %ld x %ld: refused\n", (long)f, (long)m, (long)n);
        return false;
      }
      const bool shared = f <= 64 && w.gclose == w.gpart;
      held("closing", (int)f, rows, shared ? w.gpart : w.gbig, shared ? w.wfp : (void*)w.rb1);
    }
  }
  return ok;
}

int main() {
  eodabe_ctx ctx{};
  eodabe_default_opts(&ctx.o);
  int bad = 0, n = 0;
  for (int b = 1; b <= 128; b += b < 60 ? 13 : 1)
    for (int64_t m : {1, 17, 63, 64, 65, 300, 700, 959, 960, 961, 1300, 1700, 2000, 2433, 4096, 5001, 20000, 131072, 1048576})
      for (bool cplx : {false, true}) {
        ctx.cplx_pairs = cplx;
        for (int64_t nn : {60, 200}) {
          bad += !check<float>(ctx, b, m, nn);
          bad += !check<double>(ctx, b, m, nn);
          n += 2;
        }
      }
  printf("%d geometries, %d overrun\n", n, bad);
  return bad != 0;
}

// W = P^T P (upper half) of a double panel in the digit arithmetic of the int8
// kernels (i8_digits.hpp): the columns of every K slice cut into digits by
// their largest value, the digit products of one weight summed in int32, the
// weights up to `top` joined in double, the slices added in order.
// stdin: int32 K, N, kchunk, top (0: the kernels' own for Gram matrices), then
// K x N doubles; stdout: N x N doubles.  Built by the CPU tests with a plain
// C++ compiler.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <vector>

#include "i8_digits.hpp"

int main() {
  static_assert(cd::I8_NS * (1LL << 14) * cd::I8_KMAX < (1LL << 31), "int32 sums stay exact");
  int32_t h[4];
  if (std::fread(h, 4, 4, stdin) != 4) return 1;
  const int K = h[0], N = h[1], kc = h[2], top = h[3] ? h[3] : cd::I8_TOP_GRAM;
  if (K < 1 || N < 1 || kc < 1 || kc > cd::I8_KMAX) return 1;
  std::vector<double> P(static_cast<size_t>(K) * N), W(static_cast<size_t>(N) * N, 0.0);
  if (std::fread(P.data(), 8, P.size(), stdin) != P.size()) return 1;
  std::vector<int8_t> D(static_cast<size_t>(N) * cd::I8_NS * kc);
  std::vector<int> e(N);
  for (int k0 = 0; k0 < K; k0 += kc) {
    const int nk = K - k0 < kc ? K - k0 : kc;
    for (int j = 0; j < N; ++j) {
      double mx = 0.0;
      for (int k = 0; k < nk; ++k) mx = std::fmax(mx, std::fabs(P[static_cast<size_t>(k0 + k) * N + j]));
      e[j] = 0;
      if (mx > 0.0) std::frexp(mx, &e[j]);
      for (int k = 0; k < nk; ++k) {
        const double x = P[static_cast<size_t>(k0 + k) * N + j];
        const double y = std::fma(x, std::ldexp(1.0, 46 - e[j]), cd::I8_BIAS);
        uint64_t u;
        std::memcpy(&u, &y, 8);
        int64_t v = 0;
        for (int a = 0; a < cd::I8_NS; ++a) {
          const int8_t d = static_cast<int8_t>(((u >> (8 * (cd::I8_NS - 1 - a))) & 0xff) ^ 0x80);
          D[(static_cast<size_t>(j) * cd::I8_NS + a) * kc + k] = d;
          v = v * 256 + d;
        }
        if (static_cast<double>(v) != std::nearbyint(std::ldexp(x, 46 - e[j]))) return 2;   // the digits are x's
      }
    }
    for (int i = 0; i < N; ++i)
      for (int j = i; j < N; ++j) {
        double s = 0.0;
        for (int T = 0; T <= top; ++T) {
          int32_t acc = 0;
          for (int a = 0; a < cd::I8_NS; ++a) {
            const int b = T - a;
            if (b < 0 || b >= cd::I8_NS) continue;
            const int8_t* x = &D[(static_cast<size_t>(i) * cd::I8_NS + a) * kc];
            const int8_t* y = &D[(static_cast<size_t>(j) * cd::I8_NS + b) * kc];
            for (int k = 0; k < nk; ++k) acc += static_cast<int32_t>(x[k]) * y[k];
          }
          s = s * 256.0 + acc;
        }
        W[static_cast<size_t>(i) * N + j] += std::ldexp(s, 8 * (2 * (cd::I8_NS - 1) - top) + e[i] + e[j] - 92);
      }
  }
  return std::fwrite(W.data(), 8, W.size(), stdout) == W.size() ? 0 : 1;
}

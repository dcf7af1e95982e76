// Host-side launch planning of the C ABI: pure functions of the layer sizes,
// with no HIP dependency, so that the CPU tests compile and check them with
// a plain C++ compiler.
#pragma once

#include <vector>

namespace cd {

constexpr int MAXB = 32;          // layers per batched launch of the sync branch (one shape)
// Streaming-pass launches (any shapes): at most MAXS layers and 98304 blocks
// of 4096 elements (402.7M elements, 7.25 GB of M, X and bf16 G with the
// fused skip update).  The 1.3B-shaped set then splits into 3 x 32 layers
// (eight transformer blocks of 12288 blocks each per launch); launches of 48
// or 64 layers (600-800M elements) streamed 1.7% slower there.  The
// 160M-shaped set (48 layers, 20736 blocks) runs as one launch, 3.4% faster
// than two.
constexpr int MAXS = 48;
constexpr long long MAX_STREAM_BLOCKS = 98304;   // x 4096 elements
constexpr int NTHREADS = 256;     // threads per block for the streaming kernels
// Every block of a streaming pass covers FORM_CHUNK consecutive elements of
// one layer.
constexpr int FORM_CHUNK = NTHREADS * 4 * 4;   // 4096 elements

// Launches of the streaming passes (buffer formation, local update): layers
// in group order, each launch taking whole layers until it holds max_layers
// layers or one more layer would take it past max_blocks blocks of `chunk`
// elements.  A layer larger than max_blocks gets a launch of its own.
inline std::vector<std::vector<int>> plan_stream_batches(const std::vector<long long>& numel, int max_layers,
                                                         long long max_blocks, long long chunk) {
  std::vector<std::vector<int>> out;
  long long blocks = 0;
  for (int i = 0; i < static_cast<int>(numel.size()); ++i) {
    const long long nb = (numel[i] + chunk - 1) / chunk;
    if (out.empty() || static_cast<int>(out.back().size()) == max_layers || blocks + nb > max_blocks) {
      out.emplace_back();
      blocks = 0;
    }
    out.back().push_back(i);
    blocks += nb;
  }
  return out;
}

// K slices of a product of `tiles` workgroups on the int8 MFMA: at least two
// workgroups per CU (one is resident) over the `conc` units whose products run
// side by side, slices at least 256 deep, and no more of them than `most`, the
// fp64 kernel's partials of one layer, so that the same workspace holds them.
// Slices longer than kmax, the most rows that int32 sums hold exactly, are
// halved on, grid full or not (the caller sees whether the partials fit).
inline void plan_i8_slices(long long tiles, int K, int conc, int most, int kmax, int* splits, int* kchunk) {
  int s = 1;
  while (tiles * s * conc < 512 && K / (2 * s) >= 256 && 2 * s <= most) s *= 2;
  while ((K - 1) / s + 1 > kmax) s *= 2;
  *kchunk = ((K - 1) / s + 1 + 63) / 64 * 64;
  *splits = (K - 1) / *kchunk + 1;
}

// How many units' launches a unit's K slices are planned for, where units 0 ..
// nu-1 of work[u] values each run side by side on nside + 1 streams: all of
// them, but one where all the others together have less than 1/128 of the
// unit's work and are gone before its products.  4096 x 8192 with fp32 gradients
// beside 256 x 256, 128 x 128 and 100 x 100 (1/360), r = 96: sync step 769 us
// planned for four, 665 for one; 4096 x 16384 beside 64 x 64, 80 x 80 and 96 x
// 96, r = 64: 918 and 848, bf16 720 and 667.  But with others of 1/64 and more the fewer
// slices are the better: 4096 x 4096 beside 512 x 512, r = 256: 662 us planned
// for two, 691 for one, bf16 525 and 544.
inline int plan_conc(const long long* work, int nu, int u, int nside) {
  long long others = 0;
  for (int i = 0; i < nu; ++i) others += i == u ? 0 : work[i];
  return 128 * others < work[u] ? 1 : 1 + nside;
}

// Workgroups across the launch that normalises R (n rows) and cuts the planes of P
// (m rows) beside it: as many as the larger of the two has work for, `per` rows
// or quads each, at most `most`, the smaller one's last ones idle.  Planned for n
// alone, the 65536 rows of P of a 65536 x 256 layer at r = 192 went through 64
// workgroups: 266 us, 24 with 4096 (a launch of its own 52); r = 96 in bf16 162,
// now 10.
inline long long colnorm_blocks(long long n, long long m, long long per, long long most) {
  const long long b = ((n > m ? n : m) + per - 1) / per;
  return b < most ? b : most;
}

// Tiles of the pass that finds every row's and column's largest value
// (k_gemm_i8.hip): the narrowest of 256, 512 and 1024 columns that make at most 32
// across, and as many tiles down as make at most 2048 in all (eight per CU) and
// at most 256 partial maxima per column to join.  `room`: values that the
// partials may take, m per tile across (none for one tile: those are the maxima)
// and n per tile down; false when they cannot fit.
inline long long range_partials(int m, int n, int tr, int tc) {
  const long long across = (n - 1) / tc + 1, down = (m - 1) / tr + 1;
  return (across == 1 ? 0 : across * m) + down * n;
}
inline bool plan_range(int m, int n, long long room, int* tr, int* tc) {
  *tc = 256;
  while ((n - 1) / *tc + 1 > 32 && *tc < 1024) *tc *= 2;
  const long long across = (n - 1) / *tc + 1;
  *tr = 32;
  for (;;) {
    const long long down = (m - 1) / *tr + 1;
    const bool fits = range_partials(m, n, *tr, *tc) <= room;
    if (down == 1) return fits;
    if (fits && down <= 256 && across * down <= 2048) return true;
    *tr *= 2;
  }
}

}  // namespace cd

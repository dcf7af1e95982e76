// Prints launch plans of the C ABI, one line per launch or input line, for the
// sizes read from stdin.  No argument: the streaming passes' launches for layer
// shapes "m n", "<layers> <blocks>" each; "range": the tiles of the pass for
// row and column maxima for "m n room", "<ok> <tr> <tc> <partials>"; "colnorm":
// workgroups of the launch that normalises R and cuts P for "n m per most";
// "i8": K slices of an int8 product for "tiles K conc most kmax", "<slices>
// <rows>"; "conc": units that unit u of the given work is planned for, "nside u work ...".
// Built by the CPU tests with a plain C++ compiler against the library's
// planning header (it has no HIP dependency).
#include <cstdio>
#include <cstring>
#include <sstream>
#include <vector>

#include "plan.hpp"

int main(int argc, char** argv) {
  const char* mode = argc > 1 ? argv[1] : "";
  if (!std::strcmp(mode, "range")) {
    int m, n;
    long long room;
    while (std::scanf("%d %d %lld", &m, &n, &room) == 3) {
      int tr = 0, tc = 0;
      const bool ok = cd::plan_range(m, n, room, &tr, &tc);
      std::printf("%d %d %d %lld\n", ok ? 1 : 0, tr, tc, cd::range_partials(m, n, tr, tc));
    }
    return 0;
  }
  if (!std::strcmp(mode, "colnorm")) {
    long long n, m, per, most;
    while (std::scanf("%lld %lld %lld %lld", &n, &m, &per, &most) == 4)
      std::printf("%lld\n", cd::colnorm_blocks(n, m, per, most));
    return 0;
  }
  if (!std::strcmp(mode, "i8")) {
    long long tiles;
    int K, conc, most, kmax, splits, kchunk;
    while (std::scanf("%lld %d %d %d %d", &tiles, &K, &conc, &most, &kmax) == 5) {
      cd::plan_i8_slices(tiles, K, conc, most, kmax, &splits, &kchunk);
      std::printf("%d %d\n", splits, kchunk);
    }
    return 0;
  }
  if (!std::strcmp(mode, "conc")) {
    char line[4096];
    while (std::fgets(line, sizeof line, stdin)) {
      std::istringstream in(line);
      int nside, u;
      long long w;
      std::vector<long long> work;
      in >> nside >> u;
      while (in >> w) work.push_back(w);
      std::printf("%d\n", cd::plan_conc(work.data(), static_cast<int>(work.size()), u, nside));
    }
    return 0;
  }
  std::vector<long long> numel;
  long long m, n;
  while (std::scanf("%lld %lld", &m, &n) == 2) numel.push_back(m * n);
  const auto plan = cd::plan_stream_batches(numel, cd::MAXS, cd::MAX_STREAM_BLOCKS, cd::FORM_CHUNK);
  for (const auto& b : plan) {
    long long blocks = 0;
    for (int i : b) blocks += (numel[i] + cd::FORM_CHUNK - 1) / cd::FORM_CHUNK;
    std::printf("%zu %lld\n", b.size(), blocks);
  }
  return 0;
}

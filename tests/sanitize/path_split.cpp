// Which paths the lanes of a point take (walk.hpp: group_path), on the CPU under
// UndefinedBehaviorSanitizer: every path once for small numbers, and no path past the
// last one, however often a group asks, up to the largest number of paths per point.
// Prints "ok" or the first violation.
#include <cstdio>
#include <vector>

#include "../../paper_2305_04403_amd/csrc/internal.hpp"

static int bad(const char* what, int64_t N, int shift) {
  std::printf("%s: %lld paths, 2^%d lanes\n", what, (long long)N, shift);
  return 1;
}

template <bool POOL>
static int check(int32_t N, int shift) {
  const int gshift = POOL ? shift + 1 : (shift < 6 ? shift : 6), G = 1 << gshift, lpp = 1 << shift;
  const int points = POOL ? 2 : 1;
  const bool all = N < 100000;
  std::vector<int> seen(all ? (size_t)points * N : 0, 0);
  for (int first = 0; first < (POOL ? 1 : lpp); first += G) {
    // the group's last counter that names a path
    int64_t paths = 0;  // of the group
    if (POOL) paths = 2 * (int64_t)N;
    else
      for (int l = first; l < first + G; ++l) paths += l < N ? ((int64_t)N - l + lpp - 1) / lpp : 0;
    const int64_t from = all ? 0 : paths - 4 * G;
    int64_t found = from;
    // every lane asks once past the last path
    for (int64_t c = from; c < paths + 2 * G; ++c) {
      int pl = -1, k = -1;
      const bool is = wob::group_path<POOL>((uint32_t)c, N, G, gshift, lpp, first + (int)(c % G), pl, k);
      if (is) {
        if (k < 0 || k >= N || pl < 0 || pl >= points) return bad("a path that is none", N, shift);
        ++found;
        if (all) ++seen[(size_t)pl * N + k];
      } else if (c < paths - G) {
        return bad("a path left out", N, shift);
      }
    }
    if (found != paths) return bad("paths missing or repeated", N, shift);
  }
  for (const int s : seen)
    if (s != 1) return bad("a path not taken once", N, shift);
  return 0;
}

int main() {
  const int32_t most = INT32_MAX;
  for (const int32_t N : {1, 2, 3, 63, 64, 65, 700, 1023, 1025, 5000, 1 << 29, (1 << 30) - 1, 1 << 30, most - 1100,
                          most - 1000, most - 64, most - 1, most})
    for (int shift = 0; shift <= 10; ++shift) {
      if (check<false>(N, shift)) return 1;
      if (shift <= 5 && N < wob::kMaxPooled && check<true>(N, shift)) return 1;
    }
  // and a launch never pools more
  for (const int64_t points : {1, 1000, 100000000})
    for (const int32_t N : {(1 << 30) - 1, 1 << 30, most})
      if (!wobi::split_lanes<float, 3>(wob::F_SL, true, 17, points, N, 256).spread && N >= wob::kMaxPooled)
        return bad("pooled", N, 0);
  std::printf("ok\n");
}

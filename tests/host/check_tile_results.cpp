// Host-side check of the count of per-tile results that a plan's kernel choice
// goes by, against the generic kernel's tables. Prints "ok" or the violations.
#include <algorithm>
#include <cstdio>

#include "fsi_internal.h"

using namespace fsi;

int main() {
  int fails = 0;
  for (int d = 1; d <= 20; ++d)
    for (int l = 1; l <= std::min(d, 8); ++l)
      for (int b = 1; b <= std::min(d, kMaxTileBits); b += d > 14 ? 3 : 1) {
        ClassHost C;
        const std::string err = build_class(d, l, b, ALGO_FUSED, 0, 0, &C);
        if (!err.empty() || tile_results(d, l, b) != C.Ysize) {
          std::printf("d=%d l=%d b=%d: %lld, tables %d %s\n", d, l, b, (long long)tile_results(d, l, b),
                      C.Ysize, err.c_str());
          ++fails;
        }
      }
  if (!fails) std::printf("ok\n");
  return fails != 0;
}

// Asks the launch rules of csrc/dispatch.hpp: one query a line of standard
// input, one line of numbers each on standard output.
#include <cstdio>
#include <cstdlib>
#include <iostream>
#include <sstream>
#include <string>
#include <vector>

#include "dispatch.hpp"

int main() {
  std::string line;
  while (std::getline(std::cin, line)) {
    std::istringstream in(line);
    std::string what;
    in >> what;
    if (what == "bucket") {  // T E K, pair_pos over topk_ids
      int T, E, K, in_place;
      in >> T >> E >> K >> in_place;
      const auto l = eldr::bucket_launch(T, E, K, in_place);
      std::printf("%d %d %zu\n", l.large, l.wgs, l.lds);
    } else if (what == "gate") {  // T E H
      int T, E, H;
      in >> T >> E >> H;
      const auto l = eldr::gate_launch(T, E, H);
      std::printf("%d %d\n", l.tile, l.by_token);
    } else if (what == "slim") {  // mode format T K E rows kdim
      int mode, fmt, T, K, E, rows, kdim;
      in >> mode >> fmt >> T >> K >> E >> rows >> kdim;
      std::printf("%d\n", eldr::ffn_slim_pays(eldr::FfnMode(mode), eldr::WeightFmt(fmt), T, K, E, rows, kdim));
    } else if (what == "wide") {  // mode format T K E rows kdim: taken, row tiles, workgroups an XCD
      int mode, fmt, T, K, E, rows, kdim;
      in >> mode >> fmt >> T >> K >> E >> rows >> kdim;
      const int tiles = eldr::wide_tiles(eldr::FfnMode(mode), rows);
      std::printf("%d %d %d\n", eldr::ffn_wide_pays(eldr::FfnMode(mode), eldr::WeightFmt(fmt), T, K, E, rows, kdim),
                  tiles, eldr::wide_slots(tiles, T, K, E));
    } else if (what == "groups") {  // format row-tiles, then the union's buckets: cap, whole experts, groups
      int fmt, tiles, c, cap = 2 * eldr::kWideTokens, n = 0, t16 = 0, cmax = 0;
      std::vector<int> buckets;
      in >> fmt >> tiles;
      while (in >> c) buckets.push_back(c);
      in.clear();
      for (const int b : buckets) t16 += (b + 15) / 16, cmax = std::max(cmax, b);
      do {
        cap /= 2;
        n = 0;
        for (const int b : buckets) n += (b + cap - 1) / cap;
      } while (!eldr::wide_cap_fits(eldr::WeightFmt(fmt), cap, tiles, n, t16, cmax));
      std::printf("%d %d %d\n", cap, eldr::wide_whole(eldr::WeightFmt(fmt), cap, n, t16, cmax, (int)buckets.size()), n);
    } else {
      return 2;
    }
    if (!in) return 3;
  }
}

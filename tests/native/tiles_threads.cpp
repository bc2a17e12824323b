// Tile lists built with one, two and eight host threads must be the same lists.
// argv: pattern file (n, w, slot-major columns), halo depth, tile side.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "tiles.hpp"

int main(int argc, char** argv) {
  if (argc != 4) return 2;
  std::FILE* f = std::fopen(argv[1], "rb");
  int h[2];
  if (!f || std::fread(h, sizeof(int), 2, f) != 2) return 2;
  const int n = h[0], w = h[1], KM = std::atoi(argv[2]), side = std::atoi(argv[3]);
  std::vector<int> col((size_t)n * w);
  if (std::fread(col.data(), sizeof(int), col.size(), f) != col.size()) return 2;
  std::fclose(f);
  mgl::TilePlan a;
  if (!mgl::build_tiles(n, n, w, col.data(), KM, side, side, a, 4, 1)) return 1;
  if (!mgl::check_tiles(n, n, col.data(), a, 1)) return 1;
  for (int threads : {2, 8}) {
    mgl::TilePlan b;
    if (!mgl::build_tiles(n, n, w, col.data(), KM, side, side, b, 4, threads)) return 1;
    if (!mgl::check_tiles(n, n, col.data(), b, threads)) return 1;
    if (a.ntiles != b.ntiles || a.toff != b.toff || a.node != b.node || a.cnt != b.cnt || a.goff != b.goff ||
        a.lcol != b.lcol || a.maxcnt != b.maxcnt)
      return 1;
  }
  std::printf("ok %d\n", a.ntiles);
  return 0;
}

// Checks Tiling::tile_row (a multiplication) against the division that it
// stands for, for every tile of a plane and the tiles past its end that the
// last workgroup's wavefronts take (host code only).
#include <cstdio>

#include "kernels.hpp"

int main() {
  // tiles per row, tile rows: the shapes of ordinary cells, then planes near
  // the 2^25 tiles that the host accepts, with long rows
  const int shapes[][2] = {{1, 1},     {1, 7},      {2, 5},      {3, 3},       {4, 64},
                           {8, 8},     {13, 10},    {63, 65},    {1000, 7},    {2048, 2048},
                           {4975, 177}, {5843, 128}, {65536, 1},  {65537, 1},   {65537, 300},
                           {75000, 2}, {75000, 1},  {131072, 3}, {1000003, 5}, {33554431, 1}};
  long long wrong = 0;
  for (const auto& s : shapes) {
    lbm::Tiling t{};
    t.ntx = s[0];
    t.nty = s[1];
    t.by_ntx = lbm::Tiling::reciprocal(t.ntx);
    const int tiles = t.ntx * t.nty + 16;
    for (int i = 0; i < tiles; ++i)
      if (t.tile_row(i) != i / t.ntx && ++wrong <= 10)
        std::printf("%d x %d: tile %d gets row %d\n", s[0], s[1], i, t.tile_row(i));
  }
  std::printf("%lld wrong\n", wrong);
  return wrong != 0;
}

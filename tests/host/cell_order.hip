// The neighbour search's cell walks on the CPU: for every cell away from the
// faces, the short walk visits the rows of the general one, in its order.
// sim_dev.h's device functions are compiled for the host too, so that this
// runs (under the host's undefined-behaviour sanitizer) without a GPU.
#include <hip/hip_runtime.h>
#pragma push_macro("__device__")
#undef __device__
#define __device__ __attribute__((host)) __attribute__((device))
#include "sim_dev.h"
#pragma pop_macro("__device__")

#include <algorithm>
#include <cstdio>
#include <vector>

static int check(int nx, int ny, int nz) {
  RepDev R{};
  R.nc[0] = nx;
  R.nc[1] = ny;
  R.nc[2] = nz;
  for (int k = 0; k < 3; ++k) {
    R.cell_len[k] = R.inv_cell[k] = R.rc = 1.0;
    R.L[k] = R.nc[k];
    R.hL[k] = 0.5 * R.nc[k];
  }
  // as make_rep: bricks of 8^3 cells from 32 cells per axis on, else one
  const bool bricks = nx >= 32 && ny >= 32 && nz >= 32;
  R.brick = bricks ? 8 : std::max(nx, std::max(ny, nz));
  R.bshift = bricks ? 3 : 31;
  std::vector<int32_t> row((size_t)nx * ny * nz + 1);  // two rows in each cell
  for (size_t c = 0; c < row.size(); ++c) row[c] = 2 * (int32_t)c;
  int inside = 0;
  for (int z = 0; z < nz; ++z)
    for (int y = 0; y < ny; ++y)
      for (int x = 0; x < nx; ++x) {
        if (!cell_inside(R, x, y, z)) continue;
        ++inside;
        const int self = row[(size_t)cell_key(R, x, y, z)];
        std::vector<int> a, b;
        for_candidates_inside(R, row.data(), x, y, z, self, [&](int j) { a.push_back(j); });
        for_candidates(R, row.data(), 0.37, x + 0.5, y + 0.5, z + 0.5, self,
                       [&](int j) { b.push_back(j); });
        if (a != b || a.size() != 53) {
          std::printf("%d x %d x %d cells: the walks of cell (%d, %d, %d) differ\n", nx, ny, nz, x,
                      y, z);
          return -1;
        }
      }
  return inside;
}

int main() {
  const int sizes[][3] = {{3, 3, 3},   {4, 3, 5},    {7, 9, 8},    {31, 40, 33},
                          {32, 32, 32}, {33, 39, 40}, {41, 32, 47}};
  for (const auto& s : sizes) {
    const int n = check(s[0], s[1], s[2]);
    if (n != (s[0] - 2) * (s[1] - 2) * (s[2] - 2)) return 1;
    std::printf("%d x %d x %d: %d cells\n", s[0], s[1], s[2], n);
  }
  return 0;
}

// For each "nx ny nz cols" read: the groups of the x, y and z line launches, and whether the launches hold
// their threads (qlg_internal.hpp, host build).
#include <cstdio>

#include "qlg_internal.hpp"

int main() {
  long long nx, ny, nz;
  int cols;
  while (std::scanf("%lld %lld %lld %d", &nx, &ny, &nz, &cols) == 4) {
    int64_t g[3];
    qlg::line_launch_groups(nx, ny, nz, cols, g);
    const bool fits = qlg::launch_fits(g[0], qlg::kLanes * qlg::kLineTileRows) &&
                      qlg::launch_fits(g[1], qlg::kLanes * cols) && qlg::launch_fits(g[2], qlg::kLanes * cols);
    std::printf("%lld %lld %lld %d\n", (long long)g[0], (long long)g[1], (long long)g[2], fits ? 1 : 0);
  }
}

// sum_tiles_driver.cpp -- the tiles exec runs on, read from a host-only plan:
//   sum_tiles_driver <d> <N> <inner> <f64|f32> <inplace 0|1> <cubes> ...
// prints for every group of six arguments: the edge of the sum's own tiles (0:
// the plan's), its items, the orbits of a cube, its store mode, the plan's.
#include <cstdio>
#include <cstdlib>
#include <numeric>
#include <vector>

#include "spinsum_plan_host.h"

int main(int argc, char** argv) {
  for (int k = 1; k + 6 <= argc; k += 6) {
    const int d = std::atoi(argv[k]), n = std::atoi(argv[k + 1]), inner = std::atoi(argv[k + 2]);
    const spinsum_dtype dtype = argv[k + 3][1] == '6' ? SPINSUM_F64 : SPINSUM_F32;
    std::vector<int64_t> ext{std::atoll(argv[k + 5])};
    for (int m = 0; m < d; ++m) ext.push_back(n);
    if (inner > 1) ext.push_back(inner);
    std::vector<int> perms(2 * d);  // the identity and a cyclic shift
    for (int m = 0; m < d; ++m) {
      perms[m] = m;
      perms[d + m] = (m + 1) % d;
    }
    const int nterms = 2;
    const double alpha[2] = {1.0, -0.5};
    spinsum_plan_t p = nullptr;
    if (spinsum_plan(&p, (int)ext.size(), ext.data(), 1, d, 1, &nterms, perms.data(), alpha, dtype,
                     std::atoi(argv[k + 4]), SPINSUM_FLAG_FULL_GROUP | SPINSUM_FLAG_HOST_ONLY) != SPINSUM_OK)
      return 1;
    const spinsum::Tiling& T = p->x_own ? p->Tx : p->T;
    std::printf("%d %lld %d %d %d\n", p->x_own ? T.g.bl : 0, (long long)T.nitems, (int)T.orbits.size(),
                T.nts, p->T.nts);
    spinsum_plan_destroy(p);
  }
  return 0;
}

// Reads "n_particles n_mesh n_boxes patch_default free_bytes" lines and prints for each the wide
// and the compact layout of the patch deposit (particles a chunk, slot, bytes) and whether the
// wide one is taken; built and checked by tests/test_host_patch_layout.py.
#include <cstdio>
#include <iostream>

#include "../../paper_1209_0461_amd/csrc/patch_layout.hpp"

using namespace pmnu;

int main() {
  long long np = 0, free_bytes = 0;
  int n = 0, nbox = 0, by_default = 0;
  while (std::cin >> np >> n >> nbox >> by_default >> free_bytes) {
    for (int wide = 1; wide >= 0; --wide) {
      const PatchLayout p = patch_layout(np, n, wide != 0);
      std::printf("%d %d %lld ", p.particles, p.slot, static_cast<long long>(p.bytes(nbox)));
    }
    const long long bytes = patch_layout(np, n, true).bytes(nbox);
    std::printf("%d\n", patch_wide_fits(bytes, by_default != 0, free_bytes) ? 1 : 0);
  }
}

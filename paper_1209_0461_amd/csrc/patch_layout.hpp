// Chunks and patch slots of the patch deposit (deposit modes 6..9) and the memory that they take.
// Plain C++ with no HIP dependency.
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace pmnu {

// The LDS tile holds kPatchTile nodes (mode 6, three workgroups per CU) or kPatchCap (mode 7,
// two); a box beyond the tile is summed in several passes, up to the nodes of a patch's slot:
// kPatchSlot is a 16^3 block whose halo is six nodes a side (28^3), or 16 rows of 256 particles
// in C order (5 x 20 x 256).
constexpr int kPatchCH = 4096, kPatchCap = 9216, kPatchTile = 6144, kPatchNT = 512;
constexpr int kPatchSlot = 26624;

struct PatchLayout {
  int particles = kPatchCH;   // a chunk
  int slot = kPatchCap;       // nodes of a chunk's patch, at most the mesh
  int64_t chunks = 0;         // a box
  int64_t bytes(int nbox) const { return chunks * nbox * slot * 8; }
};

// Particles a chunk: a chunk of 4096 of sparse particles spans a box beyond the patch slot's 26624
// nodes as soon as it straddles two blocks of the curve, and goes through atomics. A step, us,
// with 4096 / 2048 / 1024: 256^3 mesh with 128^3 particles 644 / 425 / 421, 154^3 645 / 565 /
// 559, 180^3 693 / 575 / 554, 200^3 503 / 498 / 516, 220^3 748 / 651 / 656; 512^3 with 310^3
// 5126 / 4468 / 4193; 64 boxes of 64^3 with 40^3 587 / 392 / 375. Nearer a particle a node
// smaller chunks lose (more halo): 256^3 with 240^3 517 / 530, 256^3 526 / 540. So 1024 up to 3/8
// of a particle a node, 2048 up to 3/4.
inline int patch_chunk_particles(int64_t np, int n) {
  const int64_t m = static_cast<int64_t>(n) * n * n;
  return 8 * np <= 3 * m ? 1024 : 4 * np <= 3 * m ? 2048 : kPatchCH;
}

// A slot wide enough for displaced or sparse particles takes up to 78 bytes a mesh node, more
// than all else that a context holds (512^3: 7.0 GB at a particle a node, 10.5 GB at 3/8), so a
// context has wide slots only where memory is no question: up to kPatchSmall, or, if the patch
// deposit is its default, up to an eighth of the device's free memory. Otherwise it has the
// compact layout, chunks of 4096 with kPatchCap nodes each, 18 bytes a particle (512^3: 2.4 and
// 0.9 GB): the sums are the same integers, but wider boxes go through atomics.
constexpr int64_t kPatchSmall = int64_t{64} << 20;
inline PatchLayout patch_layout(int64_t np, int n, bool wide) {
  const int64_t m = static_cast<int64_t>(n) * n * n;
  PatchLayout p;
  p.particles = wide ? patch_chunk_particles(np, n) : kPatchCH;
  p.slot = static_cast<int>(std::min<int64_t>(wide ? kPatchSlot : kPatchCap, m));
  p.chunks = (np + p.particles - 1) / p.particles;
  return p;
}
inline bool patch_wide_fits(int64_t wide_bytes, bool patch_default, int64_t free_bytes) {
  return wide_bytes <= kPatchSmall || (patch_default && wide_bytes <= free_bytes / 8);
}

}  // namespace pmnu

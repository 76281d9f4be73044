// Cloud-in-cell mass assignment and force interpolation (gfx950).
//
// Mesh node (i, j, l) of box b sits at (i, j, l) L/N and lives at
// grid[b N^3 + (i N + j) N + l]; particle component 0 is axis i. Per axis the particle
// coordinate u = x N / L is split in FP64 into the lower node floor(u) (mod N) and the
// fraction d = u - floor(u): the lower node gets 1 - d and the upper node d. The eight
// corner weights are the products over the axes.
//
// The deposit accumulates in 64-bit fixed point (weight * 2^40, rounded, summed with
// integer atomics). Rounding O(1) cell sums to FP32 leaves a white-noise floor of ~6e-8
// per cell, which swamps the corner-of-the-cube modes whose power is ~1e-4 of the low-k
// power and so limits the binned spectrum there to ~1e-6; integer sums are exact, so the
// density is bitwise reproducible and only delta is rounded to FP32 (in the FFT's load).
// The interpolation weights are rounded to FP32.
//
// deposit_tiled_kernel privatises the accumulation in LDS: a workgroup takes CH
// consecutive particles, finds the bounding box of their cells (periodic, relative to the
// first particle's cell), and if the box plus its upper neighbours fits in CAP cells it
// sums the chunk's weights there with 64-bit LDS atomics and then adds every non-zero
// cell to HBM with one coalesced global atomic. Chunks that are not spatially compact
// (particles in arbitrary order) take the per-particle global-atomic path instead, so
// the result does not depend on the order; the speed does. Particles kept along a
// space-filling curve (as tree codes keep them) give compact chunks.
#include <type_traits>

#include "patch_device.hpp"

namespace pmnu {
namespace {

// Per axis: lower node (mod N) and the fraction beyond it, in FP64 (u = x N / L is exact
// for an FP32 coordinate times an FP64 inverse cell size up to the product's rounding).
// The node index comes from adding 1.5 * 2^52, which leaves floor(u) in two's complement
// in the low bits for |u| < 2^51; the mask keeps any index in range. (Beyond, the coordinate's own
// spacing is more than a box; every deposit and interpolation takes the node found here.)
// The product is rounded by itself in every deposit (no fused multiply-subtract for the fraction,
// which the compiler would form in some of them), so that all give the same fixed-point weights.
constexpr double kFloorMagic = 6755399441055744.0;     // 1.5 * 2^52
__device__ __forceinline__ void axis64(float x, double inv_cell, int nmask, int& i, double& d) {
#pragma clang fp contract(off)
  const double u = static_cast<double>(x) * inv_cell;
  const double f = floor(u);
  d = u - f;
  i = static_cast<int>(__double2loint(f + kFloorMagic)) & nmask;
}

// The product a b, 0 <= a b < 2^52, rounded to the nearest integer (ties to even): adding 2^52
// in one fused operation leaves it in the low mantissa bits; only the high word needs the
// exponent taken off.
__device__ __forceinline__ unsigned long long fix_product(double a, double b) {
  return static_cast<unsigned long long>(__double_as_longlong(fma(a, b, 4503599627370496.0))) -
         0x4330000000000000ull;
}

__device__ __forceinline__ bool finite3(float x, float y, float z) {
  return isfinite(x) && isfinite(y) && isfinite(z);
}

__global__ void fill_zero_kernel(float4* __restrict__ p, int64_t n4) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n4;
       i += stride)
    p[i] = make_float4(0.f, 0.f, 0.f, 0.f);
}

__global__ void fill_zero_tail_kernel(float* __restrict__ p, int64_t start, int64_t n) {
  const int64_t i = start + threadIdx.x;
  if (i < n) p[i] = 0.f;
}

// The eight fixed-point contributions of one particle, added straight to HBM.
__device__ __forceinline__ void deposit_global(unsigned long long* g, int n, const int (&i)[3],
                                               const double (&d)[3], int nmask) {
  const double wx[2] = {(1.0 - d[0]) * kFixScale, d[0] * kFixScale};
  const double wy[2] = {1.0 - d[1], d[1]};
  const int iz0 = i[2], iz1 = (i[2] + 1) & nmask;
#pragma unroll
  for (int cx = 0; cx < 2; ++cx) {
    const int ix = (i[0] + cx) & nmask;
#pragma unroll
    for (int cy = 0; cy < 2; ++cy) {
      const int iy = (i[1] + cy) & nmask;
      const double wxy = wx[cx] * wy[cy];
      const unsigned row = (static_cast<unsigned>(ix) * n + iy) * n;
      atomicAdd(g + row + iz0, fix_product(wxy, 1.0 - d[2]));
      atomicAdd(g + row + iz1, fix_product(wxy, d[2]));
    }
  }
}

__global__ __launch_bounds__(1024) void deposit_kernel(const float* __restrict__ pos,
                                                      unsigned long long* __restrict__ rho,
                                                      int64_t np, int nbox, int n,
                                                      double inv_cell, int* __restrict__ flags) {
  const int64_t total = np * nbox;
  const int64_t m = static_cast<int64_t>(n) * n * n;
  const int nmask = n - 1;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  bool bad = false;
  for (int64_t k = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; k < total;
       k += stride) {
    const float x = pos[3 * k], y = pos[3 * k + 1], z = pos[3 * k + 2];
    if (!finite3(x, y, z)) {
      bad = true;
      continue;
    }
    int i[3];
    double d[3];
    axis64(x, inv_cell, nmask, i[0], d[0]);
    axis64(y, inv_cell, nmask, i[1], d[1]);
    axis64(z, inv_cell, nmask, i[2], d[2]);
    deposit_global(rho + (k / np) * m, n, i, d, nmask);
  }
  if (bad) atomicOr(flags, 1);
}

__device__ __forceinline__ int wave_min(int v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = min(v, __shfl_xor(v, off, 64));
  return v;
}
__device__ __forceinline__ int wave_max(int v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = max(v, __shfl_xor(v, off, 64));
  return v;
}

// Largest / smallest of three, one instruction each; a NaN operand is passed over.
__device__ __forceinline__ float max3(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
__device__ __forceinline__ float min3(float a, float b, float c) {
  float r;
  asm("v_min3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
// max with the lane that a DPP control selects (lanes without one keep their value)
template <int CTRL>
__device__ __forceinline__ float max_dpp(float v) {
  const int i = __float_as_int(v);
  const float o = __int_as_float(__builtin_amdgcn_update_dpp(i, i, CTRL, 0xf, 0xf, false));
  return o > v ? o : v;
}
// over groups of 8 lanes (every lane gets it): pairs, quads, halves of a row
__device__ __forceinline__ float max8(float v) {
  return max_dpp<0x141>(max_dpp<0x4e>(max_dpp<0xb1>(v)));
}
// over the wave, in lane 63: rows of 16, then the two broadcasts of a row's last lane
__device__ __forceinline__ float wave_max63(float v) {
  return max_dpp<0x143>(max_dpp<0x142>(max_dpp<0x140>(max8(v))));
}

// PPT * NT consecutive particles held in registers and the periodic box of their lower nodes
// and upper neighbours: origin g0 (a mesh index) and extent ext <= n nodes per axis. full: an
// axis is covered whole (ext = n), where the upper neighbour of the last node is the first.
// ok: bit q set when particle tid + q NT exists and is finite.
template <int PPT>
struct Chunk {
  float p[PPT][3];
  unsigned ok;
  int g0[3], ext[3];
  bool full, bad;
};
struct ChunkRed {
  float m[7][16];   // per wave: -min and max of each axis, then a NaN mark
  int i[6][16];
};

// floor(x inv_cell) is monotone in x, so the box of a chunk that does not wrap around the
// mesh is that of its smallest and largest coordinates: three v_min3 / v_max3 pairs for two
// particles, where finding every particle's node took 12 instructions an axis. A chunk whose
// nodes span half the mesh or more (it may wrap) takes the nodes of every particle relative to
// the first one's instead; the two give the same box where both apply. One barrier, one more in
// the second form. A chunk with a coordinate that is not finite (which may hide others in the
// extremes) or beyond 2^30 cells has the whole mesh for its box.
template <int PPT, int NT>
__device__ __forceinline__ void chunk_box(Chunk<PPT>& c, const float* p, int cnt, double inv_cell,
                                          int nmask, ChunkRed& red) {
  constexpr int NW = NT / 64;
  static_assert(PPT % 2 == 0 && NW <= 16, "pairs of particles; at most 16 waves");
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, n = nmask + 1, half = n / 2;
#pragma unroll
  for (int q = 0; q < PPT; ++q) {
    const int j = tid + q * NT, js = j < cnt ? j : 0;   // the first one again beyond the end
    c.p[q][0] = p[3 * js];
    c.p[q][1] = p[3 * js + 1];
    c.p[q][2] = p[3 * js + 2];
  }
  float mn[3], mx[3], sum = 0.f;
#pragma unroll
  for (int a = 0; a < 3; ++a) mn[a] = mx[a] = c.p[0][a];
#pragma unroll
  for (int q = 0; q < PPT; q += 2) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      mn[a] = min3(mn[a], c.p[q][a], c.p[q + 1][a]);
      mx[a] = max3(mx[a], c.p[q][a], c.p[q + 1][a]);
      sum += c.p[q][a];
      sum += c.p[q + 1][a];
    }
  }
  // an infinity shows in mn or mx, a NaN in the sum
  const bool nan = __any(!(sum == sum));
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float lo = wave_max63(-mn[a]), hi = wave_max63(mx[a]);
    if (lane == 63) {
      red.m[a][wv] = lo;
      red.m[3 + a][wv] = hi;
    }
  }
  if (lane == 63) red.m[6][wv] = nan ? 1.f : 0.f;
  __syncthreads();
  // lanes 8 a .. 8 a + 7 of every wave reduce quantity a over the waves and turn it to a node
  const int a8 = min(lane >> 3, 6), w8 = lane & 7;
  float v = red.m[a8][NW >= 8 ? w8 : w8 & (NW - 1)];
  if constexpr (NW > 8) v = fmaxf(v, red.m[a8][w8 + 8]);
  v = max8(v);
  const double u = floor(static_cast<double>(a8 < 3 ? -v : v) * inv_cell);
  const int node = fabs(u) < 1073741824.0 ? static_cast<int>(u) : 0x7fffffff;
  bool near = __builtin_amdgcn_readlane(__float_as_int(v), 48) == 0, fast = true;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const int lo = __builtin_amdgcn_readlane(node, 8 * a);
    const int hi = __builtin_amdgcn_readlane(node, 24 + 8 * a);
    near = near && lo != 0x7fffffff && hi != 0x7fffffff;
    const int span = static_cast<int>(static_cast<unsigned>(hi) - static_cast<unsigned>(lo));
    fast = fast && span < half;
    c.g0[a] = lo & nmask;
    c.ext[a] = span + 2;                 // where it is taken at most half + 1 < n
  }
  c.ok = 0u;
#pragma unroll
  for (int q = 0; q < PPT; ++q) c.ok |= tid + q * NT < cnt ? 1u << q : 0u;
  c.bad = false;
  c.full = false;
  if (near && fast) return;
  if (!near) {
#pragma unroll
    for (int q = 0; q < PPT; ++q) {
      if (((c.ok >> q) & 1u) && !finite3(c.p[q][0], c.p[q][1], c.p[q][2])) {
        c.bad = true;
        c.ok &= ~(1u << q);
      }
    }
    c.full = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      c.g0[a] = 0;
      c.ext[a] = n;
    }
    return;
  }
  int r[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    double d;
    axis64(p[a], inv_cell, nmask, r[a], d);
  }
  int in[3] = {1 << 30, 1 << 30, 1 << 30}, ix[3] = {-(1 << 30), -(1 << 30), -(1 << 30)};
#pragma unroll
  for (int q = 0; q < PPT; ++q) {
    if (!((c.ok >> q) & 1u)) continue;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      int i;
      double d;
      axis64(c.p[q][a], inv_cell, nmask, i, d);
      const int rel = ((i - r[a] + half) & nmask) - half;
      in[a] = min(in[a], rel);
      ix[a] = max(ix[a], rel);
    }
  }
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    in[a] = wave_min(in[a]);
    ix[a] = wave_max(ix[a]);
    if (lane == 0) {
      red.i[a][wv] = in[a];
      red.i[3 + a][wv] = ix[a];
    }
  }
  __syncthreads();
#pragma unroll
  for (int a = 0; a < 3; ++a) {
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      in[a] = min(in[a], red.i[a][w]);
      ix[a] = max(ix[a], red.i[3 + a][w]);
    }
    in[a] = __builtin_amdgcn_readfirstlane(in[a]);
    ix[a] = __builtin_amdgcn_readfirstlane(ix[a]);
    c.ext[a] = ix[a] - in[a] + 2;
    c.g0[a] = (__builtin_amdgcn_readfirstlane(r[a]) + in[a]) & nmask;
    if (c.ext[a] >= n) {
      c.ext[a] = n;
      c.g0[a] = 0;
      c.full = true;
    }
  }
}

// A particle's lower node relative to the box origin and its fraction on one axis; mg is
// kFloorMagic - g0, so that the node comes out relative to g0 in one addition. That is axis64's node
// less g0 only for |u| < 2^51 or g0 = 0: chunk_box gives chunks that may hold more the origin 0.
__device__ __forceinline__ void box_axis(float x, double inv_cell, double mg, int nmask, int& t,
                                         double& d) {
#pragma clang fp contract(off)               // as axis64
  const double u = static_cast<double>(x) * inv_cell;
  const double f = floor(u);
  d = u - f;
  t = static_cast<int>(__double2loint(f + mg)) & nmask;
}

// Strides of an ey x ez plane in an LDS tile: padded so that a wave's 16-lane groups of
// particles along the curve (2 x 2 x 4 blocks of nodes for lattice-ordered chunks) hit 16
// distinct 8-byte bank slots, z stride = 4 (mod 8), y stride = 2 (mod 4), unless a tile of cap
// nodes would then hold fewer planes of an ex-plane box than it takes passes without. (256^3:
// unpadded strides cost the deposit 25 M bank-conflict cycles, 85 against 77 us.)
struct TileStrides {
  int sy, sz, npl;                     // npl: planes per pass, 0 if not one plane fits
};
__device__ __forceinline__ TileStrides tile_strides(int ex, int ey, int ez, int cap) {
  TileStrides t;
  t.sz = ez + ((12 - ez % 8) % 8);
  t.sy = ey + ((6 - ey % 4) % 4);
  const int plane = ey * ez;
  const int plain = plane > 0 && plane <= cap ? min(ex, cap / plane) : 0;
  const int padded = plane > 0 && t.sy * t.sz <= cap ? min(ex, cap / (t.sy * t.sz)) : 0;
  t.npl = padded;
  if (padded == 0 || (plain > padded && (ex + plain - 1) / plain < (ex + padded - 1) / padded)) {
    t.sy = ey;
    t.sz = ez;
    t.npl = plain;
  }
  return t;
}

// The chunk's fixed-point weights added to the planes [p0, p0 + npl) of its box in tile
// ([plane][sy][sz]) with 64-bit LDS atomics. WHOLE: the planes are the whole box and no axis
// wraps inside it; otherwise every plane is checked and the upper neighbours wrap.
template <bool WHOLE, int PPT>
__device__ __forceinline__ void add_chunk(const Chunk<PPT>& c, unsigned long long* tile,
                                          double inv_cell, int nmask, int sy, int sz, int p0,
                                          int npl) {
  const int ex = c.ext[0], ey = c.ext[1], ez = c.ext[2], plane = sy * sz;
  const double mx = kFloorMagic - c.g0[0], my = kFloorMagic - c.g0[1], mz = kFloorMagic - c.g0[2];
#pragma unroll
  for (int q = 0; q < PPT; ++q) {
    if (!((c.ok >> q) & 1u)) continue;
    int t[3];
    double d[3];
    box_axis(c.p[q][0], inv_cell, mx, nmask, t[0], d[0]);
    if constexpr (!WHOLE) {
      const int up = t[0] + 1 < ex ? t[0] + 1 : 0;
      if (static_cast<unsigned>(t[0] - p0) >= static_cast<unsigned>(npl) &&
          static_cast<unsigned>(up - p0) >= static_cast<unsigned>(npl))
        continue;
    }
    box_axis(c.p[q][1], inv_cell, my, nmask, t[1], d[1]);
    box_axis(c.p[q][2], inv_cell, mz, nmask, t[2], d[2]);
    const double wx[2] = {(1.0 - d[0]) * kFixScale, d[0] * kFixScale};
    const double wy[2] = {1.0 - d[1], d[1]};
    const double wz[2] = {1.0 - d[2], d[2]};
    if constexpr (WHOLE) {
      const int base = (t[0] * sy + t[1]) * sz + t[2];
#pragma unroll
      for (int cx = 0; cx < 2; ++cx) {
#pragma unroll
        for (int cy = 0; cy < 2; ++cy) {
          const double wxy = wx[cx] * wy[cy];
          const int o = base + cx * plane + cy * sz;
          atomicAdd(&tile[o], fix_product(wxy, wz[0]));
          atomicAdd(&tile[o + 1], fix_product(wxy, wz[1]));
        }
      }
    } else {
#pragma unroll
      for (int cx = 0; cx < 2; ++cx) {
        const int lx = (t[0] + cx < ex ? t[0] + cx : 0) - p0;
        if (static_cast<unsigned>(lx) >= static_cast<unsigned>(npl)) continue;
#pragma unroll
        for (int cy = 0; cy < 2; ++cy) {
          const double wxy = wx[cx] * wy[cy];
          const int row = (lx * sy + (t[1] + cy < ey ? t[1] + cy : 0)) * sz;
          atomicAdd(&tile[row + t[2]], fix_product(wxy, wz[0]));
          atomicAdd(&tile[row + (t[2] + 1 < ez ? t[2] + 1 : 0)], fix_product(wxy, wz[1]));
        }
      }
    }
  }
}

// v nodes of the tile cleared, 16 bytes a store (tile 16-byte aligned, its size even)
template <int NT>
__device__ __forceinline__ void clear_tile(unsigned long long* tile, int v) {
  ulonglong2* t2 = reinterpret_cast<ulonglong2*>(tile);
  for (int t = threadIdx.x; t < (v + 1) / 2; t += NT) t2[t] = make_ulonglong2(0ull, 0ull);
}

// the chunk's particles straight to the grid g with global atomics
template <int PPT>
__device__ __forceinline__ void add_chunk_global(const Chunk<PPT>& c, unsigned long long* g, int n,
                                                 double inv_cell, int nmask) {
#pragma unroll
  for (int q = 0; q < PPT; ++q) {
    if (!((c.ok >> q) & 1u)) continue;
    int i[3];
    double d[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) axis64(c.p[q][a], inv_cell, nmask, i[a], d[a]);
    deposit_global(g, n, i, d, nmask);
  }
}

// Walks the rows (tx, ty) of an ex x ey x ez box with the lanes of a wave spread over
// (row, z): lane l takes z = l mod ez of row l / ez, so short rows keep the wave busy
// without a division per node. Calls f(tx, ty, tz, linear index).
template <int NT = 256, typename F>
__device__ __forceinline__ void for_box_nodes(int ex, int ey, int ez, F f) {
  constexpr int NW = NT / 64;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (ez <= 64) {
    const int rpi = 64 / ez, dr = lane / ez, tz = lane - dr * ez;
    if (dr >= rpi) return;
    const int step = NW * rpi;
    int r = wv * rpi + dr;
    int tx = r / ey, ty = r - tx * ey;
    while (tx < ex) {
      f(tx, ty, tz, r * ez + tz);
      r += step;
      ty += step;
      while (ty >= ey) {
        ty -= ey;
        ++tx;
      }
    }
  } else {
    for (int r = wv; r < ex * ey; r += NW) {
      const int tx = r / ey, ty = r - tx * ey;
      for (int tz = lane; tz < ez; tz += 64) f(tx, ty, tz, r * ez + tz);
    }
  }
}

// Deposit with the accumulation privatised in LDS: a workgroup takes CH consecutive
// particles; if their box (upper neighbours included) fits in CAP nodes, it sums the
// chunk's fixed-point weights there with 64-bit LDS atomics and adds every non-zero node
// to HBM with one global atomic. Chunks that are not spatially compact (particles in
// arbitrary order) take the per-particle global-atomic path, so the result does not depend
// on the order; the speed does. Particles kept along a space-filling curve (as tree codes
// keep them) give compact chunks.
template <int CH, int CAP, int NT>
__global__ __launch_bounds__(NT) void deposit_tiled_kernel(const float* __restrict__ pos,
                                                           unsigned long long* __restrict__ rho,
                                                           int64_t np, int n, double inv_cell,
                                                           int* __restrict__ flags,
                                                           int64_t chunks_per_box) {
  constexpr int PPT = CH / NT;
  __shared__ alignas(16) unsigned long long tile[CAP];
  __shared__ ChunkRed red;
  const int64_t box = blockIdx.x / chunks_per_box;
  const int64_t c0 = (blockIdx.x - box * chunks_per_box) * CH;
  const int cnt = static_cast<int>(min(static_cast<int64_t>(CH), np - c0));
  const int nmask = n - 1;
  unsigned long long* g = rho + box * static_cast<int64_t>(n) * n * n;
  Chunk<PPT> c;
  chunk_box<PPT, NT>(c, pos + (box * np + c0) * 3, cnt, inv_cell, nmask, red);
  if (c.bad) atomicOr(flags, 1);
  const int ex = c.ext[0], ey = c.ext[1], ez = c.ext[2];
  const TileStrides ts = tile_strides(ex, ey, ez, CAP);
  if (ts.npl == ex) {
    clear_tile<NT>(tile, ex * ts.sy * ts.sz);
    __syncthreads();
    if (c.full) add_chunk<false>(c, tile, inv_cell, nmask, ts.sy, ts.sz, 0, ex);
    else add_chunk<true>(c, tile, inv_cell, nmask, ts.sy, ts.sz, 0, ex);
    __syncthreads();
    for_box_nodes<NT>(ex, ey, ez, [&](int tx, int ty, int tz, int) {
      const unsigned long long v = tile[(tx * ts.sy + ty) * ts.sz + tz];
      if (v == 0ull) return;
      const unsigned gx = (c.g0[0] + tx) & nmask, gy = (c.g0[1] + ty) & nmask,
                     gz = (c.g0[2] + tz) & nmask;
      atomicAdd(g + (gx * n + gy) * n + gz, v);
    });
  } else {
    add_chunk_global(c, g, n, inv_cell, nmask);
  }
}

// ---------------------------------------------------------------- patch deposit ----
// Deposit without global atomics. D1: each chunk sums its particles in an LDS tile as
// above, writes the tile to its own patch slot with plain stores and registers the patch in
// every coarse cell (CB^3 nodes) that the box overlaps; a registry entry carries everything
// D2 needs (chunk, box origin, extents). A box larger than the tile is summed in passes over
// as many of its x-planes as fit, the particles staying in registers, up to the slot's
// pcap nodes. D2: one workgroup per slab of a coarse cell adds up the registered patches
// in exact integers and writes delta = rho / rho_bar - 1 once, rounded to FP32. Weights that
// cannot go through a patch (a box too large: the whole chunk; a coarse cell whose list is
// full: the box's part in that cell) are added with global atomics to a side grid kept at
// zero, which D2 folds in (and clears) only when something was added to it: one atomic per
// non-zero node of a box up to kSideBoxMax nodes, eight per particle beyond.

__device__ __forceinline__ int ceil_div_pow2(int a, int lg) { return (a + (1 << lg) - 1) >> lg; }

// Bound at 256^3 (lattice order, boxes of about 17^3) by the bytes it moves, 365 MB: 77 us, 72 at
// the copy rate; 84 before the box was found from the extreme coordinates (42 M VALU
// instructions, now 34 M). Boxes beyond the tile, us before (per-particle atomics) and now:
// displacements of 1 and 2 cells 1555 -> 102 and 3600 -> 132, C order 803 -> 166.
template <int CH, int CAP, int NT>
__global__ __launch_bounds__(NT, CAP <= kPatchTile ? 6 : CAP <= kPatchCap ? 4 : 2) void deposit_patch_kernel(
    const float* __restrict__ pos, unsigned long long* __restrict__ patches, int pcap,
    int* __restrict__ reg_count, int4* __restrict__ reg_list,
    unsigned long long* __restrict__ rho_fb, int* __restrict__ n_fb,
    int64_t np, int n, double inv_cell, int* __restrict__ flags, int64_t chunks_per_box,
    int cb_lg) {
  constexpr int PPT = CH / NT, OVER = (kPatchRegMax + 31) / 32;
  constexpr int TILE = CAP + kPatchPad;
  __shared__ alignas(16) unsigned long long tile[TILE];
  __shared__ ChunkRed red;
  __shared__ unsigned s_over[OVER];    // bit t: registry cell t of the box was full
  const int tid = threadIdx.x;
  const int64_t chunk = blockIdx.x;
  // grid sizes stay below 2^31 blocks: a 32-bit division suffices
  const int64_t box = static_cast<uint32_t>(chunk) / static_cast<uint32_t>(chunks_per_box);
  const int64_t c0 = (chunk - box * chunks_per_box) * CH;
  const int cnt = static_cast<int>(min(static_cast<int64_t>(CH), np - c0));
  const int nmask = n - 1;
  const int64_t m = static_cast<int64_t>(n) * n * n;
  unsigned long long* fb = rho_fb + box * m;
  if (tid < OVER) s_over[tid] = 0u;
  Chunk<PPT> c;
  chunk_box<PPT, NT>(c, pos + (box * np + c0) * 3, cnt, inv_cell, nmask, red);
  if (c.bad) atomicOr(flags, 1);
  const int ex = c.ext[0], ey = c.ext[1], ez = c.ext[2];
  const int plane = ey * ez, vol = ex * plane;         // < 2^28
  const int gx0 = c.g0[0], gy0 = c.g0[1], gz0 = c.g0[2];
  const TileStrides ts = tile_strides(ex, ey, ez, TILE);
  const int sy = ts.sy, sz = ts.sz, npl = ts.npl;      // npl: planes per pass
  const int nc = n >> cb_lg, cbm = (1 << cb_lg) - 1;
  const int rx = min(nc, ceil_div_pow2((gx0 & cbm) + ex, cb_lg));
  const int ry = min(nc, ceil_div_pow2((gy0 & cbm) + ey, cb_lg));
  const int rz = min(nc, ceil_div_pow2((gz0 & cbm) + ez, cb_lg));
  const bool patch = npl > 0 && vol <= pcap && rx * ry * rz <= kPatchRegMax;
  bool side = true;                    // something of the chunk goes to the side grid
  if (patch || (npl > 0 && vol <= kSideBoxMax)) {
    if (patch) {
      // register the patch in the coarse cells its box overlaps (origin and extents <= 512)
      const int64_t cells = static_cast<int64_t>(nc) * nc * nc;
      const int fx = gx0 >> cb_lg, fy = gy0 >> cb_lg, fz = gz0 >> cb_lg;
      const int4 entry = make_int4(static_cast<int>(chunk), gx0 | (gy0 << 10) | (gz0 << 20),
                                   ex | (ey << 10) | (ez << 20), 0);
      for (int t = tid; t < rx * ry * rz; t += NT) {
        const int iz = t % rz, ixy = t / rz, iy = ixy % ry, ix = ixy / ry;
        const int64_t cell = box * cells +
                             ((static_cast<int64_t>((fx + ix) % nc) * nc + (fy + iy) % nc) * nc +
                              (fz + iz) % nc);
        const int slot = atomicAdd(reg_count + cell, 1);
        if (slot < kPatchList)
          reg_list[cell * kPatchList + slot] = entry;
        else
          atomicOr(&s_over[t >> 5], 1u << (t & 31));   // t < kPatchRegMax
      }
    }
    unsigned long long* pat = patches + chunk * pcap;
    for (int p0 = 0; p0 < ex; p0 += npl) {
      const int npp = min(npl, ex - p0);
      clear_tile<NT>(tile, npp * sy * sz);
      __syncthreads();
      // the positions made opaque in every pass: the particles' nodes and weights are formed
      // again instead of being kept over the passes (which took 254 registers)
#pragma unroll
      for (int q = 0; q < PPT; ++q)
        asm volatile("" : "+v"(c.p[q][0]), "+v"(c.p[q][1]), "+v"(c.p[q][2]));
      if (npl == ex && !c.full) add_chunk<true>(c, tile, inv_cell, nmask, sy, sz, 0, ex);
      else add_chunk<false>(c, tile, inv_cell, nmask, sy, sz, p0, npp);
      __syncthreads();
      unsigned over = 0u;
      if (patch) {
        // the patch (the box unpadded): consecutive lanes at consecutive nodes, four nodes per
        // thread per round with their LDS reads ahead of the stores. Node li of the pass lies
        // in row li / ez and plane li / ez / ey; the FP32 quotients are exact: (li + 1/2) / e
        // lies at least 1 / (2e) from an integer, and its relative error of 2^-22 at most moves
        // it by less for li < 2^20.
        static_assert(TILE < (1 << 20), "nodes of a pass");
        unsigned long long* dst = pat + p0 * plane;
        const int tv = npp * plane, pad_z = sz - ez, pad_y = (sy - ey) * sz;
        const float inv_ez = 1.0f / static_cast<float>(ez), inv_ey = 1.0f / static_cast<float>(ey);
        for (int l0 = tid; l0 < tv; l0 += 4 * NT) {
          unsigned long long val[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int li = l0 + u * NT;
            const int row = static_cast<int>(fmaf(static_cast<float>(li), inv_ez, 0.5f * inv_ez));
            const int pl = static_cast<int>(fmaf(static_cast<float>(row), inv_ey, 0.5f * inv_ey));
            val[u] = li < tv ? tile[li + row * pad_z + pl * pad_y] : 0ull;
          }
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (l0 + u * NT < tv) dst[l0 + u * NT] = val[u];
        }
#pragma unroll
        for (int w = 0; w < OVER; ++w) over |= s_over[w];
        side = over != 0u;
      }
      if (side) {
        // to the side grid: the whole box, or (a patch) its part in the cells whose list was full
        for_box_nodes<NT>(npp, ey, ez, [&](int lx, int ty, int tz, int) {
          const int tx = p0 + lx;
          if (patch) {
            int ix = ((gx0 & cbm) + tx) >> cb_lg, iy = ((gy0 & cbm) + ty) >> cb_lg,
                iz = ((gz0 & cbm) + tz) >> cb_lg;
            ix -= ix >= nc ? nc : 0;                // a box as wide as the mesh wraps onto fx
            iy -= iy >= nc ? nc : 0;
            iz -= iz >= nc ? nc : 0;
            const int t = (ix * ry + iy) * rz + iz;
            if (!((s_over[t >> 5] >> (t & 31)) & 1u)) return;
          }
          const unsigned long long v = tile[(lx * sy + ty) * sz + tz];
          if (v == 0ull) return;
          const unsigned gx = (gx0 + tx) & nmask, gy = (gy0 + ty) & nmask, gz = (gz0 + tz) & nmask;
          atomicAdd(fb + (gx * n + gy) * n + gz, v);
        });
      }
      if (p0 + npl < ex) __syncthreads();           // the tile is read before the next pass clears it
    }
  } else {
    add_chunk_global(c, fb, n, inv_cell, nmask);
  }
  if (side && tid == 0) atomicAdd(n_fb, 1);
}

// D2: one workgroup of 256 threads per (slab of XD x-planes of a coarse cell, box), CB =
// 1 << cb_lg <= 16, XD <= CB (halving the slab halves the LDS copy and doubles the
// workgroups, which hides more of the load latency). A cell is mostly covered by one patch
// (the chunk whose block it is) and touched by a few others in thin layers (their halos).
// The largest overlap goes through registers: thread (iy, iz) owns the slab's column
// x = 0..XD-1 and loads it from that patch. Every other overlap is cut into boxes (up to
// two periodic pieces per axis), which wave 0 lists once in LDS with their item offsets,
// sizes and source and destination bases; all threads then stride over the flat item list,
// find an item's box by bisection and add the node into an LDS copy of the slab with
// 64-bit LDS atomics. Every thread issues all of its loads (its column and up to kBatch
// list items) before it uses any, so each workgroup waits on few load latencies. The sums
// are exact integers.
template <int XD>
__global__ __launch_bounds__(256) void patch_reduce_kernel(
    const unsigned long long* __restrict__ patches, int pcap, const int* __restrict__ reg_count,
    const int4* __restrict__ reg_list, unsigned long long* __restrict__ rho_fb,
    const int* __restrict__ n_fb, float* __restrict__ delta, int n, int cb_lg, double scale) {
  constexpr int CBM = 16, kBatch = 8, kPieces = kPatchList * 8;
  const int tid = threadIdx.x;
  const int cb = 1 << cb_lg, nc = n >> cb_lg;
  const int slabs = cb / XD;
  const int64_t cells = static_cast<int64_t>(nc) * nc * nc;
  const int64_t box = blockIdx.y;
  // workgroups go to the 8 XCDs in turn: each XCD takes a contiguous run of slabs instead,
  // so that neighbouring cells (which read the same patches' halo lines) share an L2; a
  // ragged tail keeps its own index
  const int nb = gridDim.x, per = nb / 8;
  const int bid = static_cast<int>(blockIdx.x) < per * 8
                      ? static_cast<int>(blockIdx.x % 8) * per + static_cast<int>(blockIdx.x / 8)
                      : static_cast<int>(blockIdx.x);
  const int cix = bid / slabs;
  const int64_t cell = box * cells + cix;
  const int ccz = (cix % nc) << cb_lg, ccy = ((cix / nc) % nc) << cb_lg,
            ccx = ((cix / (nc * nc)) << cb_lg) + (bid - cix * slabs) * XD;  // slab's x0
  const int iy = tid >> cb_lg, iz = tid & (cb - 1);
  const bool on = tid < cb * cb;
  const int vol_cell = XD * cb * cb;
  __shared__ unsigned long long s_acc[XD * CBM * CBM];    // [x][y][z] of the slab
  // the piece list: item offset (INT_MAX past the end), Lz | Ly << 8, source base
  // (patch element of the piece's first node), strides ez | (ey ez) << 10, LDS base
  __shared__ int p_off[kPieces + 1];
  __shared__ int p_dim[kPieces];
  __shared__ long long p_src[kPieces];
  __shared__ int p_str[kPieces];
  __shared__ int p_dst[kPieces];
  __shared__ int4 s_home;                  // home patch: chunk, origin, extents; chunk < 0: none
  __shared__ int s_total;                  // items in the piece list
  for (int i = tid; i < vol_cell; i += 256) s_acc[i] = 0ull;
  if (tid < 64) {
    // wave 0: the cell's patches (list row and count fetched together), their overlap
    // pieces, the home patch and the piece list of the others
    const int cnt_raw = reg_count[cell];
    const int4 listed =
        tid < kPatchList ? reg_list[cell * kPatchList + tid] : make_int4(-1, 0, 0, 0);
    const bool mine = tid < min(cnt_raw, kPatchList);
    const int gx = listed.y & 1023, gy = (listed.y >> 10) & 1023, gz = listed.y >> 20;
    const int ex = listed.z & 1023, ey = (listed.z >> 10) & 1023, ez = listed.z >> 20;
    Pieces px, py, pz;
    px.cnt = py.cnt = pz.cnt = 0;
    int vol = -1;
    if (mine) {
      px = overlap(gx, ex, ccx, XD, n);
      py = overlap(gy, ey, ccy, cb, n);
      pz = overlap(gz, ez, ccz, cb, n);
      int lx = 0, ly = 0, lz = 0;
#pragma unroll
      for (int q = 0; q < 2; ++q) {           // constant bounds: no indexed scratch
        lx += q < px.cnt ? px.len[q] : 0;
        ly += q < py.cnt ? py.len[q] : 0;
        lz += q < pz.cnt ? pz.len[q] : 0;
      }
      vol = lx * ly * lz;
    }
    // home: the largest volume, ties to the lowest index
    int key = vol > 0 ? (vol << 6) | (63 - tid) : -1;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) key = max(key, __shfl_xor(key, off, 64));
    const int home = key >= 0 ? 63 - (key & 63) : -1;
    if (tid == 0) s_home = make_int4(-1, 0, 0, 0);
    if (tid == home) s_home = listed;
    // exclusive prefixes of the others' piece counts and volumes
    const bool other = vol > 0 && tid != home;
    const int np_mine = other ? px.cnt * py.cnt * pz.cnt : 0;
    int inc_p = np_mine, inc_v = other ? vol : 0;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int tp = __shfl_up(inc_p, off, 64), tv = __shfl_up(inc_v, off, 64);
      if (tid >= off) {
        inc_p += tp;
        inc_v += tv;
      }
    }
    const int n_pieces = __shfl(inc_p, 63, 64);
    if (tid == 63) s_total = inc_v;
    int slot = inc_p - np_mine;
    int item = inc_v - (other ? vol : 0);
    if (other) {
      const long long src0 = static_cast<long long>(listed.x) * pcap;
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            if (a >= px.cnt || b >= py.cnt || c >= pz.cnt) continue;
            const int Lx = px.len[a], Ly = py.len[b], Lz = pz.len[c];
            p_off[slot] = item;
            p_dim[slot] = Lz | (Ly << 8);
            p_src[slot] = src0 + (px.pl[a] * ey + py.pl[b]) * ez + pz.pl[c];
            p_str[slot] = ez | ((ey * ez) << 10);
            p_dst[slot] = (px.cl[a] * cb + py.cl[b]) * cb + pz.cl[c];
            item += Lx * Ly * Lz;
            ++slot;
          }
    }
    for (int i = n_pieces + tid; i <= kPieces; i += 64) p_off[i] = 0x7fffffff;
  }
  __syncthreads();
  const int total = s_total;
  // the home patch's column loads go out first
  unsigned long long acc[XD];
#pragma unroll
  for (int x = 0; x < XD; ++x) acc[x] = 0ull;
  const int4 hl = s_home;
  if (hl.x >= 0) {
    const int hx = hl.y & 1023, hy = (hl.y >> 10) & 1023, hz = hl.y >> 20;
    const int ex = hl.z & 1023, ey = (hl.z >> 10) & 1023, ez = hl.z >> 20;
    const Pieces px = overlap(hx, ex, ccx, XD, n), py = overlap(hy, ey, ccy, cb, n),
                 pz = overlap(hz, ez, ccz, cb, n);
    int ly = -1, lz = -1;                       // this thread's row (y, z) inside the patch
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (q < py.cnt && iy >= py.cl[q] && iy < py.cl[q] + py.len[q]) ly = py.pl[q] + iy - py.cl[q];
      if (q < pz.cnt && iz >= pz.cl[q] && iz < pz.cl[q] + pz.len[q]) lz = pz.pl[q] + iz - pz.cl[q];
    }
    const bool lane_in = on && ly >= 0 && lz >= 0;
    const unsigned long long* row =
        patches + static_cast<int64_t>(hl.x) * pcap + (lane_in ? ly * ez + lz : 0);
    const int xs = ey * ez;                     // patch stride along x
#pragma unroll
    for (int x = 0; x < XD; ++x) {
      int lx = -1;                              // patch-local x of slab-local x (uniform)
      if (px.cnt > 0 && x >= px.cl[0] && x < px.cl[0] + px.len[0]) lx = px.pl[0] + x - px.cl[0];
      if (px.cnt > 1 && x >= px.cl[1] && x < px.cl[1] + px.len[1]) lx = px.pl[1] + x - px.cl[1];
      acc[x] = (lx >= 0 && lane_in) ? row[lx * xs] : 0ull;
    }
  }
  // the other overlaps: kBatch items per thread per round, all loads before the adds
  for (int base = 0; base < total; base += kBatch * 256) {
    unsigned long long v[kBatch];
    int li[kBatch];
#pragma unroll
    for (int r = 0; r < kBatch; ++r) {
      const int i = base + r * 256 + tid;
      li[r] = -1;
      v[r] = 0ull;
      if (i < total) {
        int e = 0;                              // the piece: last offset <= i
#pragma unroll
        for (int step = kPieces / 2; step > 0; step >>= 1)
          if (p_off[e + step] <= i) e += step;
        const int rem = i - p_off[e];
        const int dim = p_dim[e], str = p_str[e];
        const int Lz = dim & 255, Ly = dim >> 8;
        // exact: rem < 4096 and the divisors are at most 16
        const int t = static_cast<int>((rem + 0.5f) * (1.0f / Lz));
        const int z = rem - t * Lz;
        const int x = static_cast<int>((t + 0.5f) * (1.0f / Ly));
        const int y = t - x * Ly;
        v[r] = patches[p_src[e] + x * (str >> 10) + y * (str & 1023) + z];
        li[r] = p_dst[e] + (x * cb + y) * cb + z;
      }
    }
#pragma unroll
    for (int r = 0; r < kBatch; ++r)
      if (li[r] >= 0) atomicAdd(&s_acc[li[r]], v[r]);
  }
  __syncthreads();
  const bool fold = *n_fb > 0;
  if (on) {
    const int64_t m = static_cast<int64_t>(n) * n * n;
    const int64_t col = box * m + static_cast<int64_t>(ccy + iy) * n + ccz + iz;
#pragma unroll
    for (int x = 0; x < XD; ++x) {
      const int64_t node = col + static_cast<int64_t>(ccx + x) * n * n;
      unsigned long long val = acc[x] + s_acc[(x * cb + iy) * cb + iz];
      if (fold) {
        val += rho_fb[node];
        rho_fb[node] = 0ull;
      }
      // exact integer sum, rounded once: delta = rho / rho_bar - 1
      delta[node] = static_cast<float>(static_cast<double>(val) * scale - 1.0);
    }
  }
  // reg_count is cleared by the next kernel (the first forward FFT pass): the other slabs of
  // this cell may still read it
}

__global__ void delta_to_density_kernel(const float* __restrict__ delta, float* __restrict__ out,
                                        int64_t n, float rho_bar) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
       i += stride)
    out[i] = (delta[i] + 1.0f) * rho_bar;
}

// FP32 corner weights of one particle (the fraction rounded once to FP32).
struct Corner {
  int i[3];
  float w[3][2];
};

__device__ __forceinline__ void corner_of(float x, float y, float z, double inv_cell, int nmask,
                                          Corner& c) {
  double d;
  axis64(x, inv_cell, nmask, c.i[0], d);
  c.w[0][1] = static_cast<float>(d);
  c.w[0][0] = 1.0f - c.w[0][1];
  axis64(y, inv_cell, nmask, c.i[1], d);
  c.w[1][1] = static_cast<float>(d);
  c.w[1][0] = 1.0f - c.w[1][1];
  axis64(z, inv_cell, nmask, c.i[2], d);
  c.w[2][1] = static_cast<float>(d);
  c.w[2][0] = 1.0f - c.w[2][1];
}

// Gather of the interleaved acceleration grid ([x][y][z][3] per box) at the 8 corners.
__device__ __forceinline__ void gather_global(const float* g, int n, int nmask, const Corner& c,
                                              float& a0, float& a1, float& a2) {
  const int iz0 = c.i[2], iz1 = (c.i[2] + 1) & nmask;
#pragma unroll
  for (int cx = 0; cx < 2; ++cx) {
    const int ix = (c.i[0] + cx) & nmask;
#pragma unroll
    for (int cy = 0; cy < 2; ++cy) {
      const int iy = (c.i[1] + cy) & nmask;
      const float wxy = c.w[0][cx] * c.w[1][cy];
      const unsigned row = (static_cast<unsigned>(ix) * n + iy) * n;
#pragma unroll
      for (int cz = 0; cz < 2; ++cz) {
        const float* v = g + 3 * (row + (cz ? iz1 : iz0));
        const float w = wxy * c.w[2][cz];
        a0 += w * v[0];
        a1 += w * v[1];
        a2 += w * v[2];
      }
    }
  }
}

// Workgroups are handed to the XCDs in turn; remapping the block index gives each XCD one
// contiguous run of chunks, so neighbouring chunks (which share grid lines) hit the same L2.
__device__ __forceinline__ int64_t xcd_chunk(int64_t b, int64_t nblocks) {
  constexpr int kXcd = 8;
  const int64_t per = (nblocks + kXcd - 1) / kXcd;
  return (b % kXcd) * per + b / kXcd;
}

// Direct interpolation: PPT particles per thread (strided by the block size inside a
// contiguous chunk), gathering from HBM through the caches.
// The end of the interpolation for particle gi (global index) at position (x, y, z): store
// the acceleration, or apply the leapfrog of pm_nu_advance (u += K acc; x += D u).
template <bool LEAP>
__device__ __forceinline__ void finish_particle(const Leap& lp, float* __restrict__ acc,
                                                int64_t gi, float x, float y, float z,
                                                float a0, float a1, float a2, float kk,
                                                float dd) {
  if (!LEAP || lp.store_acc) {
    acc[3 * gi] = a0;
    acc[3 * gi + 1] = a1;
    acc[3 * gi + 2] = a2;
  }
  if (!LEAP) return;
  float* u = lp.vel + 3 * gi;
  const float u0 = u[0] + kk * a0, u1 = u[1] + kk * a1, u2 = u[2] + kk * a2;
  u[0] = u0;
  u[1] = u1;
  u[2] = u2;
  if (lp.pos) {
    float* px = lp.pos + 3 * gi;
    px[0] = wrap_box(x + dd * u0, lp.box);
    px[1] = wrap_box(y + dd * u1, lp.box);
    px[2] = wrap_box(z + dd * u2, lp.box);
  }
}

template <int PPT, bool LEAP>
__global__ __launch_bounds__(256) void interp_kernel(const float* pos,
                                                     const float* __restrict__ force,
                                                     float* __restrict__ acc, int64_t np, int n,
                                                     double inv_cell, int64_t chunks_per_box,
                                                     int64_t nchunks, Leap lp) {
  constexpr int NT = 256, CH = NT * PPT;
  const int64_t chunk = xcd_chunk(blockIdx.x, gridDim.x);
  if (chunk >= nchunks) return;
  // grid sizes stay below 2^31 blocks: a 32-bit division suffices
  const int64_t box = static_cast<uint32_t>(chunk) / static_cast<uint32_t>(chunks_per_box);
  const int64_t c0 = (chunk - box * chunks_per_box) * CH;
  const int cnt = static_cast<int>(min(static_cast<int64_t>(CH), np - c0));
  const float* p = pos + (box * np + c0) * 3;
  const float* g = force + box * static_cast<int64_t>(n) * n * n * 3;
  const int nmask = n - 1;
  float kk = 0.f, dd = 0.f;
  if (LEAP) {
    kk = static_cast<float>(lp.kd[2 * box]);
    dd = static_cast<float>(lp.kd[2 * box + 1]);
  }
#pragma unroll
  for (int q = 0; q < PPT; ++q) {
    const int j = threadIdx.x + q * NT;
    if (j >= cnt) break;
    const float x = p[3 * j], y = p[3 * j + 1], z = p[3 * j + 2];
    float a0 = 0.f, a1 = 0.f, a2 = 0.f;
    if (finite3(x, y, z)) {
      Corner c;
      corner_of(x, y, z, inv_cell, nmask, c);
      gather_global(g, n, nmask, c, a0, a1, a2);
    }
    finish_particle<LEAP>(lp, acc, box * np + c0 + j, x, y, z, a0, a1, a2, kk, dd);
  }
}

// Interpolation with the chunk's box of the acceleration grid staged in LDS (rows of
// 3 * ez consecutive floats); chunks whose box does not fit gather straight from HBM.
template <int CH, int CAP, bool LEAP>
__global__ __launch_bounds__(256, CH <= 1024 ? 6 : 1) void interp_tiled_kernel(const float* pos,
                                                           const float* __restrict__ force,
                                                           float* __restrict__ acc, int64_t np,
                                                           int n, double inv_cell,
                                                           int64_t chunks_per_box,
                                                           int64_t nchunks, Leap lp) {
  constexpr int NT = 256, PPT = CH / NT;
  __shared__ float tile[CAP * 3];
  __shared__ ChunkRed red;
  const int tid = threadIdx.x;
  const int64_t chunk = xcd_chunk(blockIdx.x, gridDim.x);
  if (chunk >= nchunks) return;
  // grid sizes stay below 2^31 blocks: a 32-bit division suffices
  const int64_t box = static_cast<uint32_t>(chunk) / static_cast<uint32_t>(chunks_per_box);
  const int64_t c0 = (chunk - box * chunks_per_box) * CH;
  const int cnt = static_cast<int>(min(static_cast<int64_t>(CH), np - c0));
  const int nmask = n - 1;
  const float* g = force + box * static_cast<int64_t>(n) * n * n * 3;
  float kk = 0.f, dd = 0.f;
  if (LEAP) {
    kk = static_cast<float>(lp.kd[2 * box]);
    dd = static_cast<float>(lp.kd[2 * box + 1]);
  }
  Chunk<PPT> c;
  chunk_box<PPT, 256>(c, pos + (box * np + c0) * 3, cnt, inv_cell, nmask, red);
  const int ex = c.ext[0], ey = c.ext[1], ez = c.ext[2];
  const int vol = ex * ey * ez;
  const bool use_tile = vol <= CAP && !c.full;
  // every particle's node in the box (three 10-bit fields) and fraction
  int rel[PPT];
  float fr[PPT][3];
#pragma unroll
  for (int q = 0; q < PPT; ++q) {
    rel[q] = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      int t;
      double d;
      box_axis(c.p[q][a], inv_cell, kFloorMagic - c.g0[a], nmask, t, d);
      rel[q] |= t << (10 * a);
      fr[q][a] = static_cast<float>(d);
    }
  }
  if (use_tile) {
    const int gx0 = c.g0[0], gy0 = c.g0[1], gz0 = c.g0[2];
    constexpr int RMAX = 32;                 // rows per wave held in registers
    const int rows = ex * ey;
    if (3 * ez <= 64 && rows <= 4 * RMAX) {
      // one row (3 ez consecutive floats, contiguous in HBM unless z wraps) per wave and
      // step; all of a wave's row loads are in flight before the LDS stores
      const int lane = tid & 63;
      const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: scalar row walk
      const int tz = lane / 3, comp = lane - 3 * tz;
      const bool on = lane < 3 * ez;
      const unsigned lane_off = 3 * ((gz0 + tz) & nmask) + comp;
      float vals[RMAX];
      int tx = wv / ey, ty = wv - (wv / ey) * ey;
#pragma unroll
      for (int i = 0; i < RMAX; ++i) {
        if (wv + 4 * i < rows) {
          const unsigned gx = (gx0 + tx) & nmask, gy = (gy0 + ty) & nmask;
          const float* rowp = g + 3 * static_cast<size_t>((gx * n + gy) * n);
          if (on) vals[i] = rowp[lane_off];
        }
        ty += 4;
        while (ty >= ey) {
          ty -= ey;
          ++tx;
        }
      }
#pragma unroll
      for (int i = 0; i < RMAX; ++i)
        if (on && wv + 4 * i < rows) tile[(wv + 4 * i) * 3 * ez + lane] = vals[i];
    } else {
      for_box_nodes(ex, ey, ez, [&](int tx, int ty, int tz, int li) {
        const unsigned gx = (gx0 + tx) & nmask, gy = (gy0 + ty) & nmask,
                       gz = (gz0 + tz) & nmask;
        const float* v = g + 3 * ((gx * n + gy) * n + gz);
        tile[3 * li] = v[0];
        tile[3 * li + 1] = v[1];
        tile[3 * li + 2] = v[2];
      });
    }
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < PPT; ++q) {
    const int j = tid + q * NT;
    if (j >= cnt) continue;
    float a0 = 0.f, a1 = 0.f, a2 = 0.f;
    if ((c.ok >> q) & 1u) {
      Corner k;                                  // from the node and fraction kept above
      int t[3];
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        t[a] = (rel[q] >> (10 * a)) & 1023;
        k.w[a][1] = fr[q][a];
        k.w[a][0] = 1.0f - k.w[a][1];
      }
      if (use_tile) {
        const int base = (t[0] * ey + t[1]) * ez + t[2];
#pragma unroll
        for (int cx = 0; cx < 2; ++cx) {
#pragma unroll
          for (int cy = 0; cy < 2; ++cy) {
            const float wxy = k.w[0][cx] * k.w[1][cy];
            const float* v = tile + 3 * (base + (cx * ey + cy) * ez);
#pragma unroll
            for (int cz = 0; cz < 2; ++cz) {
              const float w = wxy * k.w[2][cz];
              a0 += w * v[3 * cz];
              a1 += w * v[3 * cz + 1];
              a2 += w * v[3 * cz + 2];
            }
          }
        }
      } else {
#pragma unroll
        for (int a = 0; a < 3; ++a) k.i[a] = (c.g0[a] + t[a]) & nmask;
        gather_global(g, n, nmask, k, a0, a1, a2);
      }
    }
    finish_particle<LEAP>(lp, acc, box * np + c0 + j, c.p[q][0], c.p[q][1], c.p[q][2], a0, a1,
                          a2, kk, dd);
  }
}

__global__ void extract_component_kernel(const float* __restrict__ src, float* __restrict__ dst,
                                         int64_t n, int comp) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
       i += stride)
    dst[i] = src[3 * i + comp];
}

int grid_blocks(int64_t work, int block, int ppt) {
  int64_t b = (work + static_cast<int64_t>(block) * ppt - 1) / (static_cast<int64_t>(block) * ppt);
  if (b < 1) b = 1;
  if (b > (1 << 30)) b = 1 << 30;
  return static_cast<int>(b);
}

}  // namespace

hipError_t launch_fill_zero(void* ptr, int64_t bytes, hipStream_t s) {
  float* p = static_cast<float*>(ptr);
  const int64_t n = bytes / 4;
  const int64_t n4 = n / 4;
  if (n4 > 0) {
    int blocks = static_cast<int>(std::min<int64_t>((n4 + 255) / 256, 8192));
    hipLaunchKernelGGL(fill_zero_kernel, dim3(blocks), dim3(256), 0, s,
                       reinterpret_cast<float4*>(p), n4);
  }
  if (n4 * 4 < n)
    hipLaunchKernelGGL(fill_zero_tail_kernel, dim3(1), dim3(4), 0, s, p, n4 * 4, n);
  return hipGetLastError();
}

hipError_t launch_extract_component(const float* src, float* dst, int64_t n, int comp,
                                   hipStream_t s) {
  int blocks = static_cast<int>(std::min<int64_t>((n + 255) / 256, 8192));
  hipLaunchKernelGGL(extract_component_kernel, dim3(blocks), dim3(256), 0, s, src, dst, n, comp);
  return hipGetLastError();
}

template <int CH, int CAP, int NT>
hipError_t launch_tiled(const float* pos, unsigned long long* rho, int64_t np, int nbox, int n,
                        double inv_cell, int* flags, hipStream_t s) {
  const int64_t chunks = (np + CH - 1) / CH;
  hipLaunchKernelGGL((deposit_tiled_kernel<CH, CAP, NT>),
                     dim3(static_cast<unsigned>(chunks * nbox)), dim3(NT), 0, s, pos, rho, np, n,
                     inv_cell, flags, chunks);
  return hipGetLastError();
}

// Mode 4 takes chunks of 512 particles on 256 threads where the 4096-particle chunks would
// leave the chip idle, or a chunk would be most of a small mesh (boxes of 32^3, whose tile of a
// 16^3 block plus its halo is the mesh again for every chunk). A tile of 3328 nodes (27 KB) holds
// an 8^3 block with a halo of three nodes a side. Deposit alone, us, 4096 -> 512 particles a
// chunk, Morton order: one 32^3 box 10.0 -> 5.0 (8 workgroups -> 64), one 64^3 box 11.9 -> 9.4,
// 16 and 256 boxes of 32^3 28.9 -> 13.0 and 234 -> 123. From 512 chunks of 4096 on the larger
// chunk has fewer atomics to flush and wins (128^3: 30.5 against 36.1); on meshes up to 32^3,
// where many particles share a node, from 256 on, or at 32^3 from four a node on (a box of at
// most 512 particles is one chunk either way and keeps the smaller tile). There 256 threads are
// faster than 512 (64 boxes of 32^3 with 64^3 particles: 186 against 210). A step,
// us, 512 a chunk / 4096 on 256 threads, Morton order: 8^3 with 128^3 particles 92 / 77, 64
// boxes of 16^3 with 48^3 185 / 168, 32^3 with 200^3 202 / 188, 64 boxes of 32^3 with 32^3 125 /
// 437, with 50^3 240 / 464, with 64^3 418 / 359.
constexpr int64_t kSmallDeposit = 512, kSmallMeshDeposit = 256;
// mode 0: one thread per particle, global atomics (`block` threads per workgroup);
// modes 1-5: LDS-privatised chunks of 1024 / 2048 / 4096 particles with 256 threads, 4096
// with 512 threads, 8192 with 1024 threads.
hipError_t launch_deposit(const float* pos, unsigned long long* rho, int64_t np, int nbox, int n,
                          double inv_cell, int* flags, int mode, int block, hipStream_t s) {
  switch (mode) {
    case 1: return launch_tiled<1024, 3328, 256>(pos, rho, np, nbox, n, inv_cell, flags, s);
    case 2: return launch_tiled<2048, 5120, 256>(pos, rho, np, nbox, n, inv_cell, flags, s);
    case 3: return launch_tiled<4096, 9216, 256>(pos, rho, np, nbox, n, inv_cell, flags, s);
    case 4: {
      const int64_t chunks = (np + 4095) / 4096 * nbox;
      if (chunks < (n <= 32 ? kSmallMeshDeposit : kSmallDeposit) || (n <= 32 && np <= 512) ||
          (n == 32 && np < 4 * n * n * n))
        return launch_tiled<512, 3328, 256>(pos, rho, np, nbox, n, inv_cell, flags, s);
      if (n <= 32) return launch_tiled<4096, 9216, 256>(pos, rho, np, nbox, n, inv_cell, flags, s);
      return launch_tiled<4096, 9216, 512>(pos, rho, np, nbox, n, inv_cell, flags, s);
    }
    case 5: return launch_tiled<8192, 18432, 1024>(pos, rho, np, nbox, n, inv_cell, flags, s);
    default:
      hipLaunchKernelGGL(deposit_kernel, dim3(grid_blocks(np * nbox, block, 1)), dim3(block), 0,
                         s, pos, rho, np, nbox, n, inv_cell, flags);
      return hipGetLastError();
  }
}

int patch_cb_log2(int n) { return n >= 16 ? 4 : 3; }
int64_t patch_coarse_cells(int n) {
  const int64_t nc = n >> patch_cb_log2(n);
  return nc * nc * nc;
}

hipError_t launch_deposit_patch(const float* pos, unsigned long long* patches,
                                const PatchLayout& layout, int* reg_count, int4* reg_list,
                                unsigned long long* rho_fb, int* n_fb,
                                int64_t np, int nbox, int n, double inv_cell, int* flags,
                                bool big_tile, hipStream_t s) {
  if (n > 512) return hipErrorInvalidValue;      // registry entries pack extents up to n in 10 bits
  const int64_t chunks = layout.chunks;
  const dim3 grid(static_cast<unsigned>(chunks * nbox));
  const int ch = layout.particles;
  const auto launch = [&](auto tile) {
    constexpr int TILE = decltype(tile)::value;
    const auto go = [&](auto part) {
      hipLaunchKernelGGL((deposit_patch_kernel<decltype(part)::value, TILE, kPatchNT>), grid,
                         dim3(kPatchNT), 0, s, pos, patches, layout.slot, reg_count, reg_list,
                         rho_fb, n_fb, np, n, inv_cell, flags, chunks, patch_cb_log2(n));
    };
    if (ch == kPatchCH) go(std::integral_constant<int, kPatchCH>{});
    else if (ch == 2048) go(std::integral_constant<int, 2048>{});
    else go(std::integral_constant<int, 1024>{});
  };
  // one 64^3 box (64 chunks): 13.2 -> 13.4 us for boxes of one pass, 20.8 -> 18.8 (displaced by
  // two cells) and 24.2 -> 19.2 (C order) for those that the smaller tile takes several for
  if (chunks * nbox <= kPatchFewChunks) launch(std::integral_constant<int, kPatchFewTile>{});
  else if (big_tile) launch(std::integral_constant<int, kPatchCap>{});
  else launch(std::integral_constant<int, kPatchTile>{});
  return hipGetLastError();
}

hipError_t launch_patch_reduce(const unsigned long long* patches, int slot, const int* reg_count,
                               const int4* reg_list, unsigned long long* rho_fb,
                               const int* n_fb, float* delta, int nbox, int n, double scale,
                               hipStream_t s) {
  // slabs of 8 x-planes, half a 16^3 cell (a whole 8^3 one); of 2 where those leave the chip's
  // 256 CUs fewer than two workgroups each (one 64^3 box 10.1 -> 8.7 us, in C order 20.8 -> 10.5)
  const int cells = static_cast<int>(patch_coarse_cells(n)), cb = 1 << patch_cb_log2(n);
  const auto launch = [&](auto xd) {
    constexpr int XD = decltype(xd)::value;
    hipLaunchKernelGGL(patch_reduce_kernel<XD>, dim3(static_cast<unsigned>(cells * (cb / XD)), nbox),
                       dim3(256), 0, s, patches, slot, reg_count, reg_list, rho_fb, n_fb,
                       delta, n, patch_cb_log2(n), scale);
  };
  if (static_cast<int64_t>(cells) * (cb / 8) * nbox < 512) launch(std::integral_constant<int, 2>{});
  else launch(std::integral_constant<int, 8>{});
  return hipGetLastError();
}

hipError_t launch_delta_to_density(const float* delta, float* out, int64_t n, float rho_bar,
                                   hipStream_t s) {
  int blocks = static_cast<int>(std::min<int64_t>((n + 255) / 256, 8192));
  hipLaunchKernelGGL(delta_to_density_kernel, dim3(blocks), dim3(256), 0, s, delta, out, n,
                     rho_bar);
  return hipGetLastError();
}

// Blocks rounded up to whole XCD rounds; the extra blocks exit at once.
int xcd_blocks(int64_t nchunks) { return static_cast<int>((nchunks + 7) / 8 * 8); }

template <int CH, int CAP>
hipError_t launch_interp_tiled(const float* pos, const float* force, float* acc, int64_t np,
                               int nbox, int n, double inv_cell, const Leap* lp, hipStream_t s) {
  const int64_t chunks = (np + CH - 1) / CH;
  const dim3 grid(xcd_blocks(chunks * nbox));
  if (lp)
    hipLaunchKernelGGL((interp_tiled_kernel<CH, CAP, true>), grid, dim3(256), 0, s, pos, force,
                       acc, np, n, inv_cell, chunks, chunks * nbox, *lp);
  else
    hipLaunchKernelGGL((interp_tiled_kernel<CH, CAP, false>), grid, dim3(256), 0, s, pos, force,
                       acc, np, n, inv_cell, chunks, chunks * nbox, Leap());
  return hipGetLastError();
}

template <int PPT>
hipError_t launch_interp_direct(const float* pos, const float* force, float* acc, int64_t np,
                                int nbox, int n, double inv_cell, const Leap* lp,
                                hipStream_t s) {
  const int64_t chunks = (np + 256 * PPT - 1) / (256 * PPT);
  const dim3 grid(xcd_blocks(chunks * nbox));
  if (lp)
    hipLaunchKernelGGL((interp_kernel<PPT, true>), grid, dim3(256), 0, s, pos, force, acc, np, n,
                       inv_cell, chunks, chunks * nbox, *lp);
  else
    hipLaunchKernelGGL((interp_kernel<PPT, false>), grid, dim3(256), 0, s, pos, force, acc, np,
                       n, inv_cell, chunks, chunks * nbox, Leap());
  return hipGetLastError();
}

// mode 0: direct gather, `block` = particles per workgroup (256, 512 or 1024);
// modes 1-3: LDS-staged boxes of 1024 / 2048 / 4096 particles (mode 1's tile of 2048 nodes,
// 24 KB, leaves room for six workgroups per CU). lp (may be NULL): the leapfrog applied
// with each acceleration.
hipError_t launch_interp(const float* pos, const float* force, float* acc, int64_t np,
                         int nbox, int n, double inv_cell, int mode, int block, hipStream_t s,
                         const Leap* lp) {
  switch (mode) {
    case 1: return launch_interp_tiled<1024, 2048>(pos, force, acc, np, nbox, n, inv_cell, lp, s);
    case 2: return launch_interp_tiled<2048, 4608>(pos, force, acc, np, nbox, n, inv_cell, lp, s);
    case 3: return launch_interp_tiled<4096, 8192>(pos, force, acc, np, nbox, n, inv_cell, lp, s);
    default:
      if (block >= 1024)
        return launch_interp_direct<4>(pos, force, acc, np, nbox, n, inv_cell, lp, s);
      if (block >= 512)
        return launch_interp_direct<2>(pos, force, acc, np, nbox, n, inv_cell, lp, s);
      return launch_interp_direct<1>(pos, force, acc, np, nbox, n, inv_cell, lp, s);
  }
}

}  // namespace pmnu

// Stage (ii) of the step for one box without any device allocation: the CIC deposit, the
// forward real FFT and the binned P_cdm(k_b) of pm_nu_deposit + pm_nu_get_spectrum, with
// every intermediate in one file-scope device array (`scratch`) instead of a context's
// buffers. For callers that cannot allocate: code under HIP graph capture, serving loops,
// harnesses that forbid hipMalloc.
//
// The same kernels as the context's step do the work (LDS-privatised fixed-point deposit, the
// forward transform passes with the FP64 bin sums of the last one). What a context computes
// once on the host at init (bin table, mode counts, twiddles) is rebuilt here on every call,
// from edges and twiddles passed by value, so the call needs no host-to-device copy either:
// the tables by the kernel that clears the density, each bin's mode count by the workgroup
// that sums its power. Five launches; a box of 64^3 is bound by their latencies.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>

#include "response_device.hpp"

namespace pmnu {
namespace {

constexpr int kStaticMaxMesh = 64;     // largest N
constexpr int kStaticMaxBins = 256;    // largest B
constexpr int64_t kStaticBytes = 5 << 20;   // 5 MiB; the N = 64, B = 256 layout needs 3.3 MiB
constexpr int kMaxDevices = 64;

// The scratch of every call on this device (each device holds its own copy). In host code
// this name is not a device address: the address comes from hipGetSymbolAddress.
static __device__ __align__(256) unsigned char scratch[kStaticBytes];

std::mutex g_mu;
void* g_ptr[kMaxDevices] = {};   // per device: the address of `scratch` on that device

struct StaticTables {
  int edges[kStaticMaxBins + 1];      // integer |n|^2 edges of the bins
  float2 tw[kStaticMaxMesh];          // exp(-2 pi i m / N)
};

// The density cleared by every workgroup; the first ones also write the bin of every integer
// |n|^2 (as the context's host table), the bins' edges and the twiddles. One launch of N^3 / 1024 workgroups (each thread clears two nodes) instead of a
// table kernel of one workgroup, which also counted the modes there (112 us at N = 64, of 140
// for the call), and two fills.
__global__ __launch_bounds__(512) void static_setup_kernel(StaticTables t, int n, int nbins,
                                                           uint16_t* __restrict__ bin_of_n2,
                                                           int* __restrict__ edges,
                                                           float2* __restrict__ tw,
                                                           ulonglong2* __restrict__ rho,
                                                           int64_t n_pairs) {
  const int64_t gid = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (gid < n_pairs) rho[gid] = make_ulonglong2(0ull, 0ull);
  if (gid <= nbins) edges[gid] = t.edges[gid];
  if (gid < n) tw[gid] = t.tw[gid];
  if (gid <= 3 * n * n / 4) {
    const int n2 = static_cast<int>(gid);
    int lo = 0, hi = nbins - 1;        // the last b with edges[b] <= n2, at most nbins - 1
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (t.edges[mid] <= n2) lo = mid; else hi = mid - 1;
    }
    bin_of_n2[n2] = static_cast<uint16_t>(n2 == 0 ? 0 : lo);
  }
}

// Number of l in [-h, h) with l^2 < t.
__device__ __forceinline__ int lines_below(int t, int h) {
  if (t <= 0) return 0;
  int s = static_cast<int>(sqrtf(static_cast<float>(t - 1)));   // t <= 3 kStaticMaxMesh^2 / 4 + 1
  while (s * s > t - 1) --s;
  while ((s + 1) * (s + 1) <= t - 1) ++s;
  return s >= h ? 2 * h : 2 * s + 1;
}

// P_cdm of bin b from the partial sums of the forward transform, with the bin's full-sphere
// mode count taken here: the triples (i, j, l) of [-h, h)^3 with |n|^2 in the bin, as pairs
// (|i|, |j|) <= h with their multiplicity (1 for 0 and h, which only -h has; 2 between) times
// the number of l. (h + 1)^2 pairs over 256 threads are at most five each, exact integers.
__global__ __launch_bounds__(256) void static_power_kernel(StaticTables t, int n, int nbins,
                                                           const double* __restrict__ partial,
                                                           int n_partial, double norm,
                                                           double* __restrict__ pcdm) {
  __shared__ double red[256 / 64];
  __shared__ int s_cnt;
  const int b = blockIdx.x, h = n / 2, tid = threadIdx.x;
  if (tid == 0) s_cnt = 0;
  const int e0 = t.edges[b], e1 = b + 1 < nbins ? t.edges[b + 1] : 3 * n * n / 4 + 1;
  const double s = bin_mode_sum<256>(partial, n_partial, nbins, 0, b, red);   // barriers inside
  int cnt = 0;
  for (int p = tid; p < (h + 1) * (h + 1); p += 256) {
    const int i = p / (h + 1), j = p - i * (h + 1), r = i * i + j * j;
    const int mult = ((i == 0 || i == h) ? 1 : 2) * ((j == 0 || j == h) ? 1 : 2);
    cnt += mult * (lines_below(e1 - r, h) - lines_below(e0 - r, h));
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) cnt += __shfl_xor(cnt, off, 64);
  if ((tid & 63) == 0) atomicAdd(&s_cnt, cnt);
  __syncthreads();
  if (tid == 0) {
    const double c = static_cast<double>(s_cnt);
    pcdm[b] = c > 0.0 ? norm * s / c : 0.0;
  }
}

size_t align256(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }

// The address of `scratch` on the current device, looked up once per device.
int scratch_address(void** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return set_error(PM_NU_EHIP, "hipGetDevice: %s", hipGetErrorString(e));
  if (dev < 0 || dev >= kMaxDevices) return set_error(PM_NU_ENODEV, "device %d out of range", dev);
  std::lock_guard<std::mutex> lock(g_mu);
  if (!g_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
      return set_error(PM_NU_EHIP, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
    g_ptr[dev] = p;
  }
  *out = g_ptr[dev];
  return PM_NU_OK;
}

}  // namespace
}  // namespace pmnu

using namespace pmnu;

extern "C" int pm_nu_binned_power_noalloc(const float* pos, int64_t n_particles, int n_mesh,
                                          double box_size, int n_kbins, double* p_cdm,
                                          void* stream) {
  const int n = n_mesh;
  if (n < 8 || n > kStaticMaxMesh || (n & (n - 1)))
    return set_error(PM_NU_EINVAL, "n_mesh %d: the no-allocation call takes powers of two "
                                   "from 8 to %d", n, kStaticMaxMesh);
  if (n_kbins < 1 || n_kbins > kStaticMaxBins)
    return set_error(PM_NU_EINVAL, "n_kbins %d: the no-allocation call takes 1 to %d bins",
                     n_kbins, kStaticMaxBins);
  if (n_particles < 1 || !pos || !p_cdm)
    return set_error(PM_NU_EINVAL, "need n_particles >= 1, pos and p_cdm");
  if (!(box_size > 0.0) || !std::isfinite(box_size))
    return set_error(PM_NU_EINVAL, "box_size must be finite and > 0");

  // layout of the scratch for this call
  const int64_t M = static_cast<int64_t>(n) * n * n;
  const int64_t MH = static_cast<int64_t>(n) * n * (n / 2 + 1);
  const int n_partial = fwd_x_partials(n);
  size_t off = 0;
  const size_t o_rho = off;     off = align256(off + M * sizeof(unsigned long long));
  const size_t o_cb = off;      off = align256(off + MH * sizeof(float2));
  const size_t o_part = off;    off = align256(off + static_cast<size_t>(n_partial) * n_kbins * sizeof(double));
  const size_t o_bins = off;    off = align256(off + (3 * n * n / 4 + 1) * sizeof(uint16_t));
  const size_t o_edges = off;   off = align256(off + (n_kbins + 1) * sizeof(int));
  const size_t o_tw = off;      off = align256(off + n * sizeof(float2));
  const size_t o_flags = off;   off = align256(off + sizeof(int));
  if (n_partial <= 0 || off > static_cast<size_t>(kStaticBytes))
    return set_error(PM_NU_EINVAL, "n_mesh %d with %d bins needs %zu bytes of scratch (%lld held)",
                     n, n_kbins, off, static_cast<long long>(kStaticBytes));

  void* base = nullptr;
  int rc = scratch_address(&base);
  if (rc) return rc;
  unsigned char* s = static_cast<unsigned char*>(base);
  auto* rho = reinterpret_cast<unsigned long long*>(s + o_rho);
  auto* cb = reinterpret_cast<float2*>(s + o_cb);
  auto* part = reinterpret_cast<double*>(s + o_part);
  auto* bins = reinterpret_cast<uint16_t*>(s + o_bins);
  auto* edges = reinterpret_cast<int*>(s + o_edges);
  auto* tw = reinterpret_cast<float2*>(s + o_tw);
  auto* flags = reinterpret_cast<int*>(s + o_flags);

  // bin edges and twiddles exactly as a context computes them
  StaticTables t{};
  const double r2 = 3.0 * n * n / 4.0;
  for (int b = 0; b <= n_kbins; ++b)
    t.edges[b] = static_cast<int>(std::ceil(std::pow(r2, static_cast<double>(b) / n_kbins)));
  t.edges[0] = 1;
  for (int m = 0; m < n; ++m) {
    const double ph = -2.0 * kPi * m / n;
    t.tw[m] = make_float2(static_cast<float>(std::cos(ph)), static_cast<float>(std::sin(ph)));
  }
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int64_t pairs = M / 2;                  // the density as pairs of 64-bit nodes
  const int64_t threads = std::max<int64_t>(pairs, kStaticMaxBins + 1);   // the edges; M/2 > 3n^2/4
  hipLaunchKernelGGL(static_setup_kernel, dim3(static_cast<unsigned>((threads + 511) / 512)),
                     dim3(512), 0, st, t, n, n_kbins, bins, edges, tw,
                     reinterpret_cast<ulonglong2*>(rho), pairs);
  hipError_t e = hipGetLastError();
  const double scale = static_cast<double>(M) / static_cast<double>(n_particles) / kFixScale;
  const double norm = std::pow(box_size, 3) / (static_cast<double>(M) * M);
  e = e ? e : launch_deposit(pos, rho, n_particles, 1, n, n / box_size, flags, 4, 256, st);
  e = e ? e : launch_fwd_zy(n, rho, nullptr, nullptr, nullptr, 0, cb, tw, scale, 1, st);
  e = e ? e : launch_fwd_x_bin(n, cb, tw, bins, edges, part, n_kbins, 1, st);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(static_power_kernel, dim3(n_kbins), dim3(256), 0, st, t, n, n_kbins, part,
                       n_partial, norm, p_cdm);
    e = hipGetLastError();
  }
  if (e != hipSuccess)
    return set_error(PM_NU_EHIP, "no-allocation spectrum launch failed: %s", hipGetErrorString(e));
  return PM_NU_OK;
}

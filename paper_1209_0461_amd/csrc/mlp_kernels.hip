// Surrogate network for the neutrino history integral (gfx950): an MLP
// 16 -> 128 -> 128 -> 128 -> 1 with GELU hidden activations. Weights are rounded to
// bfloat16 (round to nearest even); every layer's input is carried as two bfloat16 parts,
// hi = bf16(v) and lo = bf16(v - hi) (a 16-bit significand), and multiplied by the weights as
// two bf16 products with FP32 accumulation; biases, pre-activations, GELU, the loss and all
// gradients are FP32. (A layer input rounded to one bfloat16 alone limits the network to
// about 2e-3 in ln R; the second part removes that floor.)
//
// Training and prediction run on the matrix cores, 32 rows at a time (below): the forward pass
// with the weights' share of every wave in registers, the backward pass (weight gradients
// H^T dZ and input gradients dZ W^T, with dZ rounded to bfloat16 as MFMA operand) with the
// weight gradients in registers. mlp_reduce_kernel adds up the workgroups' gradients and
// applies one Adam step to the FP32 masters.
//
// Inside the step one bin is one row, so a matrix-core tile would be 1/16 full:
// surrogate_response_kernel, one workgroup per (bin, box) like the exact response, forms
// P_cdm and the bin's inputs and takes the row through the network as FP32 dot products
// with the bfloat16 weights (packed once per weight change) held in registers, fetched at
// the start so that their latency hides behind the P_cdm reduction; it runs the exact
// integral (response_device.hpp) for a bin whose inputs fall outside the training range
// (or for every bin when checking). Its activations are FP32 where training carries them
// as hi + lo bfloat16 pairs (16-bit significand): the two agree to about 1e-5 in ln R.
#include <algorithm>

#include "response_device.hpp"
#include "surrogate_layout.hpp"

namespace pmnu {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ unsigned short f2bf(float f) {
  unsigned u = __float_as_uint(f);
  if ((u & 0x7f800000u) == 0x7f800000u) return static_cast<unsigned short>((u >> 16) | ((u & 0xffffu) ? 0x40u : 0u));
  u += 0x7fffu + ((u >> 16) & 1u);
  return static_cast<unsigned short>(u >> 16);
}
__device__ __forceinline__ float bf2f(unsigned short h) { return __uint_as_float(static_cast<unsigned>(h) << 16); }
__device__ __forceinline__ float bfr(float f) { return bf2f(f2bf(f)); }
// two values rounded to bfloat16 (nearest even), a in the low half
__device__ __forceinline__ unsigned pack_bf2(float a, float b) {
  const f32x2 v = {a, b};
  return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
}
// the second bfloat16 part of both, bf16(v - hi), given their packed first parts
__device__ __forceinline__ unsigned pack_lo2(float a, float b, unsigned hi) {
  return pack_bf2(a - __uint_as_float(hi << 16), b - __uint_as_float(hi & 0xffff0000u));
}

__device__ __forceinline__ float gelu(float x) {
  return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f));
}

// GELU and its derivative from one exponential, for the kernels whose time the erf took (384
// evaluations a row). Phi(-|x|) = exp(-x^2/2) R(|x|) with R(x) = erfcx(x / sqrt 2) / 2 as
// u p(u), u = 1 / (1 + 0.35 |x|), p the polynomial of degree 10 that minimises the largest
// relative error over 0 < u <= 1 (1.3e-8, fitted in FP64). Error of gelu over x ~ 1.5 N(0, 1):
// RMS 3.5e-8, against 3.7e-8 of 0.5 x (1 + erf) with an erf correct to the last bit.
__device__ __forceinline__ void gelu_both(float x, float& g, float& dg) {
  const float u = __builtin_amdgcn_rcpf(fmaf(0.35f, fabsf(x), 1.0f));
  float p = 0.019314134493470192f;
  p = fmaf(p, u, -0.10845651477575302f);
  p = fmaf(p, u, 0.23588690161705017f);
  p = fmaf(p, u, -0.2259197235107422f);
  p = fmaf(p, u, 0.06956905126571655f);
  p = fmaf(p, u, -0.028395146131515503f);
  p = fmaf(p, u, 0.04840278998017311f);
  p = fmaf(p, u, 0.08778655529022217f);
  p = fmaf(p, u, 0.12255290895700455f);
  p = fmaf(p, u, 0.13962922990322113f);
  p = fmaf(p, u, 0.1396297961473465f);
  const float e = __builtin_amdgcn_exp2f(x * x * -0.72134752044448170f);   // exp(-x^2/2)
  const float q = e * (p * u);
  const float phi = x > 0.f ? 1.0f - q : q;
  g = x * phi;
  dg = fmaf(x, e * 0.39894228040143268f, phi);
}

// ---------------------------------------------------- matrix-core network, rows at a time ----
// A workgroup of 512 threads (8 waves) takes TB = 32 rows through the network. Every product
// is formed transposed, Z^T = W^T H^T, so that wave w owns the 16 outputs 16 w .. +15 of every
// hidden layer: its share of the weights (16 rows of the packed [out][in] image, 16 bytes a
// lane and 32 inputs) stays in registers for all of the workgroup's rows, and a lane ends with
// 4 consecutive outputs of one row, which go to LDS as one 8-byte store. 16x16x32 bf16 MFMA:
// lane l gives row l % 16 of A and column l % 16 of B for k = 8 (l / 16) .. +7 and receives
// rows 4 (l / 16) .. +3 of column l % 16.
constexpr int TB = 32;         // rows per tile
constexpr int kNetNT = 512;    // threads per workgroup
constexpr int kHS = 136;       // LDS stride of a row's 128 activations (16-byte aligned, odd in
                               // 16-byte units over 4 banks: the b128 reads of 16 rows differ)
constexpr int kXS = 40;        // LDS stride of a row's inputs: 16 and 16 zeros (a 32-wide k step)
constexpr int kTS = 40;        // LDS stride of the transposed layouts ([unit][row])

// bfloat16 image of the weights: W1..W3 as [out][in] (A operand of the forward products and
// the in-step network), then W2, W3 as [in][out] (A operand of the backward products)
constexpr int kPackW1 = 0;
constexpr int kPackW2 = kPackW1 + 128 * 16;
constexpr int kPackW3 = kPackW2 + 128 * 128;
constexpr int kPackB2 = kPackW3 + 128 * 128;
constexpr int kPackB3 = kPackB2 + 128 * 128;
constexpr int kPackSize = kPackB3 + 128 * 128;

__device__ __forceinline__ f32x4 mfma(const uint4& a, const uint4& b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
__device__ __forceinline__ uint4 lds16(const unsigned short* p) {
  return *reinterpret_cast<const uint4*>(p);
}

struct NetLds {
  alignas(16) unsigned short x[2][TB * kXS];     // standardised inputs (bf16 hi, lo)
  alignas(16) unsigned short h[2][2][TB * kHS];  // H1, H2 (hi, lo), [row][unit]
  float red[kNetNT / 64][TB];                    // output partial sums of every wave
  float t[TB];                                   // standardised targets (NaN: not used)
};
struct TrainLds : NetLds {
  alignas(16) unsigned short xt[2][16 * kTS];       // the same transposed, [unit][row]
  alignas(16) unsigned short ht[2][2][128 * kTS];
  alignas(16) unsigned short dz[2][TB * kHS];       // dZ3, dZ2 (bf16), [row][unit]
  alignas(16) unsigned short dzt[3][128 * kTS];     // dZ3, dZ2, dZ1, [unit][row]
};

// a wave's share of the weights, biases and output weights
struct WaveNet {
  uint4 w1, w2[4], w3[4];
  float b1[4], b2[4], b3[4], w4[4], b4;
};
// 16 rows of a 128-wide matrix of the image
__device__ __forceinline__ void load_rows(const unsigned short* q, int o, int r, int g,
                                          uint4 (&w)[4]) {
#pragma unroll
  for (int kt = 0; kt < 4; ++kt) w[kt] = lds16(q + (o + r) * 128 + 32 * kt + 8 * g);
}
__device__ __forceinline__ void load_wave_weights(const unsigned short* Q, int o, int r, int g,
                                                  WaveNet& n) {
  // 16 inputs of a 32-wide k step: the upper half of the lanes holds zeros
  const uint4 w = lds16(Q + kPackW1 + (o + r) * 16 + 8 * (g & 1));
  n.w1 = make_uint4(g < 2 ? w.x : 0u, g < 2 ? w.y : 0u, g < 2 ? w.z : 0u, g < 2 ? w.w : 0u);
  load_rows(Q + kPackW2, o, r, g, n.w2);
  load_rows(Q + kPackW3, o, r, g, n.w3);
}
__device__ __forceinline__ void load_wave_biases(const float* __restrict__ P, int o, int g,
                                                 WaveNet& n) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    n.b1[q] = P[kOffB1 + o + 4 * g + q];
    n.b2[q] = P[kOffB2 + o + 4 * g + q];
    n.b3[q] = P[kOffB3 + o + 4 * g + q];
    n.w4[q] = bfr(P[kOffW4 + o + 4 * g + q]);
  }
  n.b4 = P[kOffB4];
}

// One hidden layer's pre-activations of this wave for both 16-row halves (hi then lo parts of
// the inputs over one FP32 accumulator each), without the bias.
__device__ __forceinline__ void layer128(const uint4 (&w)[4], const unsigned short (&h)[2][TB * kHS],
                                         int r, int g, f32x4 (&z)[2]) {
  z[0] = z[1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int part = 0; part < 2; ++part) {
#pragma unroll
    for (int kt = 0; kt < 4; ++kt)
#pragma unroll
      for (int m = 0; m < 2; ++m)
        z[m] = mfma(w[kt], lds16(&h[part][(16 * m + r) * kHS + 32 * kt + 8 * g]), z[m]);
    __builtin_amdgcn_sched_barrier(0);   // 8 operands in flight, not 16: registers
  }
}

// four units u .. u+3 of one row (packed bf16) into the [unit][row] layout
__device__ __forceinline__ void store_t(unsigned short* t, int u, int row, uint2 v) {
  t[u * kTS + row] = static_cast<unsigned short>(v.x);
  t[(u + 1) * kTS + row] = static_cast<unsigned short>(v.x >> 16);
  t[(u + 2) * kTS + row] = static_cast<unsigned short>(v.y);
  t[(u + 3) * kTS + row] = static_cast<unsigned short>(v.y >> 16);
}

// dZ of a layer: its FP32 sums into the bias gradient, its bfloat16 values to both layouts
__device__ __forceinline__ void store_dz(unsigned short* d, unsigned short* dt, const f32x4 (&dz)[2],
                                         float (&gb)[4], int o, int r, int g) {
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    const uint2 v = make_uint2(pack_bf2(dz[m][0], dz[m][1]), pack_bf2(dz[m][2], dz[m][3]));
    const int row = 16 * m + r, u = o + 4 * g;
    if (d) *reinterpret_cast<uint2*>(&d[row * kHS + u]) = v;
    store_t(dt, u, row, v);
#pragma unroll
    for (int q = 0; q < 4; ++q) gb[q] += dz[m][q];
  }
}

// dW += H^T dZ: this wave's 16 inputs by all 128 outputs
__device__ __forceinline__ void weight_grad32(const unsigned short (&ht)[2][128 * kTS],
                                              const unsigned short* dzt, int o, int r, int g,
                                              f32x4 (&acc)[8]) {
  const uint4 hi = lds16(&ht[0][(o + r) * kTS + 8 * g]), lo = lds16(&ht[1][(o + r) * kTS + 8 * g]);
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    const uint4 b = lds16(&dzt[(16 * t + r) * kTS + 8 * g]);
    acc[t] = mfma(hi, b, acc[t]);
    acc[t] = mfma(lo, b, acc[t]);
    if (t % 4 == 3) __builtin_amdgcn_sched_barrier(0);
  }
}

// dZ of the layer before: (W dZ^T) GELU'
__device__ __forceinline__ void backprop32(const uint4 (&wb)[4], const unsigned short* d,
                                           const float (&dg)[2][4], int r, int g, f32x4 (&dz)[2]) {
  f32x4 z[2];
  z[0] = z[1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kt = 0; kt < 4; ++kt)
#pragma unroll
    for (int m = 0; m < 2; ++m)
      z[m] = mfma(wb[kt], lds16(&d[(16 * m + r) * kHS + 32 * kt + 8 * g]), z[m]);
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int q = 0; q < 4; ++q) dz[m][q] = z[m][q] * dg[m][q];
}

// Activations of a layer from its pre-activations: H to LDS as hi + lo (with TRAIN also
// transposed) and GELU' kept for the backward pass.
template <bool TRAIN>
__device__ __forceinline__ void activate(const f32x4 (&z)[2], const float (&bias)[4], int o, int r,
                                         int g, unsigned short (&h)[2][TB * kHS],
                                         unsigned short (*ht)[128 * kTS], float (&dg)[2][4]) {
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    float v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) gelu_both(z[m][q] + bias[q], v[q], dg[m][q]);
    const uint2 hi = make_uint2(pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3]));
    const uint2 lo = make_uint2(pack_lo2(v[0], v[1], hi.x), pack_lo2(v[2], v[3], hi.y));
    const int row = 16 * m + r, u = o + 4 * g;
    *reinterpret_cast<uint2*>(&h[0][row * kHS + u]) = hi;
    *reinterpret_cast<uint2*>(&h[1][row * kHS + u]) = lo;
    if constexpr (TRAIN) {
      store_t(ht[0], u, row, hi);
      store_t(ht[1], u, row, lo);
    }
  }
}

// Forward pass of the tile whose inputs are in S.x (barrier before); the standardised outputs
// without bias are left as one partial sum per wave in S.red (barrier before reading).
template <bool TRAIN, typename L>
__device__ __forceinline__ void forward32(L& S, const WaveNet& n, int o, int r, int g,
                                          float (&dg)[3][2][4], float (&h3)[2][4]) {
  unsigned short(*ht1)[128 * kTS] = nullptr;
  unsigned short(*ht2)[128 * kTS] = nullptr;
  if constexpr (TRAIN) {
    ht1 = S.ht[0];
    ht2 = S.ht[1];
  }
  f32x4 z[2];
  z[0] = z[1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int part = 0; part < 2; ++part)
#pragma unroll
    for (int m = 0; m < 2; ++m)
      z[m] = mfma(n.w1, lds16(&S.x[part][(16 * m + r) * kXS + 8 * g]), z[m]);
  activate<TRAIN>(z, n.b1, o, r, g, S.h[0], ht1, dg[0]);
  __syncthreads();
  layer128(n.w2, S.h[0], r, g, z);
  activate<TRAIN>(z, n.b2, o, r, g, S.h[1], ht2, dg[1]);
  __syncthreads();
  layer128(n.w3, S.h[1], r, g, z);
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    float y = 0.f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      gelu_both(z[m][q] + n.b3[q], h3[m][q], dg[2][m][q]);
      y = fmaf(h3[m][q], n.w4[q], y);
    }
    y += __shfl_xor(y, 16, 64);
    y += __shfl_xor(y, 32, 64);
    if (g == 0) S.red[o >> 4][16 * m + r] = y;
  }
}

__device__ __forceinline__ float net_output(const NetLds& S, int row, float b4) {
  float y = S.red[0][row];
#pragma unroll
  for (int w = 1; w < kNetNT / 64; ++w) y += S.red[w][row];
  return y + b4;
}

// thread (row tid / 16, input tid % 16) stages its standardised input (0 beyond the rows)
__device__ __forceinline__ void stage_input(NetLds& S, float v) {
  const int s = threadIdx.x >> 4, i = threadIdx.x & 15;
  const unsigned short hi = f2bf(v);
  S.x[0][s * kXS + i] = hi;
  S.x[1][s * kXS + i] = f2bf(v - bf2f(hi));
}
__device__ __forceinline__ void zero_input_padding(NetLds& S) {
  const int s = threadIdx.x >> 4, i = 16 + (threadIdx.x & 15);
  S.x[0][s * kXS + i] = S.x[1][s * kXS + i] = 0;
}

// Rows of x through the network: a workgroup keeps its weights in registers and walks tiles
// of 32 rows, the next tile's inputs loaded while it works on one. Bound by the FP32
// arithmetic of the 384 GELUs a row; staging the weights for every 32 rows and gathering the
// MFMA operands from LDS two bytes at a time took 795 us for 200000 rows, this 75.
__global__ __launch_bounds__(kNetNT, 4) void mlp_predict_kernel(const float* __restrict__ P,
                                                                const unsigned short* __restrict__ Q,
                                                                const float* __restrict__ x,
                                                                float* __restrict__ y, int64_t n) {
  __shared__ NetLds S;
  const int tid = threadIdx.x, s = tid >> 4, i = tid & 15;
  const int64_t tiles = (n + TB - 1) / TB;
  const int r = tid & 15, g = (tid & 63) >> 4, o = 16 * (tid >> 6);
  WaveNet net;
  load_wave_weights(Q, o, r, g, net);
  load_wave_biases(P, o, g, net);
  const float mu = P[kOffMu + i], sg = P[kOffSigma + i];
  const float ymu = P[kOffYMu], ysg = P[kOffYSigma];
  auto input = [&](int64_t tile) -> float {
    const int64_t row = tile * TB + s;
    return tile < tiles && row < n ? x[row * kSurIn + i] : mu;
  };
  zero_input_padding(S);
  float xv = input(blockIdx.x);
  float dg[3][2][4], h3[2][4];
  // every LDS array is next written two barriers after its last read
  for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    stage_input(S, (xv - mu) / sg);
    xv = input(tile + gridDim.x);
    __syncthreads();
    forward32<false>(S, net, o, r, g, dg, h3);
    __syncthreads();
    const int64_t row = tile * TB + tid;
    if (tid < TB && row < n) y[row] = net_output(S, tid, net.b4) * ysg + ymu;
  }
}

// Loss and gradient of rows [row0, row0 + count) (through perm if given), one set of sums per
// workgroup in part (added up by mlp_reduce_kernel): each workgroup walks tiles of 32 rows, forward as above and backward
//   dW = H^T dZ           A = H^T from the [unit][row] copies (hi, lo), B = dZ likewise;
//                         wave w owns the inputs 16 w .. +15 of W2, W3 and the outputs of W1
//   dH^T = W dZ^T         A = its 16 rows of W ([in][out]), B = dZ [row][unit]: the result
//                         lies in the lanes as the forward pass's GELU' does
// with dZ rounded to bfloat16. The weight gradients of all its tiles stay in FP32 registers and
// leave as plain 16-byte stores: as atomics on one gradient, 256 workgroups times 35329 values,
// they took 95 us whatever the kernel did before them. 8192 rows: 98 us and 5 of Adam before, now
// 24 and 8; 100000 rows: 981 -> 123.
constexpr int kPartW3 = 0, kPartW2 = 128 * 128, kPartW1 = 2 * 128 * 128;
constexpr int kPartVec = kPartW1 + 16 * 128;         // dB1, dB2, dB3, dW4, dB4, loss
constexpr int kPartSize = kPartVec + 576;            // whole 256-byte lines
static_assert(kPartVec + 514 == kSurParams + 1, "every parameter and the loss");
constexpr int kTrainWGs = 256;                       // one per CU
__global__ __launch_bounds__(kNetNT) void mlp_train_kernel(const float* __restrict__ P,
                                                           const unsigned short* __restrict__ Q,
                                                           const float* __restrict__ x,
                                                           const float* __restrict__ y,
                                                           const int* __restrict__ perm,
                                                           int64_t row0, int64_t count,
                                                           float inv_batch,
                                                           float* __restrict__ part) {
  __shared__ TrainLds S;
  const int tid = threadIdx.x, l = tid & 63, wave = tid >> 6;
  int r = l & 15, g = l >> 4, o = __builtin_amdgcn_readfirstlane(16 * wave);
  const int64_t tiles = (count + TB - 1) / TB;
  WaveNet net;
  load_wave_biases(P, o, g, net);
  const int xs = tid >> 4, xi = tid & 15;
  const float mu = P[kOffMu + xi], sg = P[kOffSigma + xi];
  const float ymu = P[kOffYMu], ysg = P[kOffYSigma];
  // row of the batch that tile's row s holds, -1 beyond the rows
  auto row_of = [&](int64_t tile, int s) -> int64_t {
    const int64_t k = tile * TB + s;
    if (tile >= tiles || k >= count) return -1;
    return perm ? perm[row0 + k] : row0 + k;
  };
  zero_input_padding(S);
  int64_t rx = row_of(blockIdx.x, xs), ry = tid < TB ? row_of(blockIdx.x, tid) : -1;
  float xv = rx >= 0 ? x[rx * kSurIn + xi] : mu;
  float yv = ry >= 0 ? y[ry] : __builtin_nanf("");
  rx = row_of(blockIdx.x + gridDim.x, xs);
  ry = tid < TB ? row_of(blockIdx.x + gridDim.x, tid) : -1;

  f32x4 g3[8], g2[8], g1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < 8; ++t) g3[t] = g2[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  float gw4[4] = {}, gb[3][4] = {}, gb4 = 0.f, loss = 0.f;

  for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    // the lane's place made opaque: the LDS addresses are formed where they are used instead
    // of some fifty of them being kept (and spilled) over the loop
    // (likewise the weights come from the caches for every tile: they would not fit beside the
    // gradients)
    int q0 = 0;
    asm volatile("" : "+v"(r), "+v"(g), "+s"(o), "+s"(q0));
    const unsigned short* q = Q + q0;
    load_wave_weights(q, o, r, g, net);
    {
      const float v = (xv - mu) / sg;
      stage_input(S, v);
      const unsigned short hi = f2bf(v);
      S.xt[0][xi * kTS + xs] = hi;
      S.xt[1][xi * kTS + xs] = f2bf(v - bf2f(hi));
    }
    if (tid < TB) S.t[tid] = (yv - ymu) / ysg;
    // the next tile's inputs, and the rows of the one after
    xv = rx >= 0 ? x[rx * kSurIn + xi] : mu;
    yv = ry >= 0 ? y[ry] : __builtin_nanf("");
    rx = row_of(tile + 2 * static_cast<int64_t>(gridDim.x), xs);
    ry = tid < TB ? row_of(tile + 2 * static_cast<int64_t>(gridDim.x), tid) : -1;
    __syncthreads();
    float dg[3][2][4], h3[2][4];
    forward32<true>(S, net, o, r, g, dg, h3);
    __syncthreads();
    uint4 wb[4];
    load_rows(q + kPackB3, o, r, g, wb);
    // loss, dL/dy and dZ3
    f32x4 dz[2];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      const int row = 16 * m + r;
      const float t = S.t[row];
      float dy = 0.f;
      if (isfinite(t)) {
        const float res = net_output(S, row, net.b4) - t;
        dy = 2.0f * res * inv_batch;
        if (tid < 16) {
          loss = fmaf(res, res, loss);
          gb4 += dy;
        }
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        gw4[q] = fmaf(h3[m][q], dy, gw4[q]);
        dz[m][q] = dy * net.w4[q] * dg[2][m][q];
      }
    }
    store_dz(S.dz[0], S.dzt[0], dz, gb[2], o, r, g);
    __syncthreads();
    // layer 3: dW3, then dZ2
    weight_grad32(S.ht[1], S.dzt[0], o, r, g, g3);
    backprop32(wb, S.dz[0], dg[1], r, g, dz);
    load_rows(q + kPackB2, o, r, g, wb);
    store_dz(S.dz[1], S.dzt[1], dz, gb[1], o, r, g);
    __syncthreads();
    // layer 2: dW2, then dZ1
    weight_grad32(S.ht[0], S.dzt[1], o, r, g, g2);
    backprop32(wb, S.dz[1], dg[0], r, g, dz);
    store_dz(nullptr, S.dzt[2], dz, gb[0], o, r, g);
    __syncthreads();
    // layer 1: its 16 inputs by this wave's 16 outputs
    const uint4 b = lds16(&S.dzt[2][(o + r) * kTS + 8 * g]);
#pragma unroll
    for (int part = 0; part < 2; ++part) g1 = mfma(lds16(&S.xt[part][r * kTS + 8 * g]), b, g1);
    __syncthreads();                               // before the next tile's inputs
  }
  // the workgroup's sums, in the order that its lanes hold them
  float* p = part + static_cast<size_t>(blockIdx.x) * kPartSize;
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    *reinterpret_cast<f32x4*>(p + kPartW3 + ((wave * 8 + t) * 64 + l) * 4) = g3[t];
    *reinterpret_cast<f32x4*>(p + kPartW2 + ((wave * 8 + t) * 64 + l) * 4) = g2[t];
  }
  *reinterpret_cast<f32x4*>(p + kPartW1 + (wave * 64 + l) * 4) = g1;
  // sums over the rows (the 16 lanes of a group)
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    float v[4] = {gb[0][q], gb[1][q], gb[2][q], gw4[q]};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
#pragma unroll
      for (int off = 8; off > 0; off >>= 1) v[k] += __shfl_xor(v[k], off, 64);
      if (r == 0) p[kPartVec + 128 * k + o + 4 * g + q] = v[k];
    }
  }
  if (wave == 0) {
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) {
      loss += __shfl_xor(loss, off, 64);
      gb4 += __shfl_xor(gb4, off, 64);
    }
    if (tid == 0) {
      p[kPartVec + 512] = gb4;
      p[kPartVec + 513] = loss;
    }
  }
}

// the parameter that entry e of a workgroup's sums belongs to (kSurParams: the loss)
__device__ __forceinline__ int part_param(int e) {
  if (e < kPartVec) {
    const int q = e & 3, l = (e >> 2) & 63, r = l & 15, g = l >> 4, t = e >> 8;
    if (e >= kPartW1) return kOffW1 + (4 * g + q) * 128 + 16 * (t - (kPartW1 >> 8)) + r;
    const int tt = t & 63;                           // wave tt / 8, outputs 16 (tt % 8) .. +15
    return (e < kPartW2 ? kOffW3 : kOffW2) + (16 * (tt >> 3) + 4 * g + q) * 128 + 16 * (tt & 7) + r;
  }
  const int k = e - kPartVec;
  if (k >= 512) return k == 512 ? kOffB4 : kSurParams;
  const int off[4] = {kOffB1, kOffB2, kOffB3, kOffW4};
  return off[k >> 7] + (k & 127);
}

// A parameter's entries in the bfloat16 image
__device__ __forceinline__ void pack_param(unsigned short* __restrict__ Q, int i, float p) {
  const unsigned short h = f2bf(p);
  if (i < kOffB1) {
    Q[kPackW1 + (i % 128) * 16 + i / 128] = h;
  } else if (i >= kOffW2 && i < kOffB2) {
    const int j = i - kOffW2;
    Q[kPackW2 + (j % 128) * 128 + j / 128] = h;
    Q[kPackB2 + j] = h;
  } else if (i >= kOffW3 && i < kOffB3) {
    const int j = i - kOffW3;
    Q[kPackW3 + (j % 128) * 128 + j / 128] = h;
    Q[kPackB3 + j] = h;
  }
}

// Sums of the n_part workgroups of mlp_train_kernel, in a fixed order, and with ADAM one Adam
// step on them that also writes the bfloat16 image of the new weights, so that a minibatch is
// two launches; without, the gradient to grad. first: the loss starts here. One workgroup takes
// 64 entries, its four waves a quarter of the workgroups' sums each, 16 loads in flight.
template <bool ADAM>
__global__ __launch_bounds__(256) void mlp_reduce_kernel(
    const float* __restrict__ part, int n_part, int first, float* __restrict__ loss,
    float* __restrict__ grad, float* __restrict__ P, float* __restrict__ m, float* __restrict__ v,
    unsigned short* __restrict__ Q, float lr, float b1, float b2, float eps, float c1, float c2) {
  __shared__ float s_sum[4][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int e = blockIdx.x * 64 + lane;
  const bool on = e < kPartVec + 514;
  const int i = on ? part_param(e) : 0;
  const bool param = on && i < kSurParams;
  // the moments' loads go out with the sums'
  float mi = 0.f, vi = 0.f, pi = 0.f;
  if (ADAM && w == 0 && param) {
    mi = m[i];
    vi = v[i];
    pi = P[i];
  }
  float sum = 0.f;
  if (on) {
    constexpr int U = 16;
    for (int k0 = w; k0 < n_part; k0 += 4 * U) {
      float x[U];
#pragma unroll
      for (int u = 0; u < U; ++u)
        x[u] = k0 + 4 * u < n_part ? part[static_cast<size_t>(k0 + 4 * u) * kPartSize + e] : 0.f;
#pragma unroll
      for (int u = 0; u < U; ++u) sum += x[u];
    }
  }
  s_sum[w][lane] = sum;
  __syncthreads();
  if (w != 0 || !on) return;
  const float gi = (s_sum[0][lane] + s_sum[1][lane]) + (s_sum[2][lane] + s_sum[3][lane]);
  if (!param) {
    *loss = first ? gi : *loss + gi;
    return;
  }
  if constexpr (!ADAM) {
    grad[i] = gi;
    return;
  }
  mi = b1 * mi + (1.0f - b1) * gi;
  vi = b2 * vi + (1.0f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  pi -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  P[i] = pi;
  pack_param(Q, i, pi);
}

__global__ void pack_weights_kernel(const float* __restrict__ P, unsigned short* __restrict__ Q) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < kSurParams) pack_param(Q, i, P[i]);
}

// ---------------------------------------------------------------- in the step ----
// Inputs of (box, bin) as surrogate_layout.hpp defines them, from the stored history
// (hpm, hpn: this box's rows), the lag brackets the host put in the box's constants and
// box constants the host precomputed. Every value read from memory is one entry of a
// staging array, so that a workgroup can fetch them with one load per lane, all in flight
// together, before the P_cdm reduction (gather_value), and the inputs are formed once
// P_cdm^{1/2} is known (finish_features).
enum : int {
  kGLo = 0,                    // A at node sur_j[m]
  kGHi = kSurLags,             // A at node sur_j[m] + 1 (node sur_j[m] itself when sur_t = 0)
  kGT = 2 * kSurLags,          // sur_t[m]
  kGPn = 3 * kSurLags,         // P_nu^{1/2} at the last stored node
  kGLnA, kGM, kGGap, kGLnA0, kGLnX0,
  kGCount
};

__device__ __forceinline__ bool features_defined(const RespBox& bx) {
  return bx.sur_ok && bx.sur_hist && bx.kfs > 0.0;
}

__device__ __forceinline__ double gather_value(const RespBox* __restrict__ bxp,
                                               const double* hpm, const double* hpn, int nbins,
                                               int b, int i) {
  if (i < kGHi) return hpm[static_cast<size_t>(bxp->sur_j[i]) * nbins + b];
  if (i < kGT) {
    const int m = i - kGHi;
    return hpm[static_cast<size_t>(bxp->sur_j[m] + (bxp->sur_t[m] > 0.0 ? 1 : 0)) * nbins + b];
  }
  if (i < kGPn) return bxp->sur_t[i - kGT];
  switch (i) {
    case kGPn: return hpn[static_cast<size_t>(bxp->n_cur - 1) * nbins + b];
    case kGLnA: return bxp->sur_lna;
    case kGM: return bxp->m_total;
    case kGGap: return bxp->sur_gap;
    case kGLnA0: return bxp->sur_lna0;
    default: return bxp->sur_lnx0;
  }
}

// Input i (FP64, before the rounding to FP32), one input per call so that the lanes of a
// wave can form the inputs of a row together
__device__ __forceinline__ double feature_value(int i, double k, double pcdm_half,
                                                const double* g) {
  switch (i) {
    case 0: return log(k);
    case 1: return g[kGLnA];
    case 2: return g[kGM];
    case 3: return g[kGGap];
    case 4: return g[kGPn] / pcdm_half;
    case 5: return g[kGLnA0];
    case 6: return log(k) + g[kGLnX0];
    default: {
      const int m = i - 7;
      const double t = g[kGT + m];
      return ((1.0 - t) * g[kGLo + m] + t * g[kGHi + m]) / pcdm_half;
    }
  }
}

// whether input i's value keeps the row in the network's domain (input 6, the
// free-streaming argument across the last interval, at most kSurXLastMax)
__device__ __forceinline__ bool feature_in_domain(int i, double v) {
  return i != 6 || v <= kSurXLastMax;
}

__device__ __forceinline__ bool finish_features(double k, double pcdm_half, const double* g,
                                                float* f) {
  if (!(pcdm_half > 0.0)) return false;
  bool in = true;
  for (int i = 0; i < kSurIn; ++i) {
    const double v = feature_value(i, k, pcdm_half, g);
    in = in && feature_in_domain(i, v);
    f[i] = static_cast<float>(v);
  }
  return in;
}

// The inputs of one (box, bin) in one thread (training rows)
__device__ __forceinline__ bool make_features(const RespBox* __restrict__ bxp, double k,
                                              double pcdm_half, const double* hpm,
                                              const double* hpn, int nbins, int b, float* f) {
  if (!features_defined(*bxp)) return false;
  double g[kGCount];
#pragma unroll
  for (int i = 0; i < kGCount; ++i) g[i] = gather_value(bxp, hpm, hpn, nbins, b, i);
  return finish_features(k, pcdm_half, g, f);
}

__device__ __forceinline__ double approx_factor(double k, double kfs) {
  const double t = 1.0 + k / kfs;
  return 1.0 / (t * t);
}

// ---- one row through the network inside a workgroup of RT = 256 threads ----
// The weights come from the packed bfloat16 image Q ([out][in] rows) in 16-byte chunks of 8
// inputs. Layer 1 (128 x 16, 256 chunks): thread t holds chunk t, output t / 2, inputs
// 8 (t % 2) .. +7. Layers 2 and 3 (128 x 128, 2048 chunks): thread t holds chunks
// t + 256 u, u = 0..7, i.e. inputs 8 (t % 16) .. +7 of outputs t / 16 + 16 u; each load
// instruction of a wave covers 1 KB of contiguous weights. Activations stay FP32.
// The biases a thread adds are those of the output it finishes: t / 2 in layer 1 and
// hidden_out(t) in layers 2 and 3; thread t holds W4[t % 128] (threads t < 128 use it).
// Every load here is unconditional and its value first used after the P_cdm reduction, so
// that no wait for one of them stands between the loads and the reduction's own.
__device__ __forceinline__ int hidden_out(int t) {
  return (t >> 4) + 16 * (4 * ((t >> 3) & 1) + 2 * ((t >> 2) & 1) + ((t >> 1) & 1));
}

struct NetRegs {
  uint4 w1;
  uint4 w2[8], w3[8];
  float b1, b2, b3, w4;
  float b4, ymu, ysg;   // output bias, target mean and scale
};

__device__ __forceinline__ void load_net_weights(const float* __restrict__ P,
                                                 const unsigned short* __restrict__ Q, int t,
                                                 NetRegs& r) {
  const uint4* q = reinterpret_cast<const uint4*>(Q);
  r.w1 = q[kPackW1 / 8 + t];
#pragma unroll
  for (int u = 0; u < 8; ++u) r.w2[u] = q[kPackW2 / 8 + t + 256 * u];
#pragma unroll
  for (int u = 0; u < 8; ++u) r.w3[u] = q[kPackW3 / 8 + t + 256 * u];
  const int o = hidden_out(t);
  r.b1 = P[kOffB1 + (t >> 1)];
  r.b2 = P[kOffB2 + o];
  r.b3 = P[kOffB3 + o];
  r.w4 = P[kOffW4 + (t & 127)];   // used (bf16-rounded) by threads t < 128
  r.b4 = P[kOffB4];
  r.ymu = P[kOffYMu];
  r.ysg = P[kOffYSigma];
}

// sum_j a[j] w[j] over one chunk (w: 8 bfloat16 in a uint4)
__device__ __forceinline__ float chunk_dot(const float* a, const uint4& w) {
  const unsigned v[4] = {w.x, w.y, w.z, w.w};
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    s += a[2 * i] * __uint_as_float(v[i] << 16);
    s += a[2 * i + 1] * __uint_as_float(v[i] & 0xffff0000u);
  }
  return s;
}

// One 128 x 128 layer: h_out = GELU(W h_in + b). Each thread has the partial sums of 8
// outputs over its 8 inputs; the 16 threads sharing those outputs (16 consecutive lanes)
// add them in a butterfly that halves the outputs each lane carries at every step, after
// which lane pair (2v, 2v+1) of the group holds output (t / 16) + 16 u with
// u = 4 b3 + 2 b2 + b1 from the lane's bits.
__device__ __forceinline__ void hidden_128(const float* __restrict__ hin, const uint4* w,
                                           float bias, float* hout) {
  const int t = threadIdx.x, c = t & 15;
  float a[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) a[j] = hin[8 * c + j];
  float v[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) v[u] = chunk_dot(a, w[u]);
  const bool b3 = (t >> 3) & 1, b2 = (t >> 2) & 1, b1 = (t >> 1) & 1;
  float x4[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float keep = b3 ? v[4 + i] : v[i], send = b3 ? v[i] : v[4 + i];
    x4[i] = keep + __shfl_xor(send, 8, 64);
  }
  float x2[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const float keep = b2 ? x4[2 + i] : x4[i], send = b2 ? x4[i] : x4[2 + i];
    x2[i] = keep + __shfl_xor(send, 4, 64);
  }
  const float keep = b1 ? x2[1] : x2[0], send = b1 ? x2[0] : x2[1];
  float z = keep + __shfl_xor(send, 2, 64);
  z += __shfl_xor(z, 1, 64);
  if (!(t & 1)) hout[hidden_out(t)] = gelu(z + bias);
}

// The row's output y (standardised target) without the output bias, in every thread.
// x: the 16 standardised inputs in LDS; h0, h1: two 128-float LDS rows; red: RT / 64 floats.
__device__ __forceinline__ float net_forward(const NetRegs& r, const float* x, float* h0,
                                             float* h1, float* red) {
  const int t = threadIdx.x;
  {
    float a[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) a[j] = x[8 * (t & 1) + j];
    float z = chunk_dot(a, r.w1);
    z += __shfl_xor(z, 1, 64);
    if (!(t & 1)) h0[t >> 1] = gelu(z + r.b1);
  }
  __syncthreads();
  hidden_128(h0, r.w2, r.b2, h1);
  __syncthreads();
  hidden_128(h1, r.w3, r.b3, h0);
  __syncthreads();
  float s = t < 128 ? h0[t] * bfr(r.w4) : 0.f;
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) s += __shfl_xor(s, m, 64);
  if ((t & 63) == 0) red[t >> 6] = s;
  __syncthreads();
  float y = 0.f;
#pragma unroll
  for (int w = 0; w < RT / 64; ++w) y += red[w];
  return y;
}

// The surrogate's response, one workgroup per (bin b, box), as response_kernel but with the
// network in place of the history integral where it can answer: P_cdm from the deposit's
// partial sums, the bin's inputs (their memory reads and the network's weights are issued
// before the partial sums, so that the latencies overlap), the
// network's R, and the exact integral (response_device.hpp) for a bin whose inputs are not
// defined or fall outside the training range. Mode 1 keeps the network's R; mode 2 (check)
// keeps the exact result and records the network's beside it.
__global__ __launch_bounds__(RT) void surrogate_response_kernel(
    const float* __restrict__ P, const unsigned short* __restrict__ Q, int mode,
    const RespBox* __restrict__ boxes, const double* __restrict__ partial, int n_partial,
    const double* __restrict__ counts, const double* __restrict__ kmean,
    double* __restrict__ hist_pm, double* __restrict__ hist_pnu,
    const double* __restrict__ ic_pnu, const double* __restrict__ ic_theta,
    const double* __restrict__ tg_ds, const double* __restrict__ tg_l2,
    const double* __restrict__ tg_w, int nbins, int jcap, int qcap, int q_sub, int iterations,
    double norm, double* __restrict__ pcdm_out, double* __restrict__ pnu_out,
    double* __restrict__ ratio_out, double* __restrict__ sur_r, double* __restrict__ chk_exact,
    double* __restrict__ chk_sur) {
  __shared__ double red[2 * RT / 64];
  __shared__ float xs[kSurIn];
  __shared__ float h0[128], h1[128];
  __shared__ float redf[RT / 64];
  __shared__ float scal[4 * kSurIn];   // the inputs' mean, scale, minimum, maximum
  __shared__ double gsh[kGCount];      // the staged values of the inputs
  __shared__ int s_ok;
  const int tid = threadIdx.x;
  const int b = blockIdx.x, box = blockIdx.y;
  const size_t ob = static_cast<size_t>(box) * nbins + b;
  const RespBox* bxp = boxes + box;
  const RespBox bx = *bxp;
  double* hpm = hist_pm + static_cast<size_t>(box) * jcap * nbins;
  double* hpn = hist_pnu + static_cast<size_t>(box) * jcap * nbins;
  const size_t row = static_cast<size_t>(bx.n_cur) * nbins + b;
  const double cb = counts[b];
  const bool defined = cb > 0.0 && features_defined(bx);   // uniform over the workgroup
  const double kb = kmean[b];
  // fetched before the reduction: one staged value per lane and the scalers
  double gv = 0.0;
  float sc = 0.f;
  if (defined) {
    if (tid < kGCount) gv = gather_value(bxp, hpm, hpn, nbins, b, tid);
    if (tid < 4 * kSurIn) sc = P[kOffMu + tid];   // kOffMu .. kOffMax + kSurIn are contiguous
  }
  // the weights too: the reduction then waits for them as well (a wave consumes its loads
  // in issue order), which costs less than their latency after it (14.5 against 15.3 us)
  NetRegs w;
  if (defined) load_net_weights(P, Q, tid, w);
  const double msum = bin_mode_sum(partial, n_partial, nbins, box, b, red);   // has barriers
  const double pcdm = cb > 0.0 ? norm * msum / cb : 0.0;
  const double ph = sqrt(pcdm);
  if (defined) {
    if (tid < 4 * kSurIn) scal[tid] = sc;
    if (tid < kGCount) gsh[tid] = gv;
    __syncthreads();
  }
  if (tid < 64) {
    // lane i < kSurIn forms input i; the row is used when every input is in the network's
    // domain and within the training range (5% margin)
    bool in = true;
    float fv = 0.f;
    if (defined && ph > 0.0 && tid < kSurIn) {
      const double v = feature_value(tid, kb, ph, gsh);
      fv = static_cast<float>(v);
      const float lo = scal[2 * kSurIn + tid], hi = scal[3 * kSurIn + tid];
      const float mg = 0.05f * (hi - lo);
      in = feature_in_domain(tid, v) && fv >= lo - mg && fv <= hi + mg;
    }
    const bool ok = defined && ph > 0.0 && __all(in);
    if (ok && tid < kSurIn) xs[tid] = (fv - scal[tid]) / scal[kSurIn + tid];
    if (tid == 0) s_ok = ok ? 1 : 0;
  }
  if (tid == 0) {
    const bool ok = s_ok != 0;
    pcdm_out[ob] = pcdm;
    if (!(cb > 0.0)) {
      sur_r[ob] = __builtin_nan("");
      pnu_out[ob] = ratio_out[ob] = 0.0;
      hpm[row] = hpn[row] = 0.0;
      if (chk_exact) chk_exact[ob] = chk_sur[ob] = 0.0;
    } else if (!ok) {
      sur_r[ob] = __builtin_nan("");
    }
  }
  __syncthreads();
  const bool ok = s_ok != 0;
  if (ok) {
    const float y = net_forward(w, xs, h0, h1, redf) + w.b4;
    if (tid == 0) {
      const double r_net = exp(static_cast<double>(y * w.ysg + w.ymu)) *
                           approx_factor(kb, bx.kfs);
      sur_r[ob] = r_net;
      if (mode == 1) {
        const double pnu = r_net * ph;
        pnu_out[ob] = pnu;
        ratio_out[ob] = r_net;
        hpm[row] = (1.0 - bx.f_nu) * ph + bx.f_nu * pnu;
        hpn[row] = pnu;
      } else if (chk_sur) {
        chk_sur[ob] = r_net;
      }
    }
  }
  if (cb > 0.0 && (!ok || mode == 2)) {
    const double pnu = exact_pnu(bx, kb, ph, (bx.n_cur > 0 ? hpn[row - nbins] : 0.0),
                                 ic_pnu + static_cast<size_t>(box) * kMaxSpecies * nbins,
                                 ic_theta[ob], hpm, nbins, b,
                                 tg_ds + static_cast<size_t>(box) * qcap,
                                 tg_l2 + static_cast<size_t>(box) * qcap,
                                 tg_w + static_cast<size_t>(box) * qcap, q_sub, iterations, red);
    if (tid == 0) {
      const double r = ph > 0.0 ? pnu / ph : 0.0;   // no CDM power in the bin: R = 0
      pnu_out[ob] = pnu;
      ratio_out[ob] = r;
      hpm[row] = (1.0 - bx.f_nu) * ph + bx.f_nu * pnu;
      hpn[row] = pnu;
      if (chk_exact) {
        chk_exact[ob] = r;
        if (!ok) chk_sur[ob] = r;             // the network did not answer for this bin
      }
    }
  }
}

// Training rows from the step's state after an exact response: one thread per (box, bin).
__global__ void dataset_kernel(const RespBox* __restrict__ boxes, const double* __restrict__ pcdm,
                               const double* __restrict__ ratio, const double* __restrict__ kmean,
                               const double* __restrict__ hist_pm,
                               const double* __restrict__ hist_pnu, int nbins, int jcap,
                               int nbox, float* __restrict__ x, float* __restrict__ y) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nbox * nbins) return;
  const int box = i / nbins, b = i % nbins;
  const RespBox bx = boxes[box];
  const double ph = sqrt(pcdm[i]);
  const double r = ratio[i];
  float f[kSurIn];
  const size_t hoff = static_cast<size_t>(box) * jcap * nbins;
  bool ok = make_features(boxes + box, kmean[b], ph, hist_pm + hoff, hist_pnu + hoff, nbins, b,
                          f) &&
            r > 0.0;
  for (int c = 0; c < kSurIn; ++c) x[static_cast<size_t>(i) * kSurIn + c] = ok ? f[c] : 0.f;
  y[i] = ok ? static_cast<float>(log(r / approx_factor(kmean[b], bx.kfs)))
            : __builtin_nanf("");
}

}  // namespace

int64_t mlp_part_floats() { return static_cast<int64_t>(kTrainWGs) * kPartSize; }

// A workgroup per CU (its registers and LDS fill one) walks the tiles. Returns the number of
// sets of sums in *n_part.
hipError_t launch_mlp_train(const float* P, const unsigned short* Q, const float* x, const float* y,
                            const int* perm, int64_t row0, int64_t count, float inv_batch,
                            float* part, int* n_part, hipStream_t s) {
  const int64_t tiles = (count + TB - 1) / TB;
  *n_part = static_cast<int>(std::min<int64_t>(tiles, kTrainWGs));
  hipLaunchKernelGGL(mlp_train_kernel, dim3(static_cast<unsigned>(*n_part)), dim3(kNetNT), 0, s, P,
                     Q, x, y, perm, row0, count, inv_batch, part);
  return hipGetLastError();
}

hipError_t launch_mlp_predict(const float* P, const unsigned short* Q, const float* x, float* y,
                              int64_t n, hipStream_t s) {
  const int64_t tiles = (n + TB - 1) / TB;      // two workgroups per CU
  hipLaunchKernelGGL(mlp_predict_kernel, dim3(static_cast<unsigned>(std::min<int64_t>(tiles, 512))),
                     dim3(kNetNT), 0, s, P, Q, x, y, n);
  return hipGetLastError();
}

hipError_t launch_mlp_adam(const float* part, int n_part, bool first, float* loss, float* P,
                           float* m, float* v, unsigned short* Q, float lr, float b1, float b2,
                           float eps, float c1, float c2, hipStream_t s) {
  hipLaunchKernelGGL(mlp_reduce_kernel<true>, dim3((kPartVec + 514 + 63) / 64), dim3(256), 0, s, part,
                     n_part, first ? 1 : 0, loss, nullptr, P, m, v, Q, lr, b1, b2, eps, c1, c2);
  return hipGetLastError();
}

hipError_t launch_mlp_gradient(const float* part, int n_part, float* loss, float* grad,
                               hipStream_t s) {
  hipLaunchKernelGGL(mlp_reduce_kernel<false>, dim3((kPartVec + 514 + 63) / 64), dim3(256), 0, s,
                     part, n_part, 1, loss, grad, nullptr, nullptr, nullptr, nullptr, 0.f, 0.f, 0.f,
                     0.f, 0.f, 0.f);
  return hipGetLastError();
}

hipError_t launch_pack_weights(const float* P, unsigned short* Q, hipStream_t s) {
  hipLaunchKernelGGL(pack_weights_kernel, dim3((kSurParams + 255) / 256), dim3(256), 0, s, P, Q);
  return hipGetLastError();
}

int64_t packed_weight_count() { return kPackSize; }

hipError_t launch_surrogate_response(const float* P, const unsigned short* Q, int mode,
                                     const RespBox* boxes, const double* partial, int n_partial,
                                     const double* counts, const double* kmean, double* hist_pm,
                                     double* hist_pnu, const double* ic_pnu,
                                     const double* ic_theta, const double* tg_ds,
                                     const double* tg_l2, const double* tg_w, int nbins, int jcap,
                                     int qcap, int q_sub, int iterations, double norm, int nbox,
                                     double* pcdm, double* pnu, double* ratio, double* sur_r,
                                     double* chk_exact, double* chk_sur, hipStream_t s) {
  hipLaunchKernelGGL(surrogate_response_kernel, dim3(nbins, nbox), dim3(RT), 0, s, P, Q, mode,
                     boxes, partial, n_partial, counts, kmean, hist_pm, hist_pnu, ic_pnu,
                     ic_theta, tg_ds, tg_l2, tg_w, nbins, jcap, qcap, q_sub, iterations, norm, pcdm,
                     pnu, ratio, sur_r, chk_exact, chk_sur);
  return hipGetLastError();
}

hipError_t launch_surrogate_dataset(const RespBox* boxes, const double* pcdm, const double* ratio,
                                    const double* kmean, const double* hist_pm,
                                    const double* hist_pnu, int nbins, int jcap, int nbox,
                                    float* x, float* y, hipStream_t s) {
  const int n = nbox * nbins;
  hipLaunchKernelGGL(dataset_kernel, dim3((n + 255) / 256), dim3(256), 0, s, boxes, pcdm, ratio,
                     kmean, hist_pm, hist_pnu, nbins, jcap, nbox, x, y);
  return hipGetLastError();
}

}  // namespace pmnu

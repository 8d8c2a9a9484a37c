// Learned initial guess for the pressure projection on gfx950: a 3-level
// convolutional encoder-decoder (16/32/64 channels, 3x3x3 kernels, ReLU,
// 2x2x2 average pooling, nearest upsampling, skip connections by channel
// concatenation, 1x1x1 head) in bfloat16 with FP32 accumulation on the
// matrix cores, with its hand-written backward pass and Adam optimiser.
//
// Layout: activations are channels-last bfloat16, a[v * C + c] with the voxel
// index v = x + nx (y + ny z) of their resolution.  The first layer's four
// input channels are padded to 16 (zeros), so every convolution has C_in and
// C_out in multiples of 16.  A convolution is an implicit GEMM,
//   Y[v][co] = sum_{tap, ci} X[v + tap][ci] W[co][tap][ci],
// M = voxels, N = C_out, K = 27 C_in, computed 16 voxels x 16 channels x 16
// inputs of two taps at a time by v_mfma_f32_16x16x32_bf16 (k_conv).
// The backward pass w.r.t. the input is the same convolution with the
// kernel flipped in space and its channel roles swapped; the weight gradient
// is a GEMM over voxels (k_wgrad), its per-block partials summed in a fixed
// order.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <new>
#include <type_traits>
#include <vector>

#include "ns_internal.h"

namespace nsk {

namespace {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// round to nearest, ties to even
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

struct VDims {
  int nx, ny, nz;
};

__device__ __forceinline__ long vox_count(const VDims& d) { return (long)d.nx * d.ny * d.nz; }

// ------------------------------------------------------------ convolution
// 3x3x3 convolution with zero padding as an implicit GEMM on the matrix
// cores.  A block computes a 16 x 4 x 4 tile of output voxels for every
// output channel; wave w owns the four x-rows of z-plane w of the tile.  The
// input is staged in LDS 16 channels at a time with its one-voxel halo
// (18 x 6 x 6 voxels, 20.7 KB), and each v_mfma_f32_16x16x32_bf16 takes two
// taps x 16 input channels as its K = 32 (a 28th, zero tap pads the last
// pair).  With k = 16 (tap - 2p) + ci for tap pair p:
//   A (16 voxels x 32 k): lane l holds voxel row l%16, k = 8(l/16)..+7
//   B (32 k x 16 out):    lane l holds output column l%16, k = 8(l/16)..+7
//   D (16 x 16):          lane l holds column l%16, rows 4(l/16)..+3
// Each weight fragment read from the cache feeds the wave's four rows.
// The input is the channel concatenation of a tensor at this resolution
// (channels [0, ca), channel stride sa) and, for channels [ca, CIN), a tensor
// at half resolution read through nearest upsampling (channel stride sb), so
// the decoder never materialises its upsampled inputs.
// EPI 0: + bias, ReLU; 1: plain (gradient w.r.t. the input); 2: + bias,
// ReLU, then the 1x1x1 head 16 -> 1 into delta (FP32) and, if given, delta2;
// the activation is not stored.
// A tile has M rows in y (few_blocks, many_blocks), a block NB of the output channels' groups of 16: the accumulators' order of
// summation is the same in every form.
constexpr int kTX = 16, kTY = 4, kTZ = 4;
template <int M>
struct ConvTile {
  static constexpr int HX = kTX + 2, HY = M + 2, HZ = kTZ + 2, HV = HX * HY * HZ;
  // The two 8-channel halves of a staged chunk live in separate planes
  // (16-byte entries).  Adjacent 16-lane groups of an A-fragment read take the
  // two halves of the same voxels; the LDS serves half of one group with half
  // of the next, which is free of bank conflicts only when their entries are a
  // multiple of 16 apart, so the plane stride is a multiple of 16 entries.
  static constexpr int plane = (HV + 15) / 16 * 16;
  // offset of tap (dz, dy, dx) = (tap / 9, tap / 3 % 3, tap % 3) in the halo tile (0 for the pad tap)
  __host__ __device__ static constexpr int tap_off(int tap) {
    return tap >= 27 ? 0 : ((tap / 9) * HY + (tap / 3) % 3) * HX + tap % 3;
  }
};

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 u) { return __builtin_bit_cast(bf16x8, u); }

// 2x2x2 averages of a block's staged tile (per wavefront, i.e. z-plane, 16 M
// voxels of C channels) into the half-resolution tensor P, whose channels are
// all the block's; in k_pool's order
template <int C, int M>
__device__ __forceinline__ void pool_tile(const uint16_t* stg, const VDims& d, int x0, int y0, int z0, int ps, int po,
                                          uint16_t* __restrict__ P) {
  constexpr int G = C / 8, NV = 8 * (M / 2) * (kTZ / 2);
  const int e = threadIdx.x, v = e / G, g = e % G;
  const int X = v % 8, Y = v / 8 % (M / 2), Z = v / (4 * M);
  const int gx = x0 / 2 + X, gy = y0 / 2 + Y, gz = z0 / 2 + Z;
  if (v >= NV || gx >= d.nx / 2 || gy >= d.ny / 2 || gz >= d.nz / 2) return;
  float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const int i = q & 1, j = q >> 1 & 1, k = q >> 2;
    const u32x4 w = *reinterpret_cast<const u32x4*>(stg + ((2 * Z + k) * 16 * M + (2 * Y + j) * 16 + 2 * X + i) * C + 8 * g);
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      s[2 * h] += __uint_as_float(w[h] << 16);
      s[2 * h + 1] += __uint_as_float(w[h] & 0xFFFF0000u);
    }
  }
  u32x4 o;
#pragma unroll
  for (int h = 0; h < 4; ++h) o[h] = (uint32_t)f2bf(s[2 * h] * 0.125f) | ((uint32_t)f2bf(s[2 * h + 1] * 0.125f) << 16);
  *reinterpret_cast<u32x4*>(P + ((long)gx + (long)(d.nx / 2) * (gy + (long)(d.ny / 2) * gz)) * ps + po + 8 * g) = o;
}

// lane r ^ X of a row of 16 lanes
template <int X>
__device__ __forceinline__ float xor16(float v) {
  static_assert(X == 8 || X == 4 || X == 2 || X == 1, "one bit");
  const int u = __float_as_int(v);
  if constexpr (X == 8) return __int_as_float(__builtin_amdgcn_update_dpp(0, u, 0x128, 0xF, 0xF, false));   // row_ror:8
  if constexpr (X == 4) {   // row_shl:4 into the even quads, row_shr:4 into the odd ones
    const int t = __builtin_amdgcn_update_dpp(0, u, 0x104, 0xF, 0x5, false);
    return __int_as_float(__builtin_amdgcn_update_dpp(t, u, 0x114, 0xF, 0xA, false));
  }
  if constexpr (X == 2) return __int_as_float(__builtin_amdgcn_update_dpp(0, u, 0x4E, 0xF, 0xF, false));   // quad_perm
  return __int_as_float(__builtin_amdgcn_update_dpp(0, u, 0xB1, 0xF, 0xF, false));
}
// N values' sums over the 16 lanes of a row: lane r gets that of value r % N.
// Each step halves the values a lane carries, so 16 of them cost 15 exchanges;
// every sum is that of an exclusive-or butterfly.
template <int N>
__device__ __forceinline__ float sums16(float (&v)[N], int r) {
  static_assert(N == 16 || N == 8, "one row's lanes");
  auto half = [&](auto x, int n) {
    constexpr int X = decltype(x)::value;
    const bool hi = r & X;
#pragma unroll
    for (int q = 0; q < n; ++q) v[q] = (hi ? v[q + n] : v[q]) + xor16<X>(hi ? v[q] : v[q + n]);
  };
  if constexpr (N == 16)
    half(std::integral_constant<int, 8>{}, 8);
  else
#pragma unroll
    for (int q = 0; q < N; ++q) v[q] += xor16<8>(v[q]);
  half(std::integral_constant<int, 4>{}, 4);
  half(std::integral_constant<int, 2>{}, 2);
  half(std::integral_constant<int, 1>{}, 1);
  return v[0];
}

template <int CIN, int COUT, int EPI, int M, int NB, bool POOL>
__global__ void __launch_bounds__(256) k_conv(VDims d, const uint16_t* __restrict__ XA, int sa, int ca,
                                              const uint16_t* __restrict__ XB, int sb,
                                              const uint16_t* __restrict__ W, const float* __restrict__ bias,
                                              uint16_t* __restrict__ Y, int ys, int yo,
                                              const float* __restrict__ hw, const float* __restrict__ hb,
                                              float* __restrict__ delta, float* __restrict__ delta2,
                                              uint16_t* __restrict__ P) {
  static_assert(CIN % 16 == 0 && COUT % 16 == 0, "channels in multiples of 16");
  static_assert(EPI != 2 || COUT == 16, "the fused head takes 16 channels");
  using L = ConvTile<M>;
  constexpr int NG = COUT / 16 / NB, NC = CIN / 16, CB = 16 * NB;   // CB: output channels of the block
  constexpr int kHX = L::HX, kHY = L::HY, kHV = L::HV, kPlane = L::plane;
  constexpr int NE = (2 * kHV + 255) / 256;   // 16-byte tile pieces per thread
  // Weight fragments are loaded per tap pair (they stay in the caches):
  // holding a chunk's fourteen ahead in registers cost two of the wide
  // layers a wave per SIMD of occupancy, and the forward 9%.
  __shared__ u32x4 tile[2][2 * kPlane];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = lane & 15, kg = lane >> 4;
  const int x0 = blockIdx.x / NG * kTX, y0 = blockIdx.y * M, z0 = blockIdx.z * kTZ;
  const int g0 = blockIdx.x % NG * CB;   // the block's first output channel
  const int cnx = d.nx >> 1, cny = d.ny >> 1;
  const u32x4 zero = {0u, 0u, 0u, 0u};
  // this thread's tile pieces: fine and coarse voxel of each, in-grid mask
  int vf[NE], vc[NE];
  unsigned ok = 0;
#pragma unroll
  for (int i = 0; i < NE; ++i) {
    const int e = tid + 256 * i, hv = e >> 1;
    const int hx = hv % kHX, hy = (hv / kHX) % kHY, hz = hv / (kHX * kHY);
    const int gx = x0 - 1 + hx, gy = y0 - 1 + hy, gz = z0 - 1 + hz;
    vf[i] = vc[i] = 0;
    if (e < 2 * kHV && gx >= 0 && gx < d.nx && gy >= 0 && gy < d.ny && gz >= 0 && gz < d.nz) {
      ok |= 1u << i;
      vf[i] = gx + d.nx * (gy + d.ny * gz);
      vc[i] = (gx >> 1) + cnx * ((gy >> 1) + cny * (gz >> 1));
    }
  }
  const int half8 = 8 * (tid & 1);   // every piece of a thread has the same half (256 is even)
  u32x4 pre[NE];
  auto fetch = [&](int c) {
    const bool fromA = 16 * c < ca;
#pragma unroll
    for (int i = 0; i < NE; ++i) {
      pre[i] = zero;
      if (ok >> i & 1u) {
        const uint16_t* src = fromA ? XA + (long)vf[i] * sa + 16 * c + half8
                                    : XB + (long)vc[i] * sb + (16 * c - ca) + half8;
        pre[i] = *reinterpret_cast<const u32x4*>(src);
      }
    }
  };
  auto put = [&](int buf) {
#pragma unroll
    for (int i = 0; i < NE; ++i) {
      const int e = tid + 256 * i;
      if (e < 2 * kHV) tile[buf][(e & 1) * kPlane + (e >> 1)] = pre[i];
    }
  };
  // weight fragment of tap pair p, output tile t, chunk c (W in fragment order)
  const u32x4* wl = reinterpret_cast<const u32x4*>(W) + (long)(g0 / 16) * NC * 14 * 64 + lane;
  auto wfrag = [&](int p, int t, int c) -> bf16x8 { return as_bf16x8(wl[((t * NC + c) * 14 + p) * 64]); };
  const int lbase = (kg & 1) * kPlane + wave * kHY * kHX + r;   // this lane's A piece for tap 0, row 0
  f32x4 acc[M][NB];
#pragma unroll
  for (int m = 0; m < M; ++m)
#pragma unroll
    for (int t = 0; t < NB; ++t) acc[m][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  fetch(0);
  put(0);
  __syncthreads();
  // The tap pairs are software-pipelined: the four activation fragments of
  // pair p + 1 are read from LDS, and the weight fragments of pair p + WD
  // requested, before pair p's MFMAs issue, so that an MFMA never waits on
  // the read just before it (with the reads one fragment ahead, each MFMA
  // waited out an LDS round trip and the layer ran at a quarter of the MFMA
  // peak).  The first pairs' weights are requested before the next chunk's
  // tile pieces, which the in-order load counter would otherwise make them
  // wait behind.
  constexpr int WD = M == 2 ? 13 : M == 4 && NB == 1 ? 3 : 1;   // weight prefetch distance in tap pairs
  bf16x8 aq[2][M], bq[WD + 1][NB];
#pragma unroll 1
  for (int c = 0; c < NC; ++c) {
    const u32x4* T = tile[c & 1] + lbase;
    auto lda = [&](int p, bf16x8 (&a)[M]) {
      const bool tv = 2 * p + (kg >> 1) < 27;
      const int o = (kg >> 1) ? L::tap_off(2 * p + 1) : L::tap_off(2 * p);
#pragma unroll
      for (int m = 0; m < M; ++m) a[m] = as_bf16x8(tv ? T[o + m * kHX] : zero);
    };
#pragma unroll
    for (int q = 0; q < WD; ++q)
#pragma unroll
      for (int t = 0; t < NB; ++t) bq[q][t] = wfrag(q, t, c);
    if (c + 1 < NC) fetch(c + 1);
    lda(0, aq[0]);
#pragma unroll
    for (int p = 0; p < 14; ++p) {
      if (p + WD < 14) {
#pragma unroll
        for (int t = 0; t < NB; ++t) bq[(p + WD) % (WD + 1)][t] = wfrag(p + WD, t, c);
      }
      if (p + 1 < 14) lda(p + 1, aq[(p + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int m = 0; m < M; ++m)
#pragma unroll
        for (int t = 0; t < NB; ++t)
          acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aq[p & 1][m], bq[p % (WD + 1)][t], acc[m][t], 0, 0, 0);
    }
    if (c + 1 < NC) put((c + 1) & 1);
    __syncthreads();
  }
  // Epilogue.  Up to 64 output channels the wave's 16 M voxels x CB results
  // are transposed through its own slice of the (now idle) tile memory and
  // stored as 16-byte pieces of 8 channels; wider layers store directly.
  constexpr bool STAGE = CB <= 64;
  static_assert(!STAGE || 4 * 16 * M * CB * 2 <= (int)sizeof(tile), "staging fits in the tile");
  static_assert(!POOL || (STAGE && M % 2 == 0), "pooled from the staged tile");
  constexpr bool store = EPI != 2;   // (the head's layer keeps no activation)
  uint16_t* stg = reinterpret_cast<uint16_t*>(&tile[0][0]) + wave * 16 * M * CB;
  const int z = z0 + wave;
  constexpr int HR = M < 4 ? M : 4;   // rows whose head values are summed together
  float hs[4 * HR];
#pragma unroll
  for (int m = 0; m < M; ++m) {
    const int y = y0 + m;
    const long row = (long)d.nx * (y + (long)d.ny * z);
#pragma unroll
    for (int t = 0; t < NB; ++t) {
      const int cl = t * 16 + r, co = g0 + cl;
      const float bb = (EPI == 1) ? 0.f : bias[co];
      const float wh = (EPI == 2) ? hw[co] : 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int x = x0 + 4 * kg + i;
        float val = acc[m][t][i] + bb;
        if (EPI != 1) val = fmaxf(val, 0.f);
        const uint16_t q = f2bf(val);
        if (STAGE && store)
          stg[(m * 16 + 4 * kg + i) * CB + cl] = q;
        else if (store && x < d.nx && y < d.ny && z < d.nz)
          Y[(row + x) * ys + yo + co] = q;
        if (EPI == 2) hs[m % HR * 4 + i] = wh * bf2f(q);
      }
    }
    if (EPI == 2 && m % HR == HR - 1) {
      // sum the 16 channels, the 16 lanes of a row: lane r gets row r / 4's voxel r % 4
      const float h = sums16<4 * HR>(hs, r) + hb[0];
      const int yr = y - (HR - 1) + r / 4 % HR, x = x0 + 4 * kg + r % 4;
      if (r < 4 * HR && x < d.nx && yr < d.ny && z < d.nz) {
        const long v = x + (long)d.nx * (yr + (long)d.ny * z);
        delta[v] = h;
        if (delta2) delta2[v] = h;
      }
    }
  }
  if (STAGE && store) {
    __syncthreads();
    constexpr int G = CB / 8;   // 16-byte pieces per voxel
#pragma unroll
    for (int j = 0; j < (M * G + 3) / 4; ++j) {
      const int q = lane + 64 * j, vl = q / G, cg = q % G;
      const int x = x0 + (vl & 15), y = y0 + (vl >> 4);
      if (vl < 16 * M && x < d.nx && y < d.ny && z < d.nz)
        *reinterpret_cast<u32x4*>(Y + ((long)x + (long)d.nx * (y + (long)d.ny * z)) * ys + yo + g0 + 8 * cg) =
            *reinterpret_cast<const u32x4*>(stg + vl * CB + 8 * cg);
    }
    if (POOL) pool_tile<CB, M>(reinterpret_cast<uint16_t*>(&tile[0][0]), d, x0, y0, z0, COUT, g0, P);
  }
}

// The same convolution with K running over 32 input channels of one tap
// (channel-major), for the half-resolution decoder layer at inference (96
// input channels).  With the K of an MFMA inside one tap, the activation
// fragment of halo row y serves the output rows y - dy for all three dy taps
// of a (dz, dx) pair: a wave reads its ten halo rows once per (dz, dx) and
// issues 24 NT MFMAs from them, where the tap-pair form reads one fragment
// per MFMA row group.  A block computes a 16 x 8 x 4 tile of output voxels;
// wave w owns the eight x-rows of z-plane w, so each weight fragment feeds
// eight MFMAs.  Input channels are staged 32 at a time into LDS as four
// planes of 8 channels (16-byte entries; the plane stride a multiple of 16
// entries, so a 16-lane group's reads stay free of bank conflicts).
// Epilogues as k_conv.  At 256 x 128 x 128 it runs the 96 -> 32 layer in
// 108 us against k_conv's 155; for the 48 -> 16 layer (a 16-channel
// remainder chunk, run half empty or as tap pairs) it measured 348 and
// 328 us against k_conv's 321, and for 32 -> 64 (an eighth of the voxels)
// 23.5 against 21 us, so those stay on k_conv.  Its single-buffered 68 KB
// tile leaves two blocks per compute unit; a chunk's staging is hidden only
// by the other block, so the launch bound keeps the registers of two.
constexpr int kCX = 16, kCY = 8, kCZ = 4;

template <int CIN, int COUT, int M, int NB>
__global__ void __launch_bounds__(256, 2) k_conv_cm(VDims d, const uint16_t* __restrict__ XA, int sa, int ca,
                                                 const uint16_t* __restrict__ XB, int sb,
                                                 const uint16_t* __restrict__ W, const float* __restrict__ bias,
                                                 uint16_t* __restrict__ Y, int ys, int yo) {
  static_assert(CIN % 16 == 0 && COUT % 16 == 0, "channels in multiples of 16");
  static_assert(CIN % 32 == 0, "whole chunks of 32 input channels");
  constexpr int NG = COUT / 16 / NB, NC = CIN / 32, CB = 16 * NB;
  constexpr int kCHX = kCX + 2, kCHY = M + 2, kCHZ = kCZ + 2, kCHV = kCHX * kCHY * kCHZ;
  constexpr int kCPlane = (kCHV + 15) / 16 * 16;
  __shared__ u32x4 tile[4 * kCPlane];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = lane & 15, kg = lane >> 4;
  const int x0 = blockIdx.x / NG * kCX, y0 = blockIdx.y * M, z0 = blockIdx.z * kCZ;
  const int g0 = blockIdx.x % NG * CB;   // the block's first output channel
  const int cnx = d.nx >> 1, cny = d.ny >> 1;
  const u32x4 zero = {0u, 0u, 0u, 0u};
  f32x4 acc[M][NB];
#pragma unroll
  for (int m = 0; m < M; ++m)
#pragma unroll
    for (int t = 0; t < NB; ++t) acc[m][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  // weight fragment: tile t's output columns, chunk c's 32 channels of tap
  const u32x4* wl = reinterpret_cast<const u32x4*>(W) + (long)(g0 / 16) * NC * 27 * 64 + lane;
  auto wfrag = [&](int tap, int t, int c) -> bf16x8 { return as_bf16x8(wl[((t * NC + c) * 27 + tap) * 64]); };
#pragma unroll 1
  for (int c = 0; c < NC; ++c) {
    if (c > 0) __syncthreads();   // every wave is done with the previous chunk
    // stage channels [32 c, 32 c + 32): lanes 16 g .. 16 g + 15 take group g
    // (8 channels) of 16 consecutive halo voxels, so a wave reads 16 whole
    // 64-byte voxel slices and writes 16 consecutive entries of each plane.
    // Every load is issued (from a clamped address) before the first write.
    constexpr int NS = (kCHV + 63) / 64;
    const int ch = 32 * c + 8 * kg;
    u32x4 v[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int hv = 64 * s + 16 * wave + r;
      const int hx = hv % kCHX, hy = (hv / kCHX) % kCHY, hz = hv / (kCHX * kCHY);
      const int gx = x0 - 1 + hx, gy = y0 - 1 + hy, gz = z0 - 1 + hz;
      const bool in = hv < kCHV && gx >= 0 && gx < d.nx && gy >= 0 && gy < d.ny && gz >= 0 && gz < d.nz;
      const int cx = in ? gx : 0, cy = in ? gy : 0, cz = in ? gz : 0;
      const uint16_t* src = ch < ca ? XA + (long)(cx + d.nx * (cy + d.ny * cz)) * sa + ch
                                    : XB + (long)((cx >> 1) + cnx * ((cy >> 1) + cny * (cz >> 1))) * sb + (ch - ca);
      const u32x4 w = *reinterpret_cast<const u32x4*>(src);
      v[s] = in ? w : zero;
    }
    // (few blocks: nothing else hides the weights' latency, so all of the chunk's
    // are requested with its activations)
    bf16x8 ball[M == 2 ? 27 : 1][NB];
    if constexpr (M == 2) {
#pragma unroll
      for (int tap = 0; tap < 27; ++tap)
#pragma unroll
        for (int t = 0; t < NB; ++t) ball[tap][t] = wfrag(tap, t, c);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int hv = 64 * s + 16 * wave + r;
      if (hv < kCHV) tile[kg * kCPlane + hv] = v[s];
    }
    __syncthreads();
    const u32x4* T = tile + kg * kCPlane + r;
#pragma unroll
    for (int dz = 0; dz < 3; ++dz) {
#pragma unroll
      for (int dx = 0; dx < 3; ++dx) {
        bf16x8 b[3][NB];
#pragma unroll
        for (int dy = 0; dy < 3; ++dy)
#pragma unroll
          for (int t = 0; t < NB; ++t) {
            const int tap = 9 * dz + 3 * dy + dx;
            b[dy][t] = M == 2 ? ball[M == 2 ? tap : 0][t] : wfrag(tap, t, c);
          }
        bf16x8 a[kCHY];
#pragma unroll
        for (int hy = 0; hy < kCHY; ++hy) a[hy] = as_bf16x8(T[((wave + dz) * kCHY + hy) * kCHX + dx]);
#pragma unroll
        for (int dy = 0; dy < 3; ++dy)
#pragma unroll
          for (int m = 0; m < M; ++m)
#pragma unroll
            for (int t = 0; t < NB; ++t)
              acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[m + dy], b[dy][t], acc[m][t], 0, 0, 0);
      }
    }
  }
  // Epilogue: + bias, ReLU, BF16; the wave's 128 voxels x COUT results are
  // transposed through its own slice of the tile memory and stored as
  // 16-byte pieces of 8 channels.
  static_assert(M * 16 * CB * 2 * 4 <= (int)sizeof(tile), "staging fits in the tile");
  __syncthreads();
  uint16_t* stg = reinterpret_cast<uint16_t*>(&tile[0]) + wave * M * 16 * CB;
  const int z = z0 + wave;
#pragma unroll
  for (int m = 0; m < M; ++m) {
#pragma unroll
    for (int t = 0; t < NB; ++t) {
      const int cl = t * 16 + r, co = g0 + cl;
      const float bb = bias[co];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float val = fmaxf(acc[m][t][i] + bb, 0.f);
        const uint16_t q = f2bf(val);
        stg[(m * 16 + 4 * kg + i) * CB + cl] = q;
      }
    }
  }
  {
    __syncthreads();
    constexpr int G = CB / 8;   // 16-byte pieces per voxel
#pragma unroll
    for (int j = 0; j < M * G / 4; ++j) {
      const int q = lane + 64 * j, vl = q / G, cg = q % G;
      const int x = x0 + (vl & 15), y = y0 + (vl >> 4);
      if (x < d.nx && y < d.ny && z < d.nz)
        *reinterpret_cast<u32x4*>(Y + ((long)x + (long)d.nx * (y + (long)d.ny * z)) * ys + yo + g0 + 8 * cg) =
            *reinterpret_cast<const u32x4*>(stg + vl * CB + 8 * cg);
    }
  }
}

// First layer at inference, from the four feature channels in bfloat16 (8 bytes
// per voxel: k_pack_input), and K runs over (tap, channel) compactly, k = 4 tap + ci with
// 108 real entries padded to 128: four K = 32 steps instead of fourteen.
// Wc holds the four steps' fragments.  Output: + bias, ReLU, bfloat16, channel stride ys,
// and its 2x2x2 averages P.
template <int M>
__global__ void __launch_bounds__(256) k_conv_in(VDims d, const u32x2* __restrict__ xin,
                                                 const uint16_t* __restrict__ Wc, const float* __restrict__ bias,
                                                 uint16_t* __restrict__ Y, int ys, uint16_t* __restrict__ P) {
  using L = ConvTile<M>;
  constexpr int kHX = L::HX, kHY = L::HY, kHV = L::HV;
  __shared__ u32x2 tile[kHV + 8];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, kg = lane >> 4;
  const int x0 = blockIdx.x * kTX, y0 = blockIdx.y * M, z0 = blockIdx.z * kTZ;
  for (int e = threadIdx.x; e < kHV; e += 256) {
    const int hx = e % kHX, hy = (e / kHX) % kHY, hz = e / (kHX * kHY);
    const int gx = x0 - 1 + hx, gy = y0 - 1 + hy, gz = z0 - 1 + hz;
    u32x2 val = {0u, 0u};
    if (gx >= 0 && gx < d.nx && gy >= 0 && gy < d.ny && gz >= 0 && gz < d.nz) {
      val = xin[(long)gx + (long)d.nx * (gy + (long)d.ny * gz)];
    }
    tile[e] = val;
  }
  __syncthreads();
  f32x4 acc[M];
#pragma unroll
  for (int m = 0; m < M; ++m) acc[m] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int st = 0; st < 4; ++st) {
    const int t0 = 8 * st + 2 * kg, t1 = t0 + 1;   // this lane's two taps
    const bf16x8 b = as_bf16x8(reinterpret_cast<const u32x4*>(Wc)[64 * st + lane]);
    const int o0 = ((t0 / 9) * kHY + (t0 / 3) % 3) * kHX + t0 % 3;
    const int o1 = ((t1 / 9) * kHY + (t1 / 3) % 3) * kHX + t1 % 3;
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const int base = (wave * kHY + m) * kHX + r;
      const u32x2 p0 = t0 < 27 ? tile[base + o0] : u32x2{0u, 0u};
      const u32x2 p1 = t1 < 27 ? tile[base + o1] : u32x2{0u, 0u};
      const u32x4 a = {p0[0], p0[1], p1[0], p1[1]};
      acc[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(a), b, acc[m], 0, 0, 0);
    }
  }
  // transpose through LDS and store 16-byte pieces (as in k_conv)
  __shared__ uint16_t stg_all[4 * 16 * M * 16];
  uint16_t* stg = stg_all + wave * 16 * M * 16;
  const float bb = bias[r];
#pragma unroll
  for (int m = 0; m < M; ++m)
#pragma unroll
    for (int i = 0; i < 4; ++i) stg[(m * 16 + 4 * kg + i) * 16 + r] = f2bf(fmaxf(acc[m][i] + bb, 0.f));
  __syncthreads();
  const int z = z0 + wave;
#pragma unroll
  for (int j = 0; j < M / 2; ++j) {
    const int q = lane + 64 * j, vl = q >> 1, cg = q & 1;
    const int x = x0 + (vl & 15), y = y0 + (vl >> 4);
    if (x < d.nx && y < d.ny && z < d.nz)
      *reinterpret_cast<u32x4*>(Y + ((long)x + (long)d.nx * (y + (long)d.ny * z)) * ys + 8 * cg) =
          *reinterpret_cast<const u32x4*>(stg + vl * 16 + 8 * cg);
  }
  pool_tile<16, M>(stg_all, d, x0, y0, z0, 16, 0, P);
}

// Weight and bias gradient of a convolution,
//   dW[co][tap][ci] = sum_v dY[v][co] X[v + tap][ci],  db[co] = sum_v dY[v][co],
// on the matrix cores with the voxels as K: v_mfma_f32_16x16x32_bf16 takes 16
// output channels (rows) x 16 input channels (columns) x 32 voxels.  The
// tensors are channels-last, so a tile of 16 x 4 x 2 voxels is staged in LDS
// transposed, 16 x-consecutive voxels of one channel per row: a fragment is
// then one 16-byte read, and the three dx taps come from that read and its two
// edge voxels by shifts.  A block takes 16 input channels (blockIdx.y picks
// them): each of its three waves owns one dz plane of taps and keeps its
// 9 x COUT/16 accumulators in registers over all the block's tiles, so the tile
// is read from memory once for all 27 taps and only one partial per block is
// written; the next tile's loads are in flight while this one is multiplied.
// A layer of more input channels has several such blocks on a unit, which wait
// at their barriers at different times: as one block of nine waves the 48 -> 16
// layer took 63.0 us at 128 x 64 x 64, as three of three 56.7, though each reads
// dY (the 96 -> 32 layer 27.4 and 27.6).  What it replaced had one tap per
// block, read X and dY 27 times with 2-byte gathers and summed the bias in a
// kernel of its own: at 128 x 64 x 64 the 48 -> 16 layer took 538 + 62 us and
// the five layers 1.9 ms of a 2.5 ms training step.
// X is, as in k_conv, the concatenation of XA (channels [0, ca)) and a
// half-resolution XB read through nearest upsampling.
constexpr int kWX = 16, kWY = 4, kWZ = 2;                 // output voxels of a tile
constexpr int kWRows = (kWY + 2) * (kWZ + 2);             // halo rows of a channel
// dwords: a halo row holds x = 0..16 in elements 0..16 and x = -1 in element
// 23; a channel's stride is 4 modulo 8 times an odd count of 16-byte units, so
// that 16 lanes reading 16 bytes of 16 channels meet no bank conflict
constexpr int kWRow = 12, kWChan = kWRows * kWRow + 4, kWdY = kWX * kWY * kWZ / 2 + 4;

constexpr int kWCI = 16;   // input channels of a block

template <int CIN, int COUT>
__global__ void __launch_bounds__(12 * kWCI) k_wgrad(VDims d, const uint16_t* __restrict__ XA, int sa, int ca,
                                                   const uint16_t* __restrict__ XB, int sb,
                                                   const uint16_t* __restrict__ dY, int ntx, int nty, int tiles,
                                                   float* __restrict__ part) {
  static_assert(CIN % 16 == 0 && COUT % 16 == 0, "channels in multiples of 16");
  constexpr int CI = kWCI;
  constexpr int NT = 12 * CI, NO = COUT / 16, GX = CI / 8, GY = COUT / 8;
  constexpr int IX = kWRows * 10 * GX, SX = (IX + NT - 1) / NT;          // staged pieces of X: rows x 10 voxel pairs
  constexpr int IY = kWY * kWZ * 8 * GY, SY = (IY + NT - 1) / NT;        // of dY
  __shared__ uint32_t lx[CI * kWChan];
  __shared__ uint32_t ly[COUT * kWdY];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = lane & 15, kg = lane >> 4;
  const int dz = wave;
  const int c0 = (int)blockIdx.y * CI;
  const int cnx = d.nx >> 1, cny = d.ny >> 1;
  const u32x4 zero = {0u, 0u, 0u, 0u};
  u32x4 px[SX][2], py[SY][2];
  auto fetch = [&](int t) {
    const int x0 = (t % ntx) * kWX, y0 = (t / ntx) % nty * kWY, z0 = t / (ntx * nty) * kWZ;
#pragma unroll
    for (int s = 0; s < SX; ++s) {
      const int it = tid + NT * s, cg = it % GX, p = it / GX % 10, row = it / (GX * 10);
      const int gy = y0 - 1 + row % (kWY + 2), gz = z0 - 1 + row / (kWY + 2);
      const int xa = p < 9 ? x0 + 2 * p : -1, xb = p < 8 ? x0 + 2 * p + 1 : p == 9 ? x0 - 1 : -1;
      const int c = c0 + 8 * cg;
      const bool in = it < IX && gy >= 0 && gy < d.ny && gz >= 0 && gz < d.nz;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int gx = h ? xb : xa;
        px[s][h] = zero;
        if (in && gx >= 0 && gx < d.nx) {
          const uint16_t* src = c < ca ? XA + (long)(gx + d.nx * (gy + d.ny * gz)) * sa + c
                                       : XB + (long)((gx >> 1) + cnx * ((gy >> 1) + cny * (gz >> 1))) * sb + (c - ca);
          px[s][h] = *reinterpret_cast<const u32x4*>(src);
        }
      }
    }
#pragma unroll
    for (int s = 0; s < SY; ++s) {
      const int it = tid + NT * s, cg = it % GY, p = it / GY % 8, row = it / (GY * 8);
      const int gx = x0 + 2 * p, gy = y0 + row % kWY, gz = z0 + row / kWY;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        py[s][h] = zero;   // a voxel outside the grid contributes nothing
        if (it < IY && gx + h < d.nx && gy < d.ny && gz < d.nz)
          py[s][h] = *reinterpret_cast<const u32x4*>(dY + (long)(gx + h + d.nx * (gy + d.ny * gz)) * COUT + 8 * cg);
      }
    }
  };
  // two voxels' eight channels to eight rows, one dword (both voxels) each
  auto put8 = [](uint32_t* o, int stride, const u32x4& a, const u32x4& b) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      o[(2 * e) * stride] = (a[e] & 0xFFFFu) | (b[e] << 16);
      o[(2 * e + 1) * stride] = (a[e] >> 16) | (b[e] & 0xFFFF0000u);
    }
  };
  auto put = [&]() {
#pragma unroll
    for (int s = 0; s < SX; ++s) {
      const int it = tid + NT * s, cg = it % GX, p = it / GX % 10, row = it / (GX * 10);
      if (it < IX) put8(lx + 8 * cg * kWChan + row * kWRow + (p == 9 ? 11 : p), kWChan, px[s][0], px[s][1]);
    }
#pragma unroll
    for (int s = 0; s < SY; ++s) {
      const int it = tid + NT * s, cg = it % GY, p = it / GY % 8, row = it / (GY * 8);
      if (it < IY) put8(ly + 8 * cg * kWdY + row * 8 + p, kWdY, py[s][0], py[s][1]);
    }
  };
  f32x4 acc[3][3][NO], accb[NO];
#pragma unroll
  for (int o = 0; o < NO; ++o) {
    accb[o] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < 9; ++q) acc[q / 3][q % 3][o] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const bool bias = dz == 1 && blockIdx.y == 0;   // this wave also sums dY itself
  const bf16x8 ones = as_bf16x8(u32x4{0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u});
  const uint32_t* xw = lx + r * kWChan;
  int t = blockIdx.x;
  if (t < tiles) fetch(t);
  for (; t < tiles; t += gridDim.x) {
    put();
    __syncthreads();
    if (t + (int)gridDim.x < tiles) fetch(t + gridDim.x);
    // 32 voxels a step: row pair 2 (s & 1) of plane s >> 1, x half kg & 1
    // (not unrolled: with four steps' reads in flight the wider layers spilled)
#pragma unroll 1
    for (int s = 0; s < 4; ++s) {
      const int z = s >> 1, y = 2 * (s & 1) + (kg >> 1);
      bf16x8 a[NO];
#pragma unroll
      for (int o = 0; o < NO; ++o)
        a[o] = as_bf16x8(*reinterpret_cast<const u32x4*>(ly + (16 * o + r) * kWdY + (z * kWY + y) * 8 + 4 * (kg & 1)));
      if (bias)
#pragma unroll
        for (int o = 0; o < NO; ++o) accb[o] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[o], ones, accb[o], 0, 0, 0);
#pragma unroll
      for (int dy = 0; dy < 3; ++dy) {
        const uint32_t* row = xw + ((z + dz) * (kWY + 2) + y + dy) * kWRow;
        const u32x4 m = *reinterpret_cast<const u32x4*>(row + 4 * (kg & 1));
        const uint32_t lo = row[(kg & 1) ? 3 : 11], hi = row[(kg & 1) ? 8 : 4];
        // the fragments one voxel to the left (dx = 0) and right (dx = 2)
        const u32x4 left = {__builtin_amdgcn_alignbit(m[0], lo, 16), __builtin_amdgcn_alignbit(m[1], m[0], 16),
                            __builtin_amdgcn_alignbit(m[2], m[1], 16), __builtin_amdgcn_alignbit(m[3], m[2], 16)};
        const u32x4 right = {left[1], left[2], left[3], __builtin_amdgcn_alignbit(hi, m[3], 16)};
#pragma unroll
        for (int o = 0; o < NO; ++o) {
          acc[dy][0][o] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[o], as_bf16x8(left), acc[dy][0][o], 0, 0, 0);
          acc[dy][1][o] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[o], as_bf16x8(m), acc[dy][1][o], 0, 0, 0);
          acc[dy][2][o] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[o], as_bf16x8(right), acc[dy][2][o], 0, 0, 0);
        }
      }
    }
    __syncthreads();
  }
  // D lane layout: column (input channel) r, rows (output channels) 4 kg + i;
  // the partial is laid out as the gradient, weights then biases
  float* out = part + (size_t)blockIdx.x * (27 * COUT * CIN + COUT);
#pragma unroll
  for (int o = 0; o < NO; ++o)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int co = 16 * o + 4 * kg + i;
#pragma unroll
      for (int q = 0; q < 9; ++q) out[(size_t)(co * 27 + dz * 9 + q) * CIN + c0 + r] = acc[q / 3][q % 3][o][i];
      if (bias && r == 0) out[27 * COUT * CIN + co] = accb[o][i];
    }
}

// out[q] = sum over b of part[b n + q], b = 0 .. nblk - 1: 32 values per block,
// eight threads per value (b modulo 8, in order) whose sums are added in order.
// Bound by the latency of a thread's up to 32 loads, so eight are in flight at
// once, in the same order of additions: 256 partials of 20.8 k values 9.2 -> 4.8 us
// (median of the six sums of a training step at 128 x 64 x 64).
__global__ void __launch_bounds__(256) k_part_reduce(const float* __restrict__ part, int nblk, int n,
                                                     float* __restrict__ out) {
  __shared__ float sm[8][33];
  const int c = threadIdx.x & 31, w = threadIdx.x >> 5, q = blockIdx.x * 32 + c;
  float s = 0.f;
  if (q < n)
  {
    const float* p = part + q;
    int b = w;
    for (; b + 56 < nblk; b += 64) {
      float v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = p[(size_t)(b + 8 * i) * n];
#pragma unroll
      for (int i = 0; i < 8; ++i) s += v[i];
    }
    for (; b < nblk; b += 8) s += p[(size_t)b * n];
  }
  sm[w][c] = s;
  __syncthreads();
  if (w == 0 && q < n) {
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) t += sm[i][c];
    out[q] = t;
  }
}

// ------------------------------------------------------- resampling, head
// 2x2x2 average of a fine tensor (channel stride is, offset io) into a dense
// coarse one; a thread takes 8 channels of one coarse voxel
__global__ void k_pool(VDims fine, const uint16_t* __restrict__ in, int is, int io, int C,
                       uint16_t* __restrict__ out) {
  const VDims c{fine.nx / 2, fine.ny / 2, fine.nz / 2};
  const long q = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const int groups = C / 8;
  if (q >= vox_count(c) * groups) return;
  const int g = (int)(q % groups);
  const long v = q / groups;
  const int X = (int)(v % c.nx), Y = (int)((v / c.nx) % c.ny), Z = (int)(v / ((long)c.nx * c.ny));
  float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int k = 0; k < 2; ++k)
    for (int j = 0; j < 2; ++j)
      for (int i = 0; i < 2; ++i) {
        const long f = (2L * X + i) + (long)fine.nx * ((2L * Y + j) + (long)fine.ny * (2L * Z + k));
        const u32x4 w = *reinterpret_cast<const u32x4*>(in + f * is + io + 8 * g);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          s[2 * e] += __uint_as_float(w[e] << 16);
          s[2 * e + 1] += __uint_as_float(w[e] & 0xFFFF0000u);
        }
      }
  u32x4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = (uint32_t)f2bf(s[2 * e] * 0.125f) | ((uint32_t)f2bf(s[2 * e + 1] * 0.125f) << 16);
  *reinterpret_cast<u32x4*>(out + v * C + 8 * g) = o;
}

// delta = b + sum_c w_c a_c (1x1x1 head, FP32 out)
__global__ void k_head(long nv, const uint16_t* __restrict__ a, const float* __restrict__ w,
                       const float* __restrict__ b, float* __restrict__ delta) {
  const long v = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= nv) return;
  float s = b[0];
#pragma unroll
  for (int c = 0; c < 16; ++c) s += w[c] * bf2f(a[v * 16 + c]);
  delta[v] = s;
}

// ------------------------------------------------------------- backward
// The elementwise kernels of the backward pass take eight channels of a voxel
// per thread (16-byte accesses).
__device__ __forceinline__ void unpack8(const u32x4& w, float (&f)[8]) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    f[2 * e] = __uint_as_float(w[e] << 16);
    f[2 * e + 1] = __uint_as_float(w[e] & 0xFFFF0000u);
  }
}
__device__ __forceinline__ u32x4 pack8(const float (&f)[8]) {
  u32x4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = (uint32_t)f2bf(f[2 * e]) | ((uint32_t)f2bf(f[2 * e + 1]) << 16);
  return o;
}
__device__ __forceinline__ u32x4 ld8(const uint16_t* __restrict__ p) { return *reinterpret_cast<const u32x4*>(p); }

// d5 = ddelta w_c (a_c > 0), and per block the partials of the head's gradient,
// (sum ddelta a_c for c < 16, sum ddelta), from the same read of a.  A thread
// keeps to one half of the channels (its stride is even); lanes of one half are
// added by exchanges, the block's waves in order.  Bound by the bytes of a and d5
// with few waves per block's tail: four loads of a thread are in flight.
// As two kernels, the second one thread's 256 sums long: 9.8 + 7.0 us at
// 128 x 64 x 64, this one 8.9 us.
__global__ void __launch_bounds__(256) k_head_bwd(long nv, const float* __restrict__ dd,
                                                  const uint16_t* __restrict__ a, const float* __restrict__ w,
                                                  uint16_t* __restrict__ d5, float* __restrict__ part) {
  __shared__ float sm[4][17];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane & 1;
  const long n = 2 * nv, step = 256L * gridDim.x;
  float wv[8], s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, sd = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) wv[e] = w[8 * g + e];
  for (long q0 = (long)blockIdx.x * 256 + threadIdx.x; q0 < n; q0 += 4 * step) {
    u32x4 in[4];
    float gv[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const long q = q0 + u * step < n ? q0 + u * step : q0;   // (past the end: loaded, not used)
      in[u] = ld8(a + 8 * q);
      gv[u] = dd[q >> 1];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const long q = q0 + u * step;
      if (q >= n) break;
      float av[8], o[8];
      unpack8(in[u], av);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        o[e] = av[e] > 0.f ? gv[u] * wv[e] : 0.f;
        s[e] += gv[u] * av[e];
      }
      sd += gv[u];
      *reinterpret_cast<u32x4*>(d5 + 8 * q) = pack8(o);
    }
  }
#pragma unroll
  for (int m = 2; m < 64; m <<= 1) {
#pragma unroll
    for (int e = 0; e < 8; ++e) s[e] += __shfl_xor(s[e], m);
    sd += __shfl_xor(sd, m);
  }
  if (lane < 2) {
#pragma unroll
    for (int e = 0; e < 8; ++e) sm[wave][8 * g + e] = s[e];
    if (lane == 0) sm[wave][16] = sd;
  }
  __syncthreads();
  if (threadIdx.x < 17)
    part[(size_t)blockIdx.x * 17 + threadIdx.x] =
        ((sm[0][threadIdx.x] + sm[1][threadIdx.x]) + sm[2][threadIdx.x]) + sm[3][threadIdx.x];
}

// d (coarse, dense C) = (sum over the 8 children of dC[child][oo + c]) (a > 0)
__global__ void k_up_bwd_mask(VDims coarse, const uint16_t* __restrict__ dC, int os, int oo, int C,
                              const uint16_t* __restrict__ a, uint16_t* __restrict__ d) {
  const VDims f{coarse.nx * 2, coarse.ny * 2, coarse.nz * 2};
  const long q = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const int groups = C / 8;
  if (q >= vox_count(coarse) * groups) return;
  const int g = (int)(q % groups);
  const long v = q / groups;
  const int X = (int)(v % coarse.nx), Y = (int)((v / coarse.nx) % coarse.ny),
            Z = (int)(v / ((long)coarse.nx * coarse.ny));
  u32x4 in[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const long fv = (2L * X + (c & 1)) + (long)f.nx * ((2L * Y + (c >> 1 & 1)) + (long)f.ny * (2L * Z + (c >> 2)));
    in[c] = ld8(dC + fv * os + oo + 8 * g);
  }
  float av[8], s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  unpack8(ld8(a + v * C + 8 * g), av);
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    float t[8];
    unpack8(in[c], t);
#pragma unroll
    for (int e = 0; e < 8; ++e) s[e] += t[e];
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) s[e] = av[e] > 0.f ? s[e] : 0.f;
  *reinterpret_cast<u32x4*>(d + v * C + 8 * g) = pack8(s);
}

// d (fine, dense C) = (dC[v][c] (stride os) + dp[parent][c] / 8) (a[v][c] > 0, dense)
__global__ void k_skip_mask(VDims fine, const uint16_t* __restrict__ dC, int os, const uint16_t* __restrict__ dp,
                            const uint16_t* __restrict__ a, int C, uint16_t* __restrict__ d) {
  const VDims c{fine.nx / 2, fine.ny / 2, fine.nz / 2};
  const long q = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const int groups = C / 8;
  if (q >= vox_count(fine) * groups) return;
  const int g = (int)(q % groups);
  const long v = q / groups;
  const int x = (int)(v % fine.nx), y = (int)((v / fine.nx) % fine.ny), z = (int)(v / ((long)fine.nx * fine.ny));
  const long p = (x / 2) + (long)c.nx * ((y / 2) + (long)c.ny * (z / 2));
  float av[8], dv[8], pv[8], o[8];
  unpack8(ld8(a + v * C + 8 * g), av);
  unpack8(ld8(dC + v * os + 8 * g), dv);
  unpack8(ld8(dp + p * C + 8 * g), pv);
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = av[e] > 0.f ? dv[e] + 0.125f * pv[e] : 0.f;
  *reinterpret_cast<u32x4*>(d + v * C + 8 * g) = pack8(o);
}

// The bfloat16 copies of the master weights in one launch, in the order the
// convolutions' lanes read them: a fragment's 64 pieces of 8 channels (1 KB) are
// consecutive.  From rows of 27 CIN channels a fragment touched 16 lines: 64 x
// 32 x 32 inference 41.9 -> 35.9 us, 256 x 128 x 128 446 -> 420, a 128 x 64 x 64
// training step 500 -> 475.  blockIdx.y: the layer l of W, then l of
// W'[ci][26 - tap][co] = W[co][tap][ci] for the input gradient, and last the first
// layer's compact form, k = 4 tap + ci.  A thread fills one piece.
//   k_conv:    piece ((t NC + c) 14 + p) 64 + lane: output 16 t + lane % 16, tap
//              2 p + lane / 32 (the 28th zero), inputs 16 c + 8 (lane / 16 % 2) ..
//   k_conv_cm: piece ((t NC + c) 27 + tap) 64 + lane: inputs 32 c + 8 (lane / 16) ..
struct WeightCopies {
  const float* w[5];
  uint16_t *wf[5], *wt[5], *wc0;
  int cin[5], cout[5];
  int cm;   // the layer that k_conv_cm takes (-1: none)
};
__global__ void __launch_bounds__(256) k_weight_copies(WeightCopies W) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x, l = blockIdx.y % 5;
  const int lane = q & 63, r = lane & 15, kg = lane >> 4;
  u32x4 o = {0u, 0u, 0u, 0u};
  uint16_t v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  uint16_t* out;
  if (blockIdx.y == 10) {
    if (q >= 4 * 64) return;
    out = W.wc0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int k = 32 * (q >> 6) + 8 * kg + e;
      if (k < 108) v[e] = f2bf(W.w[0][(r * 27 + k / 4) * 16 + k % 4]);
    }
  } else {
    const bool back = blockIdx.y >= 5, cm = !back && l == W.cm;
    const int cin = back ? W.cout[l] : W.cin[l], cout = back ? W.cin[l] : W.cout[l];
    const int nc = cin / (cm ? 32 : 16), np = cm ? 27 : 14;
    if (q >= cout / 16 * nc * np * 64) return;
    out = back ? W.wt[l] : W.wf[l];
    const int p = (q >> 6) % np, tc = (q >> 6) / np, c = tc % nc, co = 16 * (tc / nc) + r;
    const int tap = cm ? p : 2 * p + (kg >> 1), ci = cm ? 32 * c + 8 * kg : 16 * c + 8 * (kg & 1);
    if (tap < 27) {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        v[e] = f2bf(back ? W.w[l][((ci + e) * 27 + 26 - tap) * cout + co] : W.w[l][(co * 27 + tap) * cin + ci + e]);
    }
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = (uint32_t)v[2 * e] | ((uint32_t)v[2 * e + 1] << 16);
  reinterpret_cast<u32x4*>(out)[q] = o;
}

// Adam with bias correction; padded (always-zero-gradient) entries stay put
__global__ void k_adam(float* __restrict__ th, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, long n, float lr, float c1, float c2) {
  const long q = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= n) return;
  const float gq = g[q];
  const float mq = 0.9f * m[q] + 0.1f * gq;
  const float vq = 0.999f * v[q] + 0.001f * gq * gq;
  m[q] = mq;
  v[q] = vq;
  th[q] -= lr * (mq / c1) / (sqrtf(vq / c2) + 1e-8f);
}

// ------------------------------------------------ features, loss, guess
// four input channels (channel-first FP32): rhs h^2 rho_w / P0, the
// log-density fraction, p_prev / P0 and the residual (b - A p_prev) h^2 rho_w / P0
// (PACK: as k_pack_input leaves them)
__device__ __forceinline__ u32x2 pack4(float a, float b, float c, float d) {
  return u32x2{(uint32_t)f2bf(a) | ((uint32_t)f2bf(b) << 16), (uint32_t)f2bf(c) | ((uint32_t)f2bf(d) << 16)};
}
template <bool PACK>
__global__ void k_features(long nv, double s, double lr_w, double inv_lr, double inv_P0,
                           const double* __restrict__ b, const double* __restrict__ rho,
                           const double* __restrict__ pprev, const double* __restrict__ Ap,
                           float* __restrict__ feat) {
  const long v = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= nv) return;
  const double bb = b[v];
  const float f0 = (float)(bb * s), f1 = (float)((log(rho[v]) - lr_w) * inv_lr);
  const float f2 = (float)(pprev[v] * inv_P0), f3 = (float)((bb - Ap[v]) * s);
  if (PACK) {
    reinterpret_cast<u32x2*>(feat)[v] = pack4(f0, f1, f2, f3);
    return;
  }
  feat[v] = f0;
  feat[nv + v] = f1;
  feat[2 * nv + v] = f2;
  feat[3 * nv + v] = f3;
}

// channel-first FP32 features -> bfloat16, the four channels of a voxel together
// (the inference input: the first layer reads a voxel once per tile and halo,
// 2.5 times, which at 256 x 128 x 128 cost it 82 us from the FP32 planes)
__global__ void k_pack_input(long nv, const float* __restrict__ feat, u32x2* __restrict__ xin) {
  const long v = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (v < nv) xin[v] = pack4(feat[v], feat[nv + v], feat[2 * nv + v], feat[3 * nv + v]);
}

// channel-first FP32 features -> channels-last bfloat16 input, padded to 16
__global__ void k_set_input(long nv, const float* __restrict__ feat, uint16_t* __restrict__ x0) {
  const long v = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= nv) return;
  u32x4 lo = {0u, 0u, 0u, 0u};
  lo[0] = (uint32_t)f2bf(feat[v]) | ((uint32_t)f2bf(feat[nv + v]) << 16);
  lo[1] = (uint32_t)f2bf(feat[2 * nv + v]) | ((uint32_t)f2bf(feat[3 * nv + v]) << 16);
  u32x4* o = reinterpret_cast<u32x4*>(x0 + v * 16);
  o[0] = lo;
  o[1] = u32x4{0u, 0u, 0u, 0u};
}

// p = p_prev + P0 delta
__global__ void k_apply_delta(long nv, const double* __restrict__ pprev, const float* __restrict__ delta,
                              double P0, double* __restrict__ p) {
  const long v = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (v < nv) p[v] = pprev[v] + P0 * (double)delta[v];
}

// target delta = (p* - p_prev) / P0
__global__ void k_target(long nv, const double* __restrict__ p, const double* __restrict__ pprev, double inv_P0,
                         float* __restrict__ t) {
  const long v = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (v < nv) t[v] = (float)((p[v] - pprev[v]) * inv_P0);
}

// y = A x in FP32 on the finest grid (sum_f beta_f (x_c - x_nb), open top
// face coupling to -x_c; the 1/h^2 factor cancels in the loss ratio)
__global__ void __launch_bounds__(256) k_spmv_f32(VDims d, const float* __restrict__ bx,
                                                  const float* __restrict__ by, const float* __restrict__ bz,
                                                  const float* __restrict__ x, float* __restrict__ y) {
  const long c = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= vox_count(d)) return;
  const int i = (int)(c % d.nx), j = (int)((c / d.nx) % d.ny), k = (int)(c / ((long)d.nx * d.ny));
  const long sxy = (long)d.nx * d.ny;
  const long fx = i + (long)(d.nx + 1) * (j + (long)d.ny * k);
  const long fy = i + (long)d.nx * (j + (long)(d.ny + 1) * k);
  const float xc = x[c];
  float a = 0.f;
  if (i > 0) a += bx[fx] * (xc - x[c - 1]);
  if (i < d.nx - 1) a += bx[fx + 1] * (xc - x[c + 1]);
  if (j > 0) a += by[fy] * (xc - x[c - d.nx]);
  if (j < d.ny - 1) a += by[fy + d.nx] * (xc - x[c + d.nx]);
  if (k > 0) a += bz[c] * (xc - x[c - sxy]);
  a += (k < d.nz - 1) ? bz[c + sxy] * (xc - x[c + sxy]) : 2.f * bz[c + sxy] * xc;
  y[c] = a;
}

// e = t - delta (the guess's error in units of P0)
__global__ void k_err(long nv, const float* __restrict__ delta, const float* __restrict__ t, float* __restrict__ e) {
  const long v = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (v < nv) e[v] = t[v] - delta[v];
}

// per-block (sum e Ae, sum t At)
__global__ void __launch_bounds__(256) k_loss_part(long nv, const float* __restrict__ e, const float* __restrict__ Ae,
                                                   const float* __restrict__ t, const float* __restrict__ At,
                                                   double* __restrict__ part) {
  __shared__ double sa[256], sb[256];
  double a = 0.0, b = 0.0;
  for (long v = (long)blockIdx.x * 256 + threadIdx.x; v < nv; v += (long)gridDim.x * 256) {
    a += (double)e[v] * (double)Ae[v];
    b += (double)t[v] * (double)At[v];
  }
  sa[threadIdx.x] = a;
  sb[threadIdx.x] = b;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
      sa[threadIdx.x] += sa[threadIdx.x + s];
      sb[threadIdx.x] += sb[threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = sa[0];
    part[2 * blockIdx.x + 1] = sb[0];
  }
}

// out[0] = loss = e'Ae / t'At, out[1] = -2 / t'At (one wave; lane q sums partials
// q, q + 64, .. in order, then a fixed tree)
__global__ void k_loss_fin(const double* __restrict__ part, int nblk, double* __restrict__ out) {
  double a = 0.0, b = 0.0;
  for (int q = threadIdx.x; q < nblk; q += 64) {
    a += part[2 * q];
    b += part[2 * q + 1];
  }
  for (int o = 32; o > 0; o >>= 1) {
    a += __shfl_down(a, o, 64);
    b += __shfl_down(b, o, 64);
  }
  if (threadIdx.x != 0) return;
  out[0] = b > 0.0 ? a / b : 0.0;
  out[1] = b > 0.0 ? -2.0 / b : 0.0;
}

// dL/ddelta = -2 A e / t'At  (A symmetric)
__global__ void k_dloss(long nv, const float* __restrict__ Ae, const double* __restrict__ out, float* __restrict__ dd) {
  const long v = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (v < nv) dd[v] = (float)(out[1] * (double)Ae[v]);
}

__global__ void k_finite_count(long n, const float* __restrict__ a, int* __restrict__ bad) {
  const long q = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (q < n && !isfinite(a[q])) atomicAdd(bad, 1);
}

inline dim3 g1(long n, int b = 256) { return dim3((unsigned)((n + b - 1) / b)); }

}  // namespace

// ==================================================================== the net
// conv layers 1..5 (index 0..4): padded C_in, C_out, and the head (16 -> 1)
static const int kCin[5] = {16, 16, 32, 96, 48};
static const int kCinTrue[5] = {4, 16, 32, 96, 48};
static const int kCout[5] = {16, 32, 64, 32, 16};

}  // namespace nsk

using namespace nsk;

struct ns_net {
  VDims res0, res1, res2;
  long v0, v1, v2;
  int training;
  hipStream_t st;
  // internal parameter layout: per conv layer W[co][tap][ci_pad] then b[co];
  // then the head w[16], b[1]
  size_t np;
  size_t ow[5], ob[5], ohw, ohb;
  float *theta, *m, *v, *g;
  uint16_t *wf[5], *wt[5];
  uint16_t* wc0;   // first layer, compact K (inference)
  uint16_t *x0, *C1, *p1, *C2, *p2, *a3, *a4, *a5;
  float* delta;
  // backward
  float* dd;
  uint16_t *d5, *dC1, *d4, *dC2, *d3, *dp2, *d2, *dp1, *d1;
  float* wpart;
  size_t wpart_elems;
  double* red;
  int* bad;
  double* host;
  // learned-guess staging
  float* feat;
  float* target;
  float* eb;
  double* pprev;
  double* Ap;
  int step;
  char err[256];
};

namespace {

constexpr size_t kAlignN = 256;

struct NetCarve {
  char* base;
  size_t off;
  template <typename T>
  T* take(size_t count) {
    off = (off + kAlignN - 1) / kAlignN * kAlignN;
    T* p = base ? reinterpret_cast<T*>(base + off) : nullptr;
    off += count * sizeof(T);
    return p;
  }
};

// blocks of the head's backward kernel: two per compute unit, of at least 1024
// voxels (eight 16-byte pieces a thread)
int head_blocks(long v0) { return (int)std::min<long>((v0 + 1023) / 1024, 512); }

// Blocks of a layer's weight gradient per 16 input channels: enough
// to fill the chip's 256 compute units with one block each, few enough that
// the partials, written and read once, stay within 24 MB.  The 16 -> 16 layer has
// no second block on a unit to work while one waits at a barrier: it takes two
// blocks a unit where each still has four tiles (its partials are the smallest,
// so the room is the same): 128 x 64 x 64 38.0 -> 25.4 us.
int wgrad_tiles(int nx, int ny, int nz) {
  return (nx + kWX - 1) / kWX * ((ny + kWY - 1) / kWY) * ((nz + kWZ - 1) / kWZ);
}
int wgrad_blocks(int nx, int ny, int nz, int cin, int cout) {
  const long most = (24L << 20) / (4L * (27L * cin * cout + cout)), tiles = wgrad_tiles(nx, ny, nz);
  const long two = cin == 16 && cout == 16 ? std::min(tiles / 4, 512L) : 0;
  return (int)std::min(std::max(std::min(tiles, 256L), two), most);
}

size_t net_layout(ns_net* N, int nx, int ny, int nz, int training, char* base) {
  NetCarve cv{base, 0};
  VDims d0{nx, ny, nz}, d1{nx / 2, ny / 2, nz / 2}, d2{nx / 4, ny / 4, nz / 4};
  const long v0 = (long)nx * ny * nz, v1 = v0 / 8, v2 = v0 / 64;
  size_t np = 0, ow[5], ob[5];
  for (int l = 0; l < 5; ++l) {
    ow[l] = np;
    np += (size_t)kCout[l] * 27 * kCin[l];
    ob[l] = np;
    np += kCout[l];
  }
  const size_t ohw = np;
  np += 16;
  const size_t ohb = np;
  np += 1;
  float* theta = cv.take<float>(np);
  float *m = nullptr, *v = nullptr, *g = nullptr;
  if (training) {
    m = cv.take<float>(np);
    v = cv.take<float>(np);
    g = cv.take<float>(np);
  }
  uint16_t *wf[5], *wt[5];
  for (int l = 0; l < 5; ++l) {
    wf[l] = cv.take<uint16_t>((size_t)kCout[l] * 28 * kCin[l]);
    wt[l] = cv.take<uint16_t>((size_t)kCout[l] * 28 * kCin[l]);
  }
  uint16_t* wc0 = cv.take<uint16_t>(16 * 128);
  uint16_t* x0 = cv.take<uint16_t>(v0 * 16);
  uint16_t* C1 = cv.take<uint16_t>(v0 * 48);
  uint16_t* p1 = cv.take<uint16_t>(v1 * 16);
  uint16_t* C2 = cv.take<uint16_t>(v1 * 96);
  uint16_t* p2 = cv.take<uint16_t>(v2 * 32);
  uint16_t* a3 = cv.take<uint16_t>(v2 * 64);
  uint16_t* a4 = cv.take<uint16_t>(v1 * 32);
  uint16_t* a5 = cv.take<uint16_t>(v0 * 16);
  float* delta = cv.take<float>(v0);
  float* feat = cv.take<float>(4 * v0);
  float* target = cv.take<float>(v0);
  float* eb = cv.take<float>(3 * v0);   // e, A e, A t of the loss
  double* pprev = cv.take<double>(v0);
  double* Ap = cv.take<double>(v0);
  double* red = cv.take<double>(4096);
  int* bad = cv.take<int>(64);
  float* dd = nullptr;
  uint16_t *d5 = nullptr, *dC1 = nullptr, *d4 = nullptr, *dC2 = nullptr, *d3 = nullptr, *dp2 = nullptr,
           *d2p = nullptr, *dp1 = nullptr, *d1p = nullptr;
  float* wpart = nullptr;
  size_t wpart_elems = 0;
  if (training) {
    dd = cv.take<float>(v0);
    d5 = cv.take<uint16_t>(v0 * 16);
    dC1 = cv.take<uint16_t>(v0 * 48);
    d4 = cv.take<uint16_t>(v1 * 32);
    dC2 = cv.take<uint16_t>(v1 * 96);
    d3 = cv.take<uint16_t>(v2 * 64);
    dp2 = cv.take<uint16_t>(v2 * 32);
    d2p = cv.take<uint16_t>(v1 * 32);
    dp1 = cv.take<uint16_t>(v1 * 16);
    d1p = cv.take<uint16_t>(v0 * 16);
    // the largest partials over the layers, and the head's
    for (int l = 0; l < 5; ++l) {
      const int sh = (l == 0 || l == 4) ? 0 : (l == 1 || l == 3) ? 1 : 2;
      const size_t nb = (size_t)wgrad_blocks(nx >> sh, ny >> sh, nz >> sh, kCin[l], kCout[l]);
      wpart_elems = std::max(wpart_elems, nb * (27 * (size_t)kCout[l] * kCin[l] + kCout[l]));
    }
    wpart_elems = std::max(wpart_elems, (size_t)head_blocks(v0) * 17);
    wpart = cv.take<float>(wpart_elems);
  }
  if (N) {
    N->res0 = d0;
    N->res1 = d1;
    N->res2 = d2;
    N->v0 = v0;
    N->v1 = v1;
    N->v2 = v2;
    N->training = training;
    N->np = np;
    for (int l = 0; l < 5; ++l) {
      N->ow[l] = ow[l];
      N->ob[l] = ob[l];
      N->wf[l] = wf[l];
      N->wt[l] = wt[l];
    }
    N->ohw = ohw;
    N->ohb = ohb;
    N->theta = theta;
    N->m = m;
    N->v = v;
    N->g = g;
    N->wc0 = wc0;
    N->x0 = x0;
    N->C1 = C1;
    N->p1 = p1;
    N->C2 = C2;
    N->p2 = p2;
    N->a3 = a3;
    N->a4 = a4;
    N->a5 = a5;
    N->delta = delta;
    N->feat = feat;
    N->target = target;
    N->eb = eb;
    N->pprev = pprev;
    N->Ap = Ap;
    N->red = red;
    N->bad = bad;
    N->dd = dd;
    N->d5 = d5;
    N->dC1 = dC1;
    N->d4 = d4;
    N->dC2 = dC2;
    N->d3 = d3;
    N->dp2 = dp2;
    N->d2 = d2p;
    N->dp1 = dp1;
    N->d1 = d1p;
    N->wpart = wpart;
    N->wpart_elems = wpart_elems;
  }
  return cv.off + kAlignN;
}

ns_status nfail(ns_net* N, ns_status s, const char* msg) {
  if (N) snprintf(N->err, sizeof(N->err), "%s", msg);
  return s;
}

// Where a level has fewer than 128 tiles of every output channel, tiles of two rows
// and 16 channels: 64 x 32 x 32 inference, 32 -> 64 channels on 4 blocks 13.0
// us, on 32 6.2; 96 -> 32 on 16 blocks 27.7 us, on 128 14.4.  With 256 tiles
// the smaller ones lose (the same grid's 48 -> 16 layer 10.0 us, 12.0 so).
inline bool few_blocks(const dim3& g) { return (long)g.x * g.y * g.z < 128; }
// Where tiles of eight rows leave four blocks per compute unit, the layers of 16
// output channels take them: a row's fragment feeds one MFMA there, and eight of
// them per tap pair cover the LDS latency that four do not (256 x 128 x 128: 48 ->
// 16 channels 295 -> 245 us; 96 x 64 x 48, on 576 blocks, 80 us in all against 82)
inline bool many_blocks(const VDims& d) {
  return (long)((d.nx + kTX - 1) / kTX) * ((d.ny + 7) / 8) * ((d.nz + kTZ - 1) / kTZ) >= 1024;
}

template <int CIN, int COUT, int EPI, bool POOL = false>
void conv(const ns_net* N, VDims d, const uint16_t* XA, int sa, int ca, const uint16_t* XB, int sb,
          const uint16_t* W, const float* bias, uint16_t* Y, int ys, int yo, const float* hw = nullptr,
          const float* hb = nullptr, float* delta = nullptr, float* delta2 = nullptr, uint16_t* P = nullptr) {
  constexpr int NT = COUT / 16;
  dim3 grid((d.nx + kTX - 1) / kTX, (d.ny + kTY - 1) / kTY, (d.nz + kTZ - 1) / kTZ);
  if (EPI == 2 && many_blocks(d)) {
    grid.y = (d.ny + 7) / 8;
    hipLaunchKernelGGL((k_conv<CIN, COUT, EPI, EPI == 2 ? 8 : kTY, NT, POOL>), grid, dim3(256), 0, N->st, d, XA, sa, ca,
                       XB, sb, W, bias, Y, ys, yo, hw, hb, delta, delta2, P);
    return;
  }
  if (!few_blocks(grid)) {
    hipLaunchKernelGGL((k_conv<CIN, COUT, EPI, kTY, NT, POOL>), grid, dim3(256), 0, N->st, d, XA, sa, ca, XB, sb, W, bias,
                       Y, ys, yo, hw, hb, delta, delta2, P);
    return;
  }
  grid.x *= NT;
  grid.y = (d.ny + 1) / 2;
  hipLaunchKernelGGL((k_conv<CIN, COUT, EPI, 2, 1, POOL>), grid, dim3(256), 0, N->st, d, XA, sa, ca, XB, sb, W, bias, Y,
                     ys, yo, hw, hb, delta, delta2, P);
}

template <int CIN, int COUT>
void conv_cm(const ns_net* N, VDims d, const uint16_t* XA, int sa, int ca, const uint16_t* XB, int sb,
             const uint16_t* W, const float* bias, uint16_t* Y, int ys, int yo) {
  constexpr int NT = COUT / 16;
  dim3 grid((d.nx + kCX - 1) / kCX, (d.ny + kCY - 1) / kCY, (d.nz + kCZ - 1) / kCZ);
  if (!few_blocks(grid)) {
    hipLaunchKernelGGL((k_conv_cm<CIN, COUT, kCY, NT>), grid, dim3(256), 0, N->st, d, XA, sa, ca, XB, sb, W, bias, Y, ys,
                       yo);
    return;
  }
  grid.x *= NT;
  grid.y = (d.ny + 1) / 2;
  hipLaunchKernelGGL((k_conv_cm<CIN, COUT, 2, 1>), grid, dim3(256), 0, N->st, d, XA, sa, ca, XB, sb, W, bias, Y, ys, yo);
}

// bf16 copies (forward and flipped-transposed) of the FP32 master weights
void refresh_weights(ns_net* N) {
  WeightCopies W;
  int most = 4 * 64;
  for (int l = 0; l < 5; ++l) {
    W.w[l] = N->theta + N->ow[l];
    W.wf[l] = N->wf[l];
    W.wt[l] = N->wt[l];
    W.cin[l] = kCin[l];
    W.cout[l] = kCout[l];
    most = std::max(most, kCout[l] * 28 * kCin[l] / 8);
  }
  W.wc0 = N->wc0;
  W.cm = N->training ? -1 : 3;   // (training runs every layer on k_conv)
  hipLaunchKernelGGL(k_weight_copies, dim3((most + 255) / 256, 11), dim3(256), 0, N->st, W);
}

// Training forward: every activation the backward pass reads is stored (a1 and
// a2 dense, in the memory of C1 and C2, and the last activation a5).  As at
// inference the decoder convolutions read the skip and the coarse tensor
// directly, and so do their weight gradients.
void forward_train(ns_net* N) {
  const float* th = N->theta;
  uint16_t *a1 = N->C1, *a2 = N->C2;
  conv<16, 16, 0>(N, N->res0, N->x0, 16, 16, nullptr, 0, N->wf[0], th + N->ob[0], a1, 16, 0);
  hipLaunchKernelGGL(k_pool, g1(N->v1 * 2), dim3(256), 0, N->st, N->res0, a1, 16, 0, 16, N->p1);
  conv<16, 32, 0>(N, N->res1, N->p1, 16, 16, nullptr, 0, N->wf[1], th + N->ob[1], a2, 32, 0);
  hipLaunchKernelGGL(k_pool, g1(N->v2 * 4), dim3(256), 0, N->st, N->res1, a2, 32, 0, 32, N->p2);
  conv<32, 64, 0>(N, N->res2, N->p2, 32, 32, nullptr, 0, N->wf[2], th + N->ob[2], N->a3, 64, 0);
  conv<96, 32, 0>(N, N->res1, a2, 32, 32, N->a3, 64, N->wf[3], th + N->ob[3], N->a4, 32, 0);
  conv<48, 16, 0>(N, N->res0, a1, 16, 16, N->a4, 32, N->wf[4], th + N->ob[4], N->a5, 16, 0);
  hipLaunchKernelGGL(k_head, g1(N->v0), dim3(256), 0, N->st, N->v0, N->a5, th + N->ohw, th + N->ohb, N->delta);
}

// Inference forward: the decoder convolutions read the skip tensor and the
// coarse tensor directly (no upsampled copies), and the head is fused into
// the last convolution, so a5 is never stored.
// The input is the packed features in N->feat; delta2, if given, receives a copy
// of the result.
void forward_infer(ns_net* N, float* delta2) {
  const float* th = N->theta;
  uint16_t* a1 = N->C1;   // dense [v0][16] in the concatenation buffer's memory
  uint16_t* a2 = N->C2;   // dense [v1][32]
  {
    const VDims d = N->res0;
    const bool many = many_blocks(d);
    const int rows = many ? 8 : kTY;
    const dim3 grid((d.nx + kTX - 1) / kTX, (d.ny + rows - 1) / rows, (d.nz + kTZ - 1) / kTZ);
    hipLaunchKernelGGL(many ? k_conv_in<8> : k_conv_in<kTY>, grid, dim3(256), 0, N->st, d,
                       reinterpret_cast<const u32x2*>(N->feat), N->wc0, th + N->ob[0], a1, 16, N->p1);
  }
  conv<16, 32, 0, true>(N, N->res1, N->p1, 16, 16, nullptr, 0, N->wf[1], th + N->ob[1], a2, 32, 0, nullptr, nullptr,
                        nullptr, nullptr, N->p2);
  conv<32, 64, 0>(N, N->res2, N->p2, 32, 32, nullptr, 0, N->wf[2], th + N->ob[2], N->a3, 64, 0);
  conv_cm<96, 32>(N, N->res1, a2, 32, 32, N->a3, 64, N->wf[3], th + N->ob[3], N->a4, 32, 0);
  conv<48, 16, 2>(N, N->res0, a1, 16, 16, N->a4, 32, N->wf[4], th + N->ob[4], nullptr, 16, 0, th + N->ohw,
                  th + N->ohb, N->delta, delta2);
}

void forward(ns_net* N) {
  if (N->training)
    forward_train(N);
  else
    forward_infer(N, nullptr);
}

template <int CIN, int COUT>
void wgrad(ns_net* N, VDims d, const uint16_t* XA, int sa, int ca, const uint16_t* XB, int sb, const uint16_t* dY,
           int layer) {
  const int nb = wgrad_blocks(d.nx, d.ny, d.nz, CIN, COUT), n = 27 * COUT * CIN + COUT;
  hipLaunchKernelGGL((k_wgrad<CIN, COUT>), dim3(nb, CIN / kWCI), dim3(12 * kWCI), 0, N->st, d, XA, sa, ca, XB, sb, dY,
                     (d.nx + kWX - 1) / kWX, (d.ny + kWY - 1) / kWY, wgrad_tiles(d.nx, d.ny, d.nz), N->wpart);
  // (a layer's biases follow its weights in the gradient)
  hipLaunchKernelGGL(k_part_reduce, g1(n, 32), dim3(256), 0, N->st, N->wpart, nb, n, N->g + N->ow[layer]);
}

void backward(ns_net* N) {
  const float* th = N->theta;
  hipStream_t st = N->st;
  const uint16_t *a1 = N->C1, *a2 = N->C2;
  // head
  {
    const int nb = head_blocks(N->v0);
    hipLaunchKernelGGL(k_head_bwd, dim3(nb), dim3(256), 0, st, N->v0, N->dd, N->a5, th + N->ohw, N->d5, N->wpart);
    hipLaunchKernelGGL(k_part_reduce, dim3(1), dim3(256), 0, st, N->wpart, nb, 17, N->g + N->ohw);
  }
  // layer 5: input [a1, up(a4)] (48), output 16
  wgrad<48, 16>(N, N->res0, a1, 16, 16, N->a4, 32, N->d5, 4);
  conv<16, 48, 1>(N, N->res0, N->d5, 16, 16, nullptr, 0, N->wt[4], nullptr, N->dC1, 48, 0);
  hipLaunchKernelGGL(k_up_bwd_mask, g1(N->v1 * 4), dim3(256), 0, st, N->res1, N->dC1, 48, 16, 32, N->a4, N->d4);
  // layer 4: input [a2, up(a3)] (96), output 32
  wgrad<96, 32>(N, N->res1, a2, 32, 32, N->a3, 64, N->d4, 3);
  conv<32, 96, 1>(N, N->res1, N->d4, 32, 32, nullptr, 0, N->wt[3], nullptr, N->dC2, 96, 0);
  hipLaunchKernelGGL(k_up_bwd_mask, g1(N->v2 * 8), dim3(256), 0, st, N->res2, N->dC2, 96, 32, 64, N->a3, N->d3);
  // layer 3: input p2 (32), output 64
  wgrad<32, 64>(N, N->res2, N->p2, 32, 32, nullptr, 0, N->d3, 2);
  conv<64, 32, 1>(N, N->res2, N->d3, 64, 64, nullptr, 0, N->wt[2], nullptr, N->dp2, 32, 0);
  hipLaunchKernelGGL(k_skip_mask, g1(N->v1 * 4), dim3(256), 0, st, N->res1, N->dC2, 96, N->dp2, a2, 32, N->d2);
  // layer 2: input p1 (16), output 32
  wgrad<16, 32>(N, N->res1, N->p1, 16, 16, nullptr, 0, N->d2, 1);
  conv<32, 16, 1>(N, N->res1, N->d2, 32, 32, nullptr, 0, N->wt[1], nullptr, N->dp1, 16, 0);
  hipLaunchKernelGGL(k_skip_mask, g1(N->v0 * 2), dim3(256), 0, st, N->res0, N->dC1, 48, N->dp1, a1, 16, N->d1);
  // layer 1: input x0 (16), output 16
  wgrad<16, 16>(N, N->res0, N->x0, 16, 16, nullptr, 0, N->d1, 0);
}

// canonical parameter index (the flat order of ns_net_set_params and
// ns_net_get_params) <-> internal index
// conv layer l: canonical w[co][ci][kz][ky][kx] (ci < true C_in) then b[co];
// internal W[co][tap][ci_pad], tap = (kz * 3 + ky) * 3 + kx
template <typename F>
void for_each_param(const ns_net* N, F f) {
  size_t c = 0;
  for (int l = 0; l < 5; ++l) {
    const int cin = kCinTrue[l], cinp = kCin[l], cout = kCout[l];
    for (int co = 0; co < cout; ++co)
      for (int ci = 0; ci < cin; ++ci)
        for (int tap = 0; tap < 27; ++tap) f(c++, N->ow[l] + ((size_t)co * 27 + tap) * cinp + ci);
    for (int co = 0; co < cout; ++co) f(c++, N->ob[l] + co);
  }
  for (int q = 0; q < 16; ++q) f(c++, N->ohw + q);
  f(c++, N->ohb);
}

size_t canonical_count() {
  size_t n = 0;
  for (int l = 0; l < 5; ++l) n += (size_t)kCout[l] * kCinTrue[l] * 27 + kCout[l];
  return n + 17;
}

}  // namespace

// ------------------------------------------------------------------ ABI
extern "C" {

size_t ns_net_param_count(void) { return canonical_count(); }

size_t ns_net_workspace_bytes(int nx, int ny, int nz, int training) {
  if (nx < 4 || ny < 4 || nz < 4 || nx % 4 || ny % 4 || nz % 4) return 0;
  return net_layout(nullptr, nx, ny, nz, training ? 1 : 0, nullptr);
}

ns_status ns_net_create(int nx, int ny, int nz, int training, void* ws, size_t bytes, void* stream,
                        ns_net** out) {
  if (!out) return NS_EINVAL;
  *out = nullptr;
  if (nx < 4 || ny < 4 || nz < 4 || nx % 4 || ny % 4 || nz % 4) return NS_EINVAL;
  if (!ws || ((uintptr_t)ws % kAlignN) != 0) return NS_EINVAL;
  const size_t need = net_layout(nullptr, nx, ny, nz, training ? 1 : 0, nullptr);
  if (bytes < need) return NS_EINVAL;
  ns_net* N = new (std::nothrow) ns_net();
  if (!N) return NS_EINVAL;
  net_layout(N, nx, ny, nz, training ? 1 : 0, (char*)ws);
  N->st = (hipStream_t)stream;
  N->step = 0;
  if (hipHostMalloc((void**)&N->host, 8 * sizeof(double), hipHostMallocDefault) != hipSuccess) {
    delete N;
    return NS_EHIP;
  }
  if (hipMemsetAsync(N->theta, 0, N->np * sizeof(float), N->st) != hipSuccess) {
    (void)hipHostFree(N->host);
    delete N;
    return NS_EHIP;
  }
  if (training && (hipMemsetAsync(N->m, 0, N->np * sizeof(float), N->st) != hipSuccess ||
                   hipMemsetAsync(N->v, 0, N->np * sizeof(float), N->st) != hipSuccess ||
                   hipMemsetAsync(N->g, 0, N->np * sizeof(float), N->st) != hipSuccess)) {
    ns_net_destroy(N);
    return NS_EHIP;
  }
  *out = N;
  return NS_OK;
}

void ns_net_destroy(ns_net* N) {
  if (!N) return;
  if (N->host) (void)hipHostFree(N->host);
  delete N;
}

const char* ns_net_last_error(ns_net* N) { return N ? N->err : "null net"; }

ns_status ns_net_set_params(ns_net* N, const float* host_params, size_t n) {
  if (!N || !host_params) return NS_EINVAL;
  if (n != canonical_count()) return nfail(N, NS_EINVAL, "parameter count mismatch");
  std::vector<float> internal(N->np, 0.0f);
  for_each_param(N, [&](size_t c, size_t i) { internal[i] = host_params[c]; });
  if (hipMemcpyAsync(N->theta, internal.data(), N->np * sizeof(float), hipMemcpyHostToDevice, N->st) != hipSuccess)
    return nfail(N, NS_EHIP, "upload failed");
  if (N->training) {
    (void)hipMemsetAsync(N->m, 0, N->np * sizeof(float), N->st);
    (void)hipMemsetAsync(N->v, 0, N->np * sizeof(float), N->st);
    N->step = 0;
  }
  refresh_weights(N);
  if (hipStreamSynchronize(N->st) != hipSuccess) return nfail(N, NS_EHIP, "synchronise failed");
  return NS_OK;
}

static ns_status download(ns_net* N, const float* dev, float* host, size_t n) {
  if (n != canonical_count()) return nfail(N, NS_EINVAL, "parameter count mismatch");
  std::vector<float> internal(N->np);
  if (hipMemcpyAsync(internal.data(), dev, N->np * sizeof(float), hipMemcpyDeviceToHost, N->st) != hipSuccess ||
      hipStreamSynchronize(N->st) != hipSuccess)
    return nfail(N, NS_EHIP, "download failed");
  for_each_param(N, [&](size_t c, size_t i) { host[c] = internal[i]; });
  return NS_OK;
}

ns_status ns_net_get_params(ns_net* N, float* host_params, size_t n) {
  if (!N || !host_params) return NS_EINVAL;
  return download(N, N->theta, host_params, n);
}

ns_status ns_net_get_grads(ns_net* N, float* host_grads, size_t n) {
  if (!N || !host_grads) return NS_EINVAL;
  if (!N->training) return nfail(N, NS_ESTATE, "not a training net");
  return download(N, N->g, host_grads, n);
}

ns_status ns_net_set_input(ns_net* N, const float* feat4) {
  if (!N || !feat4) return NS_EINVAL;
  if (N->training)
    hipLaunchKernelGGL(k_set_input, g1(N->v0), dim3(256), 0, N->st, N->v0, feat4, N->x0);
  else
    hipLaunchKernelGGL(k_pack_input, g1(N->v0), dim3(256), 0, N->st, N->v0, feat4, reinterpret_cast<u32x2*>(N->feat));
  return hipGetLastError() == hipSuccess ? NS_OK : nfail(N, NS_EHIP, "launch failed");
}

ns_status ns_net_forward(ns_net* N, float* delta_out) {
  if (!N) return NS_EINVAL;
  if (!N->training) {
    forward_infer(N, delta_out);
  } else {
    forward_train(N);
    if (delta_out)
      if (hipMemcpyAsync(delta_out, N->delta, N->v0 * sizeof(float), hipMemcpyDeviceToDevice, N->st) != hipSuccess)
        return nfail(N, NS_EHIP, "copy failed");
  }
  return hipGetLastError() == hipSuccess ? NS_OK : nfail(N, NS_EHIP, "launch failed");
}

ns_status ns_net_train_step(ns_net* N, const float* feat4, const float* target, const float* bx, const float* by,
                            const float* bz, float lr, int update, double* loss) {
  if (!N || !feat4 || !target || !bx || !by || !bz) return NS_EINVAL;
  if (!N->training) return nfail(N, NS_ESTATE, "not a training net");
  hipStream_t st = N->st;
  hipLaunchKernelGGL(k_set_input, g1(N->v0), dim3(256), 0, st, N->v0, feat4, N->x0);
  forward(N);
  // energy-norm loss L = e'Ae / t'At with e = t - delta
  float *e = N->eb, *Ae = N->eb + N->v0, *At = N->eb + 2 * N->v0;
  const int nb = 256;
  hipLaunchKernelGGL(k_err, g1(N->v0), dim3(256), 0, st, N->v0, N->delta, target, e);
  hipLaunchKernelGGL(k_spmv_f32, g1(N->v0), dim3(256), 0, st, N->res0, bx, by, bz, e, Ae);
  hipLaunchKernelGGL(k_spmv_f32, g1(N->v0), dim3(256), 0, st, N->res0, bx, by, bz, target, At);
  hipLaunchKernelGGL(k_loss_part, dim3(nb), dim3(256), 0, st, N->v0, e, Ae, target, At, N->red);
  hipLaunchKernelGGL(k_loss_fin, dim3(1), dim3(64), 0, st, N->red, nb, N->red + 2 * nb);
  hipLaunchKernelGGL(k_dloss, g1(N->v0), dim3(256), 0, st, N->v0, Ae, N->red + 2 * nb, N->dd);
  backward(N);
  if (update) {
    ++N->step;
    const float c1 = 1.0f - powf(0.9f, (float)N->step), c2 = 1.0f - powf(0.999f, (float)N->step);
    hipLaunchKernelGGL(k_adam, g1((long)N->np), dim3(256), 0, st, N->theta, N->g, N->m, N->v, (long)N->np, lr, c1, c2);
    refresh_weights(N);
  }
  if (hipMemcpyAsync(N->host, N->red + 2 * nb, 2 * sizeof(double), hipMemcpyDeviceToHost, st) != hipSuccess ||
      hipStreamSynchronize(st) != hipSuccess)
    return nfail(N, NS_EHIP, "train step failed");
  if (loss) *loss = N->host[0];
  return std::isfinite(N->host[0]) ? NS_OK : nfail(N, NS_ENAN, "non-finite loss");
}

}  // extern "C"

// --------------------------------------------- hooks used by the projection
namespace nsk {

void net_features(ns_net* N, const Dims& n, double h, double rho_w, double rho_a, double P0, const double* b,
                  const double* rho, const double* pprev, const double* Ap, float* feat, hipStream_t st) {
  const long nv = (long)n.nx * n.ny * n.nz;
  const bool pack = N && !N->training && feat == N->feat;
  hipLaunchKernelGGL(pack ? k_features<true> : k_features<false>, g1(nv), dim3(256), 0, st, nv, h * h * rho_w / P0, log(rho_w),
                     1.0 / (log(rho_a) - log(rho_w)), 1.0 / P0, b, rho, pprev, Ap, feat);
}

int net_matches(const ns_net* N, const Dims& n) {
  return N && N->res0.nx == n.nx && N->res0.ny == n.ny && N->res0.nz == n.nz;
}

double* net_pprev(ns_net* N) { return N->pprev; }
double* net_Ap(ns_net* N) { return N->Ap; }
float* net_feat(ns_net* N) { return N->feat; }

// p = p_prev + P0 delta from the current features; returns the number of
// non-finite outputs (device counter read back synchronously); done, if
// given, is recorded once p is written
int net_guess(ns_net* N, double P0, double* p, hipStream_t st, hipEvent_t done) {
  hipStream_t keep = N->st;
  N->st = st;
  if (N->training) hipLaunchKernelGGL(k_set_input, g1(N->v0), dim3(256), 0, st, N->v0, N->feat, N->x0);
  forward(N);
  (void)hipMemsetAsync(N->bad, 0, sizeof(int), st);
  hipLaunchKernelGGL(k_finite_count, g1(N->v0), dim3(256), 0, st, N->v0, N->delta, N->bad);
  hipLaunchKernelGGL(k_apply_delta, g1(N->v0), dim3(256), 0, st, N->v0, N->pprev, N->delta, P0, p);
  if (done) (void)hipEventRecord(done, st);
  int bad = 0;
  (void)hipMemcpyAsync(N->host, N->bad, sizeof(int), hipMemcpyDeviceToHost, st);
  (void)hipStreamSynchronize(st);
  memcpy(&bad, N->host, sizeof(int));
  N->st = keep;
  return bad;
}

void net_target(long nv, const double* p, const double* pprev, double P0, float* t, hipStream_t st) {
  hipLaunchKernelGGL(k_target, g1(nv), dim3(256), 0, st, nv, p, pprev, 1.0 / P0, t);
}

}  // namespace nsk

// Learned coarse-grid corrector of liblbm.so: 3x3x3 periodic convolutions
// on bf16 matrix cores (v_mfma_f32_32x32x16_bf16, FP32 accumulation),
// forward, backward-data and backward-weight kernels, the training loss and
// an FP32 Adam step.  The C ABI is in lbm_nn.h.
//
// Layouts.  Activations are bf16, channels-last: a[v][C] with v the node
// index (x fastest) and C = 16 (the network input, zero-padded) or 32 (every
// layer output, zero-padded past the layer's width).  Weights are kept in
// FP32 as W[t][i][o] (tap t = (dx+1) + 3(dy+1) + 9(dz+1)) and packed to bf16
// for the matrix cores as wp[t][i/16][o][i%16] (forward) and, for the
// gradient with respect to the layer input, as the convolution with the
// mirrored taps and exchanged channels, wb[t][o/16][i][o%16].
//
// Matrix-core tiles (v_mfma_f32_32x32x16_bf16: lane l supplies
// A[m = l%32][k = 8(l/32) .. +7] and B[k = 8(l/32) .. +7][n = l%32];
// accumulator i of lane l holds C[m = 8(i/4) + 4(l/32) + i%4][n = l%32]).
// Convolution: A = weights (m = output channel, k = input channel), B =
// activations (n = node of a 32-node row), so a lane ends with four
// consecutive output channels of one node per accumulator group.  Weight
// gradient: A = input activations (m = input channel, k = node), B = output
// gradient (n = output channel), summed over nodes.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "lbm_internal.h"
#include "lbm_nn.h"

namespace lbmnn {

typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef float f16v __attribute__((ext_vector_type(16)));
typedef float f4v __attribute__((ext_vector_type(4)));

struct Grid {
  int nx, ny, nz;
};

__device__ inline int wrap(int a, int n) { return a < 0 ? a + n : (a >= n ? a - n : a); }

// planar FP32 x[c][v] (c < cin) -> bf16 a[v][16], (x - mean) / std, zero padded
__global__ void __launch_bounds__(256) pack_input_kernel(const float* __restrict__ x, int cin, const float* __restrict__ mean,
                                                         const float* __restrict__ inv_std, __bf16* __restrict__ a, int V) {
  const int v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= V) return;
  bf8 lo, hi;
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    lo[c] = (__bf16)(c < cin ? (x[(size_t)c * V + v] - mean[c]) * inv_std[c] : 0.f);
    hi[c] = (__bf16)(c + 8 < cin ? (x[(size_t)(c + 8) * V + v] - mean[c + 8]) * inv_std[c + 8] : 0.f);
  }
  *(bf8*)(a + (size_t)v * 16) = lo;
  *(bf8*)(a + (size_t)v * 16 + 8) = hi;
}

// Output tile of the convolution kernel: 32 nodes along x (the matrix-core
// N dimension) times kTY rows along y times kTZ planes along z; row q of the
// tile is (y0 + q % kTY, z0 + q / kTY) and wave w computes rows w kR ..
// w kR + kR - 1.  The input tile with its one-node periodic halo is staged in
// LDS once per block and read 27 times.
constexpr int kTX = 32, kTY = 4, kTZ = 4;
constexpr int kW = 4;                   // wavefronts per work-group (3% faster than 8: each weight operand serves 4 rows)
constexpr int kR = kTY * kTZ / kW;      // output rows (32 nodes each) per wavefront
constexpr int kHX = kTX + 2, kHY = kTY + 2, kHZ = kTZ + 2;

// Consecutive hardware work-group ids go round the eight XCDs (each with its
// own L2); the logical tile order is rebuilt so that every XCD runs one
// contiguous range of tiles, whose halos then overlap inside that XCD's L2.
__device__ inline int xcd_tile(int b, int nblocks) {
  const int q8 = nblocks >> 3, r8 = nblocks & 7, xcd = b & 7;
  return xcd * q8 + min(xcd, r8) + (b >> 3);
}

// 16-byte chunk c of the node at halo column hx is stored at chunk
// c ^ f(hx).  A 16-byte LDS read is served sixteen lanes at a time over 64
// banks of 4 bytes (256 bytes); sixteen consecutive lanes (consecutive hx,
// same c, any alignment) then hit sixteen disjoint groups of four banks.
// (The swizzle that is conflict-free for eight lanes over 32 banks,
// c ^ ((hx >> 1) & 3), measured 46% of the LDS cycles as bank conflicts.)
template <int CIN>
__device__ inline int swizzle(int c, int hx) {
  return CIN == 32 ? (c ^ ((hx >> 2) & 3)) : (c ^ ((hx >> 3) & 1));
}

// out[v][o] = bias[o] + sum_t sum_i in[v + s_t][i] w[t][i][o]  (cross-correlation)
// as the product W^T (32 outputs x K) times the input columns (K x 32 nodes),
// K = 27 taps x CIN: A[m = o][k = i] from wp, B[k = i][n = node] from LDS;
// accumulator i of lane l holds output channel 8(i/4) + 4(l/32) + i%4 of node
// x0 + l%32.  CIN: channels of in (16 or 32).  OUT_PLANAR: FP32 planes
// out[o][v] for o < cout, else bf16 out[v][32].  relu: max(., 0).  mask (bf16
// [v][32], may be null): zero where mask <= 0 (the derivative of the ReLU that
// produced it).  bias may be null; it holds cout values.
// Requires nx % 32 == 0, ny % 4 == 0, nz % 4 == 0; grid = tiles.
// Stages the input tile of output tile (x0, y0, z0) with its one-node
// periodic halo in LDS, swizzled (every thread issues all its loads before
// its first LDS write, so the tile costs one memory latency instead of one
// per chunk), and waits for the work-group.
template <int CIN>
__device__ inline void stage_tile(const __bf16* __restrict__ in, __bf16* tile, const Grid& g, int x0, int y0, int z0) {
  constexpr int CH = CIN / 8;                           // 16-byte chunks per node
  constexpr int NCH = kHZ * kHY * kHX * CH;            // 16-byte chunks of the halo tile
  constexpr int NIT = (NCH + 64 * kW - 1) / (64 * kW);  // chunks per thread
  bf8 stage[NIT];
#pragma unroll
  for (int k = 0; k < NIT; ++k) {
    const int e = threadIdx.x + k * 64 * kW;
    if (e < NCH) {
      const int c = e % CH, node = e / CH;
      const int hx = node % kHX, hy = (node / kHX) % kHY, hz = node / (kHX * kHY);
      const int gx = wrap(x0 + hx - 1, g.nx), gy = wrap(y0 + hy - 1, g.ny), gz = wrap(z0 + hz - 1, g.nz);
      stage[k] = *(const bf8*)(in + (size_t)(gx + g.nx * (gy + g.ny * gz)) * CIN + c * 8);
    }
  }
#pragma unroll
  for (int k = 0; k < NIT; ++k) {
    const int e = threadIdx.x + k * 64 * kW;
    if (e < NCH) {
      const int c = e % CH, node = e / CH;
      *(bf8*)(tile + node * CIN + swizzle<CIN>(c, node % kHX) * 8) = stage[k];
    }
  }
  __syncthreads();
}

// Bias, ReLU, ReLU-derivative mask and store of a wavefront's kR output rows
// (32 x 32 accumulator layout: accumulator i of lane l holds output channel
// 8(i/4) + 4(l/32) + i%4 of node x0 + l%32).
template <bool OUT_PLANAR>
__device__ inline void conv_epilogue(const f16v* acc, const float* bo, int relu, const __bf16* __restrict__ mask,
                                     void* __restrict__ out, int cout, const Grid& g, int V, int x0, int y0, int z0,
                                     int w, int r, int half) {
#pragma unroll
  for (int j = 0; j < kR; ++j) {
    const int q = w * kR + j;
    const int v = (x0 + r) + g.nx * ((y0 + q % kTY) + g.ny * (z0 + q / kTY));
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int c0 = 8 * q + 4 * half;
      float y[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        y[k] = acc[j][4 * q + k] + bo[4 * q + k];
        if (relu) y[k] = y[k] > 0.f ? y[k] : 0.f;
      }
      if (mask) {
        typedef __bf16 bf4 __attribute__((ext_vector_type(4)));
        const bf4 mk = *(const bf4*)(mask + (size_t)v * 32 + c0);
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (!((float)mk[k] > 0.f)) y[k] = 0.f;
      }
      if (OUT_PLANAR) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (c0 + k < cout) static_cast<float*>(out)[(size_t)(c0 + k) * V + v] = y[k];
      } else {
        typedef __bf16 bf4 __attribute__((ext_vector_type(4)));
        bf4 o;
#pragma unroll
        for (int k = 0; k < 4; ++k) o[k] = (__bf16)y[k];
        *(bf4*)(static_cast<__bf16*>(out) + (size_t)v * 32 + c0) = o;
      }
    }
  }
}

template <int CIN, bool OUT_PLANAR>
__global__ void __launch_bounds__(64 * kW) conv_kernel(const __bf16* __restrict__ in, const __bf16* __restrict__ wp,
                                                   const float* __restrict__ bias, int relu,
                                                   const __bf16* __restrict__ mask, void* __restrict__ out, int cout,
                                                   const Grid g, int V) {
  __shared__ __attribute__((aligned(16))) __bf16 tile[kHZ * kHY * kHX * CIN];
  const int tx = g.nx / kTX, ty = g.ny / kTY;
  const int b = xcd_tile(blockIdx.x, gridDim.x);
  const int x0 = (b % tx) * kTX, y0 = ((b / tx) % ty) * kTY, z0 = (b / (tx * ty)) * kTZ;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int r = lane & 31, half = lane >> 5;
  // Wave w owns the kTY output rows of plane z = w of the tile.  For one
  // (dz, dx) pair and 16-channel block, each of the kTY + 2 input rows of
  // the halo column is read from LDS once and feeds the (up to three)
  // output rows it reaches through the taps dy = -1, 0, 1, each with its own
  // weights: half the LDS reads of one read per tap and row.  The weights of
  // group (dz, dx) come from L2 while the group before it computes (two
  // register sets, one group of matrix-core work ahead); the first group's
  // and the biases are requested before the tile is staged.
  static_assert(kR == kTY && kW == kTZ, "a wavefront owns one plane of the tile");
  constexpr int NC = CIN / 16;
  bf8 a[2][NC][3];  // [set][16-channel block][dy + 1]
  auto load_group = [&](int gi, bf8(&dst)[NC][3]) {
    const int dz = gi / 3 - 1, dx = gi % 3 - 1;
#pragma unroll
    for (int cc = 0; cc < NC; ++cc)
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const int t = (dx + 1) + 3 * k + 9 * (dz + 1);
        dst[cc][k] = *(const bf8*)(wp + ((size_t)(t * NC + cc) * 32 + r) * 16 + 8 * half);
      }
  };
  load_group(0, a[0]);
  float bo[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int c = 8 * (i >> 2) + 4 * half + (i & 3);
    bo[i] = bias && c < cout ? bias[c] : 0.f;
  }
  stage_tile<CIN>(in, tile, g, x0, y0, z0);
  f16v acc[kR] = {};
#pragma unroll
  for (int gi = 0; gi < 9; ++gi) {
    if (gi + 1 < 9) load_group(gi + 1, a[(gi + 1) & 1]);
    __builtin_amdgcn_sched_barrier(0);  // keep the prefetch ahead of this group's work
    const int dz = gi / 3 - 1, dx = gi % 3 - 1;
    const int hz = w + dz + 1, hx = r + dx + 1;
    const __bf16* col = tile + hx * CIN + hz * kHY * kHX * CIN;
#pragma unroll
    for (int cc = 0; cc < NC; ++cc) {
      const int off = swizzle<CIN>(2 * cc + half, hx) * 8;
#pragma unroll
      for (int hy = 0; hy < kTY + 2; ++hy) {
        const bf8 bv = *(const bf8*)(col + hy * kHX * CIN + off);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const int j = hy - k;  // output row reached through dy = k - 1
          if (j >= 0 && j < kTY)
            acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[gi & 1][cc][k], bv, acc[j], 0, 0, 0);
        }
      }
    }
  }
  conv_epilogue<OUT_PLANAR>(acc, bo, relu, mask, out, cout, g, V, x0, y0, z0, w, r, half);
}

// Input layer of at most 8 channels (the corrector's 5: rho, u, T): the
// input activations hold 16 channels per node of which the first 8 are
// staged (16 bytes per node), and the matrix-core K dimension of 16 takes two
// taps at a time, 8 channels each: lane half h supplies tap 2p + h of pair p.
// 14 products per output row instead of 27.  wq[p][o][k]: k < 8 channel k
// of tap 2p, k >= 8 channel k - 8 of tap 2p + 1 (tap 27 does not exist: its
// weights are zero and its B operand repeats tap 26).  Output as
// conv_kernel (bf16 [v][32]).  PLANAR_IN: the input is read straight from
// the FP32 planes x[c][v] (c < cin) and normalised as pack_input_kernel does
// (the same expression, so the staged bf16 values are the same), for calls
// that need no packed copy of it (inference).  Otherwise in holds `stride`
// channels per node.  The gradient of an output layer of at most 8 channels
// goes back through it too: stride 8, the mirrored weights and the ReLU
// derivative's mask (64^3: 13.5 us; as 32 channels through conv_kernel 20.8).
template <bool PLANAR_IN>
__global__ void __launch_bounds__(64 * kW) conv_pair_kernel(const __bf16* __restrict__ in, int stride,
                                                            const float* __restrict__ x, int cin,
                                                            const float* __restrict__ mean,
                                                            const float* __restrict__ inv_std,
                                                            const __bf16* __restrict__ wq,
                                                            const float* __restrict__ bias, int relu,
                                                            const __bf16* __restrict__ mask,
                                                            __bf16* __restrict__ out, int cout, const Grid g, int V) {
  constexpr int NN = kHZ * kHY * kHX;  // halo nodes; one 16-byte chunk each
  __shared__ __attribute__((aligned(16))) __bf16 tile[NN * 8];
  const int tx = g.nx / kTX, ty = g.ny / kTY;
  const int b = xcd_tile(blockIdx.x, gridDim.x);
  const int x0 = (b % tx) * kTX, y0 = ((b / tx) % ty) * kTY, z0 = (b / (tx * ty)) * kTZ;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int r = lane & 31, half = lane >> 5;
  // every weight operand and the biases are requested before the staging
  bf8 a[14];
#pragma unroll
  for (int p = 0; p < 14; ++p) a[p] = *(const bf8*)(wq + ((size_t)p * 32 + r) * 16 + 8 * half);
  float bo[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int c = 8 * (i >> 2) + 4 * half + (i & 3);
    bo[i] = bias && c < cout ? bias[c] : 0.f;
  }
  if constexpr (PLANAR_IN) {
    // Rows (hy, hz) of the halo block: the 32 interior nodes of a row are 8
    // aligned groups of 4 consecutive x (one 16-byte load per channel; x0
    // and nx are multiples of 32), its two end nodes (x0 - 1 and x0 + 32,
    // wrapped) are loaded one by one.
    constexpr int PER_ROW = kTX / 4 + 2, ITEMS = kHZ * kHY * PER_ROW;
    constexpr int NIT = (ITEMS + 64 * kW - 1) / (64 * kW);
    float4 xs[NIT][8];
#pragma unroll
    for (int k = 0; k < NIT; ++k) {
      const int item = threadIdx.x + k * 64 * kW;
      if (item < ITEMS) {
        const int row = item / PER_ROW, e = item % PER_ROW, hy = row % kHY, hz = row / kHY;
        const int gy = wrap(y0 + hy - 1, g.ny), gz = wrap(z0 + hz - 1, g.nz);
        const int gx = e < kTX / 4 ? x0 + 4 * e : wrap(e == kTX / 4 ? x0 - 1 : x0 + kTX, g.nx);
        const size_t v = (size_t)gx + (size_t)g.nx * (gy + (size_t)g.ny * gz);
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          xs[k][c] = float4{0.f, 0.f, 0.f, 0.f};
          if (c < cin) {
            if (e < kTX / 4) xs[k][c] = *(const float4*)(x + (size_t)c * V + v);
            else xs[k][c].x = x[(size_t)c * V + v];
          }
        }
      }
    }
#pragma unroll
    for (int k = 0; k < NIT; ++k) {
      const int item = threadIdx.x + k * 64 * kW;
      if (item < ITEMS) {
        const int row = item / PER_ROW, e = item % PER_ROW;
        const int base = row * kHX;  // node index of hx = 0 in this row
        // normalised as pack_input_kernel does (the same expression, so the staged bf16 values are the same)
        auto node_chunk = [&](int n) {
          bf8 val;
#pragma unroll
          for (int c = 0; c < 8; ++c) val[c] = (__bf16)(c < cin ? (xs[k][c][n] - mean[c]) * inv_std[c] : 0.f);
          return val;
        };
        if (e < kTX / 4) {
#pragma unroll
          for (int n = 0; n < 4; ++n) *(bf8*)(tile + (base + 4 * e + n + 1) * 8) = node_chunk(n);
        } else {
          *(bf8*)(tile + (base + (e == kTX / 4 ? 0 : kHX - 1)) * 8) = node_chunk(0);
        }
      }
    }
    __syncthreads();
  } else {
    constexpr int NIT = (NN + 64 * kW - 1) / (64 * kW);
    bf8 stage[NIT];
#pragma unroll
    for (int k = 0; k < NIT; ++k) {
      const int node = threadIdx.x + k * 64 * kW;
      if (node < NN) {
        const int hx = node % kHX, hy = (node / kHX) % kHY, hz = node / (kHX * kHY);
        const int gx = wrap(x0 + hx - 1, g.nx), gy = wrap(y0 + hy - 1, g.ny), gz = wrap(z0 + hz - 1, g.nz);
        stage[k] = *(const bf8*)(in + ((size_t)gx + (size_t)g.nx * (gy + (size_t)g.ny * gz)) * stride);
      }
    }
#pragma unroll
    for (int k = 0; k < NIT; ++k) {
      const int node = threadIdx.x + k * 64 * kW;
      if (node < NN) *(bf8*)(tile + node * 8) = stage[k];
    }
    __syncthreads();
  }
  f16v acc[kR] = {};
#pragma unroll
  for (int p = 0; p < 14; ++p) {
    const int t = min(2 * p + half, 26);
    const int dx = t % 3 - 1, dy = (t / 3) % 3 - 1, dz = t / 9 - 1;
    const __bf16* col = tile + (r + dx + 1) * 8;
#pragma unroll
    for (int j = 0; j < kR; ++j) {
      const int q = w * kR + j, hy = q % kTY + dy + 1, hz = q / kTY + dz + 1;
      const bf8 bv = *(const bf8*)(col + (hz * kHY + hy) * kHX * 8);
      acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[p], bv, acc[j], 0, 0, 0);
    }
  }
  conv_epilogue<false>(acc, bo, relu, mask, out, cout, g, V, x0, y0, z0, w, r, half);
}

// Output layer with at most 16 channels (the corrector's 3): the same
// convolution on v_mfma_f32_16x16x32_bf16 (A 16 x 32, B 32 x 16; lane l
// supplies A[l%16][8(l/16) .. +7] and B[8(l/16) .. +7][l%16] and holds
// D[4(l/16) .. +3][l%16]), with A = weights (m = output channel, padded to
// 16 instead of 32, k = the 32 input channels of one tap) and B = the
// activations of 16 nodes: half the matrix-core work of conv_kernel for such
// a layer.  FP32 planes out[o][v] for o < cout.  wn[t][o][i] (o < 16,
// i < 32).  Same tile and staging as conv_kernel; input width 32.
__global__ void __launch_bounds__(64 * kW) conv_narrow_kernel(const __bf16* __restrict__ in,
                                                              const __bf16* __restrict__ wn,
                                                              const float* __restrict__ bias,
                                                              float* __restrict__ out, int cout, const Grid g, int V) {
  __shared__ __attribute__((aligned(16))) __bf16 tile[kHZ * kHY * kHX * 32];
  const int tx = g.nx / kTX, ty = g.ny / kTY;
  const int b = xcd_tile(blockIdx.x, gridDim.x);
  const int x0 = (b % tx) * kTX, y0 = ((b / tx) % ty) * kTY, z0 = (b / (tx * ty)) * kTZ;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int n16 = lane & 15, grp = lane >> 4;
  // weights of group (dz, dx), taps dy = -1, 0, 1: A[o = l%16][i = 8(l/16) + j];
  // one group ahead, as in conv_kernel
  bf8 a[2][3];
  auto load_group = [&](int gi, bf8(&dst)[3]) {
    const int dz = gi / 3 - 1, dx = gi % 3 - 1;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int t = (dx + 1) + 3 * k + 9 * (dz + 1);
      dst[k] = *(const bf8*)(wn + ((size_t)t * 16 + n16) * 32 + 8 * grp);
    }
  };
  load_group(0, a[0]);
  float bo[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) bo[v] = bias && 4 * grp + v < cout ? bias[4 * grp + v] : 0.f;
  stage_tile<32>(in, tile, g, x0, y0, z0);
  f4v acc[kTY][2] = {};
#pragma unroll
  for (int gi = 0; gi < 9; ++gi) {
    if (gi + 1 < 9) load_group(gi + 1, a[(gi + 1) & 1]);
    __builtin_amdgcn_sched_barrier(0);  // keep the prefetch ahead of this group's work
    const int dz = gi / 3 - 1, dx = gi % 3 - 1;
    const int hz = w + dz + 1;
#pragma unroll
    for (int hy = 0; hy < kTY + 2; ++hy) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int hx = 16 * h + n16 + dx + 1;
        const bf8 bv = *(const bf8*)(tile + ((hz * kHY + hy) * kHX + hx) * 32 + swizzle<32>(grp, hx) * 8);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const int j = hy - k;
          if (j >= 0 && j < kTY)
            acc[j][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[gi & 1][k], bv, acc[j][h], 0, 0, 0);
        }
      }
    }
  }
#pragma unroll
  for (int j = 0; j < kTY; ++j)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int v = (x0 + 16 * h + n16) + g.nx * ((y0 + j) + g.ny * (z0 + w));
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c = 4 * grp + q;
        if (c < cout) out[(size_t)c * V + v] = acc[j][h][q] + bo[q];
      }
    }
}

// Weight and bias gradients of one layer, per work-group partial sums over
// the layer's real channels (i < cin, o < cout):
//   slot t < 27: part[t][b][i][o] = sum over the group's nodes v of in[v + s_t][i] dout[v][o]
//   slot 27:     part[27][b][i][o] = sum over the group's nodes v of dout[v][o] (every row i)
// (the bias gradient as the product with a row of ones).  Work-group b takes
// tiles b tpb .. b tpb + tpb - 1 of 32 x 4 x 2 nodes (x fastest, then y, z), its
// two halves of four wavefronts in turn.  Per tile the input with its one-node
// halo and the output gradient are staged in LDS channel-major, so that the
// node index runs along the matrix-core K dimension: lane (r, h) reads 8
// consecutive nodes of channel r as one 16-byte word.  The x offset of a tap is
// 0, 1 or 2 elements inside two aligned words and is taken out with funnel
// shifts.  Wave w of a half owns seven slots (the three dx taps of two (dy, dz)
// pairs and one more; see the loop) and keeps their sums in registers across
// the tiles.
// What binds is not the matrix cores but what surrounds them.  With 512
// work-groups of one half each at 64^3, a work-group's partials (114 KB at 32
// channels) were nearly as much as the two tiles that it reads (137 KB); the halves
// add theirs in LDS and one work-group per compute unit writes, for four tiles.
// The next tile's input is requested before the products of the present one, and
// two neighbouring nodes of a channel go to LDS as one 4-byte word.  64^3, 32
// channels: 27.5 us (32.2 us in the former launch, without these).
constexpr int kGX = 32, kGY = 4, kGZ = 2;
constexpr int kGHY = kGY + 2, kGHZ = kGZ + 2, kGHX = kGX + 2;
constexpr int kGRow = 40;                           // halo row: 34 nodes, padded to a 16-byte multiple
constexpr int kGPlaneIn = kGHZ * kGHY * kGRow + 8;  // per channel; the 16 extra bytes spread the
constexpr int kGPlaneD = kGZ * kGY * kGX + 8;       // channel planes over the LDS banks
constexpr int kGMaxBlocks = 256;

typedef unsigned int u4 __attribute__((ext_vector_type(4)));

// Channel j of two neighbouring nodes as one word of channel-major LDS, eight
// channels.
__device__ inline void transpose(const u4 (&v)[2], __bf16* dst, int plane) {
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const unsigned a = v[0][j / 2], b = v[1][j / 2];
    *(unsigned*)(dst + j * plane) =
        j % 2 ? __builtin_amdgcn_perm(b, a, 0x07060302u) : __builtin_amdgcn_perm(b, a, 0x05040100u);
  }
}

// The 8 elements from element o (0, 1 or 2) of lo.
__device__ inline bf8 shifted(const u4& lo, const u4& hi, int o) {
  u4 v;
  if (o == 0) {
    v = lo;
  } else if (o == 2) {
    v = u4{lo.y, lo.z, lo.w, hi.x};
  } else {
    v = u4{__builtin_amdgcn_alignbit(lo.y, lo.x, 16), __builtin_amdgcn_alignbit(lo.z, lo.y, 16),
           __builtin_amdgcn_alignbit(lo.w, lo.z, 16), __builtin_amdgcn_alignbit(hi.x, lo.w, 16)};
  }
  return __builtin_bit_cast(bf8, v);
}

template <int CIN>
__global__ void __launch_bounds__(512) wgrad_kernel(const __bf16* __restrict__ in, const __bf16* __restrict__ dout,
                                                    float* __restrict__ part, const Grid g, int ntiles, int tpb,
                                                    int cin, int cout) {
  constexpr int kHalf = CIN * kGPlaneIn + 32 * kGPlaneD;  // bf16 elements of one half's tile
  constexpr int NI = CIN / 2;                             // accumulator registers that hold input channels < CIN
  static_assert(4 * 7 * NI * 64 * sizeof(float) <= 2 * kHalf * sizeof(__bf16), "the halves' sums fit the tiles' LDS");
  __shared__ __attribute__((aligned(16))) __bf16 lds[2 * kHalf];
  const int half_wg = threadIdx.x >> 8, t = threadIdx.x & 255;
  __bf16* inT = lds + half_wg * kHalf;
  __bf16* dT = inT + CIN * kGPlaneIn;
  const int lane = t & 63, w = t >> 6;
  const int r = lane & 31, half = lane >> 5;
  const int tx = g.nx / kGX, ty = g.ny / kGY;
  bf8 ones;
#pragma unroll
  for (int j = 0; j < 8; ++j) ones[j] = (__bf16)1.f;
  f16v acc[7] = {};
  const int bl = xcd_tile(blockIdx.x, gridDim.x);  // logical block: tiles and partial slot
  const int first = bl * tpb, last = min(first + tpb, ntiles);
  // Items of two x neighbours times 8 channels (16 bytes a node).
  constexpr int NIN = (kGHX / 2) * kGHY * kGHZ * (CIN / 8), NITI = (NIN + 255) / 256;
  constexpr int ND = (kGX / 2) * kGY * kGZ * 4, NITD = ND / 256;
  static_assert(ND % 256 == 0 && kGHX % 2 == 0, "whole items");
  u4 si[NITI][2];
  auto origin = [&](int tile, int& x0, int& y0, int& z0) {
    x0 = (tile % tx) * kGX, y0 = ((tile / tx) % ty) * kGY, z0 = (tile / (tx * ty)) * kGZ;
  };
  auto request = [&](int tile) {
    int x0, y0, z0;
    origin(tile, x0, y0, z0);
#pragma unroll
    for (int k = 0; k < NITI; ++k) {
      const int e = t + k * 256;
      if (e < NIN) {
        const int pair = e % (kGHX / 2), c8 = (e / (kGHX / 2)) % (CIN / 8), row = e / (kGHX / 2 * (CIN / 8));
        const int gy = wrap(y0 + row % kGHY - 1, g.ny), gz = wrap(z0 + row / kGHY - 1, g.nz);
        const __bf16* base = in + (size_t)(g.nx * (gy + g.ny * gz)) * CIN + 8 * c8;
#pragma unroll
        for (int q = 0; q < 2; ++q)
          si[k][q] = *(const u4*)(base + (size_t)wrap(x0 + 2 * pair + q - 1, g.nx) * CIN);
      }
    }
  };
  int tile = first + half_wg;
  if (tile < last) request(tile);
  for (int step = 0; step < tpb; step += 2, tile += 2) {  // the same number of steps in both halves
    const bool active = tile < last;
    __syncthreads();  // every wave is done with the previous tiles
    if (active) {
      // the output gradient's values arrive while the input's go to LDS (held a
      // tile ahead as well, they would not fit the registers)
      u4 sd[NITD][2];
      int x0, y0, z0;
      origin(tile, x0, y0, z0);
#pragma unroll
      for (int k = 0; k < NITD; ++k) {
        const int e = t + k * 256;
        const int pair = e % (kGX / 2), c8 = (e / (kGX / 2)) % 4, row = e / (kGX / 2 * 4);
        const __bf16* base =
            dout + (size_t)(x0 + 2 * pair + g.nx * (y0 + row % kGY + g.ny * (z0 + row / kGY))) * 32 + 8 * c8;
#pragma unroll
        for (int q = 0; q < 2; ++q) sd[k][q] = *(const u4*)(base + q * 32);
      }
#pragma unroll
      for (int k = 0; k < NITI; ++k) {
        const int e = t + k * 256;
        if (e < NIN) {
          const int pair = e % (kGHX / 2), c8 = (e / (kGHX / 2)) % (CIN / 8), row = e / (kGHX / 2 * (CIN / 8));
          transpose(si[k], inT + 8 * c8 * kGPlaneIn + row * kGRow + 2 * pair, kGPlaneIn);
        }
      }
#pragma unroll
      for (int k = 0; k < NITD; ++k) {
        const int e = t + k * 256;
        const int pair = e % (kGX / 2), c8 = (e / (kGX / 2)) % 4, row = e / (kGX / 2 * 4);
        transpose(sd[k], dT + 8 * c8 * kGPlaneD + row * kGX + 2 * pair, kGPlaneD);
      }
    }
    __syncthreads();
    if (tile + 2 < last) request(tile + 2);
    if (!active) continue;
    // The three slots of one (dy, dz) pair (dx = -1, 0, 1) read the same two
    // words of a channel row and differ by a shift of 0, 1 or 2 elements, so a
    // wave owns whole pairs: wave w takes the pairs 2w and 2w + 1 (slots 6w ..
    // 6w + 5) and a seventh slot, dx = w - 1 of pair 8 (slot 24 + w) for w < 3
    // and the bias (slot 27) for w = 3.  Two LDS reads serve three products.
#pragma unroll 1
    for (int row = 0; row < kGY * kGZ; ++row) {
      const int yy = row % kGY, zz = row / kGY;
#pragma unroll
      for (int kb = 0; kb < kGX; kb += 16) {
        // the output gradient of these 16 nodes serves all seven slots of the wave
        const bf8 b = *(const bf8*)(dT + r * kGPlaneD + (zz * kGY + yy) * kGX + kb + 8 * half);
        auto words = [&](int pair, u4& lo, u4& hi) {
          const int dy = pair % 3 - 1, dz = pair / 3 - 1;
          const __bf16* src = inT + r * kGPlaneIn + ((zz + dz + 1) * kGHY + yy + dy + 1) * kGRow + kb + 8 * half;
          lo = *(const u4*)src;
          hi = *(const u4*)(src + 8);
        };
#pragma unroll
        for (int gp = 0; gp < 2; ++gp) {
          u4 lo{}, hi{};
          if (r < CIN) words(2 * w + gp, lo, hi);
#pragma unroll
          for (int o = 0; o < 3; ++o)
            acc[3 * gp + o] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(shifted(lo, hi, o), b, acc[3 * gp + o], 0, 0, 0);
        }
        bf8 a = ones;
        if (w < 3) {
          u4 lo{}, hi{};
          if (r < CIN) words(8, lo, hi);
          a = shifted(lo, hi, w);
        }
        acc[6] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[6], 0, 0, 0);
      }
    }
  }
  // the second half's sums through LDS into the first half's
  if (tpb > 1) {
    __syncthreads();
    float* sums = (float*)lds + (w * 7 * NI) * 64 + lane;
    if (half_wg == 1) {
#pragma unroll
      for (int k = 0; k < 7; ++k)
#pragma unroll
        for (int i = 0; i < NI; ++i) sums[(k * NI + i) * 64] = acc[k][i];
    }
    __syncthreads();
    if (half_wg == 0) {
#pragma unroll
      for (int k = 0; k < 7; ++k)
#pragma unroll
        for (int i = 0; i < NI; ++i) acc[k][i] += sums[(k * NI + i) * 64];
    }
  }
  if (half_wg) return;
  // accumulator i of lane l holds input channel m = 8(i/4) + 4(l/32) + i%4
  // and output channel r = l%32
#pragma unroll
  for (int k = 0; k < 7; ++k) {
    const int slot = k < 6 ? 6 * w + k : (w < 3 ? 24 + w : 27);
    float* dst = part + ((size_t)slot * gridDim.x + bl) * cin * cout;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int m = 8 * (i >> 2) + 4 * half + (i & 3);
      if (m < cin && r < cout) dst[m * cout + r] = acc[k][i];
    }
  }
}

// The same partials for a layer with at most 8 channels on one side: an output
// layer (IN false; wide: the input, narrow: dout, 8 channels per node) or an input
// layer (IN true; wide: dout, narrow: the input, the first 8 of `stride` channels
// per node).  The product is turned round: the 32 rows are the channels of the
// wide side at the tile's own nodes u, and the 32 columns are four taps times 8
// channels of the narrow side at u - s_t (u + s_t for an input layer), so that
// nine columns' worth of (dy, dz) pairs per dx take three products where a tap at a
// time takes nine, the wide side needs no halo and the narrow side is four times
// smaller.  Waves 0 to 2 of a half own dx = -1, 0, 1; wave 3 owns the bias (a
// product with ones).
// 64^3: 32 to 3 channels 15.5 us (17.9 with one work-group per compute unit; 27.4
// in wgrad_kernel); 5 to 32 channels 19.0 us on a card 4% slower (23.4 in
// wgrad_kernel).  Two work-groups fit a compute unit, and the partials of so few
// channels cost little.
constexpr int kNMaxBlocks = 512;

template <bool IN>
__global__ void __launch_bounds__(512, 4) wgrad_narrow_kernel(const __bf16* __restrict__ wide,
                                                           const __bf16* __restrict__ narrow, int stride,
                                                           float* __restrict__ part, const Grid g, int ntiles, int tpb,
                                                           int cin, int cout) {
  constexpr int kHalf = 32 * kGPlaneD + 8 * kGPlaneIn;  // bf16 elements of one half's tile
  static_assert(4 * 3 * 16 * 64 * sizeof(float) <= 2 * kHalf * sizeof(__bf16), "the halves' sums fit the tiles' LDS");
  __shared__ __attribute__((aligned(16))) __bf16 lds[2 * kHalf];
  const int half_wg = threadIdx.x >> 8, t = threadIdx.x & 255;
  __bf16* wT = lds + half_wg * kHalf;
  __bf16* nT = wT + 32 * kGPlaneD;
  const int lane = t & 63, w = t >> 6;
  const int r = lane & 31, half = lane >> 5;
  const int tx = g.nx / kGX, ty = g.ny / kGY;
  bf8 ones;
#pragma unroll
  for (int j = 0; j < 8; ++j) ones[j] = (__bf16)1.f;
  f16v acc[3] = {};
  const int bl = xcd_tile(blockIdx.x, gridDim.x);
  const int first = bl * tpb, last = min(first + tpb, ntiles);
  // items of two x neighbours times 8 channels
  constexpr int NW = (kGX / 2) * kGY * kGZ * 4, NITW = NW / 256;
  constexpr int NN = (kGHX / 2) * kGHY * kGHZ, NITN = (NN + 255) / 256;
  static_assert(NW % 256 == 0 && kGHX % 2 == 0, "whole items");
  u4 sw[NITW][2], sn[NITN][2];
  auto request = [&](int tile) {
    const int x0 = (tile % tx) * kGX, y0 = ((tile / tx) % ty) * kGY, z0 = (tile / (tx * ty)) * kGZ;
#pragma unroll
    for (int k = 0; k < NITW; ++k) {
      const int e = t + k * 256;
      const int pair = e % (kGX / 2), c8 = (e / (kGX / 2)) % 4, row = e / (kGX / 2 * 4);
      const __bf16* base =
          wide + ((size_t)(x0 + 2 * pair) + (size_t)g.nx * (y0 + row % kGY + g.ny * (z0 + row / kGY))) * 32 + 8 * c8;
#pragma unroll
      for (int q = 0; q < 2; ++q) sw[k][q] = *(const u4*)(base + q * 32);
    }
#pragma unroll
    for (int k = 0; k < NITN; ++k) {
      const int e = t + k * 256;
      if (e < NN) {
        const int pair = e % (kGHX / 2), row = e / (kGHX / 2);
        const int gy = wrap(y0 + row % kGHY - 1, g.ny), gz = wrap(z0 + row / kGHY - 1, g.nz);
        const __bf16* base = narrow + (size_t)(g.nx * (gy + g.ny * gz)) * stride;
#pragma unroll
        for (int q = 0; q < 2; ++q) sn[k][q] = *(const u4*)(base + (size_t)wrap(x0 + 2 * pair + q - 1, g.nx) * stride);
      }
    }
  };
  int tile = first + half_wg;
  if (tile < last) request(tile);
  for (int step = 0; step < tpb; step += 2, tile += 2) {  // the same number of steps in both halves
    const bool active = tile < last;
    __syncthreads();  // every wave is done with the previous tiles
    if (active) {
#pragma unroll
      for (int k = 0; k < NITW; ++k) {
        const int e = t + k * 256;
        const int pair = e % (kGX / 2), c8 = (e / (kGX / 2)) % 4, row = e / (kGX / 2 * 4);
        transpose(sw[k], wT + 8 * c8 * kGPlaneD + row * kGX + 2 * pair, kGPlaneD);
      }
#pragma unroll
      for (int k = 0; k < NITN; ++k) {
        const int e = t + k * 256;
        if (e < NN) transpose(sn[k], nT + e / (kGHX / 2) * kGRow + 2 * (e % (kGHX / 2)), kGPlaneIn);
      }
    }
    __syncthreads();
    if (tile + 2 < last) request(tile + 2);
    if (!active) continue;
#pragma unroll 1
    for (int row = 0; row < kGY * kGZ; ++row) {
      const int yy = row % kGY, zz = row / kGY;
#pragma unroll
      for (int kb = 0; kb < kGX; kb += 16) {
        auto column = [&](int pair, int shift) {  // narrow channel r % 8 at u -+ s of these nodes
          const int dy = IN ? pair % 3 - 1 : 1 - pair % 3, dz = IN ? pair / 3 - 1 : 1 - pair / 3;
          const __bf16* src =
              nT + (r & 7) * kGPlaneIn + ((zz + dz + 1) * kGHY + yy + dy + 1) * kGRow + kb + 8 * half;
          return shifted(*(const u4*)src, *(const u4*)(src + 8), shift);
        };
        bf8 a = ones;
        if (w < 3 || IN) a = *(const bf8*)(wT + r * kGPlaneD + row * kGX + kb + 8 * half);
        if (w < 3) {
#pragma unroll
          for (int j = 0; j < 3; ++j)
            acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, column(min(4 * j + (r >> 3), 8), IN ? w : 2 - w), acc[j],
                                                             0, 0, 0);
        } else {
          const bf8 b = IN ? ones : column(4, 1);
          acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[0], 0, 0, 0);
        }
      }
    }
  }
  // the second half's sums through LDS into the first half's
  if (tpb > 1) {
    __syncthreads();
    float* sums = (float*)lds + (w * 3 * 16) * 64 + lane;
    if (half_wg == 1) {
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int i = 0; i < 16; ++i) sums[(k * 16 + i) * 64] = acc[k][i];
    }
    __syncthreads();
    if (half_wg == 0) {
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[k][i] += sums[(k * 16 + i) * 64];
    }
  }
  if (half_wg) return;
  // accumulator i of lane l holds row m = 8(i/4) + 4(l/32) + i%4, column r = l%32
  const int c = r & 7;  // narrow channel
  const int cw = IN ? cout : cin, cn = IN ? cin : cout;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int pair = 4 * k + (r >> 3);
    const bool bias = w == 3 && k == 0 && r < 8;
    if (c >= cn || !(bias || (w < 3 && pair < 9))) continue;
    const int slot = w == 3 ? 27 : 3 * pair + w;
    float* dst = part + ((size_t)slot * gridDim.x + bl) * cin * cout;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int m = 8 * (i >> 2) + 4 * half + (i & 3);
      if (m < cw) dst[IN ? c * cout + m : m * cout + c] = acc[k][i];
    }
  }
}

// grad[t][i][o] += sum_b part[t][b][i][o] (t < 27) and grad_b[o] += sum_b
// part[27][b][0][o] of up to kSumLayers layers, part laid out
// [28][nblk][cin][cout].  A work-group takes 64 consecutive (i, o) of one slot; its
// wavefront s adds the s-th of sixteen equal runs of b, eight loads in flight,
// and the runs are added in order: a fixed summation order.  The work-group past
// the layers' adds a sample's loss to the running sum, where there is one.
// One launch for a sample's layers: 64^3, 5-32-32-32-3 channels 13.8 us (four
// launches of 5.3 us and one of 5 for the loss, and the gaps between them).
constexpr int kGRuns = 16;
constexpr int kSumLayers = 8;

struct SumLayer {
  const float* part;
  float *grad, *grad_b;
  int nblk, cin, cout;
  int first;  // its first work-group
};

struct SumTable {
  SumLayer layer[kSumLayers];
  int layers = 0, blocks = 0;      // layers in use, their work-groups
  const double* lpart = nullptr;   // loss partials (NULL: none)
  int lcount = 0;
  double lscale = 0.0;
  double* loss = nullptr;
};

// acc[0] += scale * (sum of partial[0 .. n-1]) in a fixed order: the loss of one
// sample added to a device-side running sum, by the first 256 threads.
__device__ inline void loss_accumulate(const double* __restrict__ partial, int n, double scale,
                                       double* __restrict__ acc, double* red) {
  const int t = threadIdx.x;
  if (t < 256) {
    double s = 0.0;
    for (int i = t; i < n; i += 256) s += partial[i];
    red[t] = s;
  }
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (t < w) red[t] += red[t + w];
    __syncthreads();
  }
  if (t == 0) acc[0] += scale * red[0];
}

__global__ void __launch_bounds__(64 * kGRuns) wgrad_sum_kernel(const SumTable tab) {
  __shared__ double shared[kGRuns * 64 / 2];
  if ((int)blockIdx.x >= tab.blocks) {
    loss_accumulate(tab.lpart, tab.lcount, tab.lscale, tab.loss, shared);
    return;
  }
  float(*red)[64] = reinterpret_cast<float(*)[64]>(shared);
  int l = 0;
  while (l + 1 < tab.layers && (int)blockIdx.x >= tab.layer[l + 1].first) ++l;
  const SumLayer& ly = tab.layer[l];
  const int cio = ly.cin * ly.cout, per_slot = (cio + 63) / 64, nblk = ly.nblk;
  const int t = ((int)blockIdx.x - ly.first) / per_slot;
  const int lane = threadIdx.x & 63, s = threadIdx.x >> 6;
  const int io = ((int)blockIdx.x - ly.first - t * per_slot) * 64 + lane;
  const int b0 = nblk * s / kGRuns, b1 = nblk * (s + 1) / kGRuns;
  float acc = 0.f;
  if (io < cio) {
    const float* src = ly.part + ((size_t)t * nblk + b0) * cio + io;
    int b = b0;
    for (; b + 8 <= b1; b += 8, src += (size_t)8 * cio) {
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = src[(size_t)j * cio];
#pragma unroll
      for (int j = 0; j < 8; ++j) acc += v[j];
    }
    for (; b < b1; ++b, src += cio) acc += *src;
  }
  red[s][lane] = acc;
  __syncthreads();
  if (s || io >= cio || (t == 27 && io >= ly.cout)) return;
#pragma unroll
  for (int k = 1; k < kGRuns; ++k) acc += red[k][lane];
  if (t < 27) ly.grad[(size_t)t * cio + io] += acc;
  else ly.grad_b[io] += acc;
}

// r_c = y_c + (x_f - target_f) / out_std_c with f = off + c; loss partial sums
// of r^2; dout[v][c] = 2 r / (C V), of 32 channels or, for C <= 8, of 8
template <int CH>
__global__ void __launch_bounds__(256) loss_kernel(const float* __restrict__ y, const float* __restrict__ x,
                                                   const float* __restrict__ tgt, const float* __restrict__ inv_std,
                                                   int C, int off, int V, __bf16* __restrict__ dout,
                                                   double* __restrict__ partial) {
  __shared__ double red[256];
  const int v = blockIdx.x * blockDim.x + threadIdx.x;
  double s = 0.0;
  if (v < V) {
    const float scale = 2.f / ((float)C * (float)V);
    bf8 o[CH / 8];  // the node's gradient channels, stored as 16-byte words
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      float g = 0.f;
      if (c < C) {
        const size_t f = (size_t)(off + c) * V + v;
        const float rr = y[(size_t)c * V + v] + (x[f] - tgt[f]) * inv_std[c];
        s += (double)rr * rr;
        g = scale * rr;
      }
      o[c / 8][c % 8] = (__bf16)g;
    }
#pragma unroll
    for (int q = 0; q < CH / 8; ++q) *(bf8*)(dout + (size_t)v * CH + 8 * q) = o[q];
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

__global__ void __launch_bounds__(256) adam_kernel(float* __restrict__ p, const float* __restrict__ g,
                                                   float* __restrict__ m, float* __restrict__ v, long long n, float lr,
                                                   float b1, float b2, float eps, float gscale, float c1, float c2) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i] * gscale;
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  p[i] -= lr * (mi * c1) / (sqrtf(vi * c2) + eps);
}

// bf16 copies of one layer's FP32 weights W[t][i][o] (cin x cout):
// wp[t][i/16][o][i%16] (CINP padded inputs, 32 outputs) and
// wb[t][o/16][i][o%16] = W[26 - t][i][o] (32 padded outputs as inputs, 32 rows)
// and, for an output layer of at most 16 channels, wn[t][o][i] = W[t][i][o]
// (16 padded outputs, 32 padded inputs); for an input layer of at most 8
// channels, wq[p][o][k] (taps 2p and 2p + 1, 8 channels each); for an output
// layer of at most 8, wr[p][i][k] the same of the mirrored convolution
//
// One launch (grid y = layer) packs up to kPackLayers layers: 4.4 us for four (four
// launches of 3.8 us, and the gaps between them).
constexpr int kPackLayers = 8;

struct PackLayer {
  const float* W;
  int cin, cout, cinp;
  __bf16 *wp, *wb, *wn, *wq, *wr;
};

struct PackTable {
  PackLayer layer[kPackLayers];
};

__global__ void __launch_bounds__(256) pack_weights_kernel(const PackTable tab) {
  const PackLayer& ly = tab.layer[blockIdx.y];
  const float* __restrict__ W = ly.W;
  const int cin = ly.cin, cout = ly.cout, cinp = ly.cinp;
  __bf16 *__restrict__ wp = ly.wp, *__restrict__ wb = ly.wb, *__restrict__ wn = ly.wn, *__restrict__ wq = ly.wq,
         *__restrict__ wr = ly.wr;
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e < 27 * cinp * 32) {  // wp element (t, cc, o, k)
    const int k = e % 16, o = (e / 16) % 32, cc = (e / 512) % (cinp / 16), t = e / (512 * (cinp / 16));
    const int i = cc * 16 + k;
    wp[e] = (__bf16)(i < cin && o < cout ? W[((size_t)t * cin + i) * cout + o] : 0.f);
  }
  if (wq && e < 14 * 32 * 16) {  // wq element (p, o, k): tap 2p + k / 8, channel k % 8
    const int k = e % 16, o = (e / 16) % 32, p = e / 512;
    const int t = 2 * p + k / 8, i = k % 8;
    wq[e] = (__bf16)(t < 27 && i < cin && o < cout ? W[((size_t)t * cin + i) * cout + o] : 0.f);
  }
  if (wr && e < 14 * 32 * 16) {  // wr element (p, i, k): tap 2p + k / 8, output channel k % 8
    const int k = e % 16, i = (e / 16) % 32, p = e / 512;
    const int t = 2 * p + k / 8, o = k % 8;
    wr[e] = (__bf16)(t < 27 && i < cin && o < cout ? W[((size_t)(26 - t) * cin + i) * cout + o] : 0.f);
  }
  if (wn && e < 27 * 16 * 32) {  // wn element (t, o, i)
    const int i = e % 32, o = (e / 32) % 16, t = e / 512;
    wn[e] = (__bf16)(i < cin && o < cout ? W[((size_t)t * cin + i) * cout + o] : 0.f);
  }
  if (wb && e < 27 * 32 * 32) {  // wb element (t, oc, i, k): input channel of the mirrored conv = o
    const int k = e % 16, i = (e / 16) % 32, oc = (e / 512) % 2, t = e / 1024;
    const int o = oc * 16 + k;
    wb[e] = (__bf16)(i < cin && o < cout ? W[((size_t)(26 - t) * cin + i) * cout + o] : 0.f);
  }
}

// FP64 fields of a lattice Boltzmann handle (rho, u planes, T) -> FP32 planes
__global__ void __launch_bounds__(256) fields_to_input_kernel(const double* __restrict__ rho, const double* __restrict__ u,
                                                              const double* __restrict__ T, int D, int V,
                                                              float* __restrict__ x) {
  const int v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= V) return;
  x[v] = (float)rho[v];
  for (int a = 0; a < D; ++a) x[(size_t)(1 + a) * V + v] = (float)u[(size_t)a * V + v];
  x[(size_t)(1 + D) * V + v] = (float)T[v];
}

}  // namespace lbmnn

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

namespace {

int nn_fail(int code, const std::string& msg) { return lbm::set_error(code, msg); }

int nn_hip(hipError_t e, const char* what) {
  return nn_fail(LBM_EDEVICE, std::string(what) + ": " + hipGetErrorString(e));
}

#define NN_HIP(expr, what)                            \
  do {                                                \
    hipError_t e_ = (expr);                           \
    if (e_ != hipSuccess) return nn_hip(e_, what);    \
  } while (0)

struct Layer {
  int cin, cout, cinp;          // channels, padded input channels (16 or 32)
  long long w_off, b_off;       // offsets in the parameter vector
  __bf16 *wp = nullptr, *wb = nullptr;
  __bf16* wn = nullptr;         // output layer of <= 16 channels from 32 inputs: weights for conv_narrow_kernel
  __bf16* wq = nullptr;         // input layer of <= 8 channels (not the last): weights for conv_pair_kernel
  __bf16* wr = nullptr;         // output layer of <= 8 channels (not the first): mirrored, for conv_pair_kernel
};

}  // namespace

struct lbm_nn_ctx {
  int L = 0;
  std::vector<int> ch;
  lbmnn::Grid g{};
  int V = 0;
  int device = 0;
  hipStream_t stream = nullptr;
  std::vector<Layer> layers;
  long long nparam = 0;
  float *params = nullptr, *grads = nullptr, *m = nullptr, *v = nullptr;
  float *mean = nullptr, *inv_std = nullptr;          // input scaling (device, 16 each)
  float *out_std = nullptr, *inv_out_std = nullptr;   // output scaling (device, 32 each)
  std::vector<__bf16*> act;     // act[l]: input of layer l (bf16 [V][16 or 32]); act[L] unused
  __bf16 *dA = nullptr, *dB = nullptr;  // gradient ping-pong, bf16 [V][32]
  float* y = nullptr;                   // network output planes [c_L][V]
  float* part = nullptr;                // weight-gradient partials, per work-group
  size_t part_size = 0;                 // floats of it
  int out_off = 0;                      // output c corrects / is compared with field out_off + c
  double limit = 0.0;                   // lbm_nn_correct clips outputs to [-limit, limit] (0: no clip)
  double* lpart = nullptr;              // loss partials
  double* loss_acc = nullptr;           // running sum of asynchronous losses (device, 1 value)
  long long loss_count = 0;             // losses added to it since the last lbm_nn_take_loss
  float* fld = nullptr;                 // the corrector's input planes
};

namespace {

int nn_select(lbm_nn n) {
  int cur = -1;
  NN_HIP(hipGetDevice(&cur), "hipGetDevice");
  if (cur != n->device) NN_HIP(hipSetDevice(n->device), "hipSetDevice");
  return LBM_OK;
}

int nn_pack_weights(lbm_nn n) {
  for (int first = 0; first < n->L; first += lbmnn::kPackLayers) {
    const int count = std::min(n->L - first, lbmnn::kPackLayers);
    lbmnn::PackTable tab{};
    for (int k = 0; k < count; ++k) {
      const Layer& ly = n->layers[first + k];
      tab.layer[k] = {n->params + ly.w_off, ly.cin, ly.cout, ly.cinp, ly.wp, ly.wb, ly.wn, ly.wq, ly.wr};
    }
    hipLaunchKernelGGL(lbmnn::pack_weights_kernel, dim3(27 * 32 * 32 / 256, count), dim3(256), 0, n->stream, tab);
    NN_HIP(hipGetLastError(), "pack weights");
  }
  return LBM_OK;
}

// An output layer whose gradient is kept as 8 channels per node.
bool narrow_output(const lbm_nn_ctx& n, int l) { return l > 0 && l == n.L - 1 && n.layers[l].cout <= 8; }

// A layer with at most 8 channels on one side and 32 on the other, or an output
// layer of them.
bool narrow_side(const lbm_nn_ctx& n, int l) {
  return narrow_output(n, l) || (l == 0 && n.L > 1 && n.layers[l].cin <= 8);
}

// Work-groups of a weight gradient, and the tiles each of them takes.
void gradient_blocks(const lbmnn::Grid& g, int& ntiles, int& tpb, int& nblk, int most) {
  ntiles = (g.nx / lbmnn::kGX) * (g.ny / lbmnn::kGY) * (g.nz / lbmnn::kGZ);
  tpb = (ntiles + most - 1) / most;
  nblk = (ntiles + tpb - 1) / tpb;
}

template <int CIN, bool PLANAR>
hipError_t conv(lbm_nn n, const __bf16* in, const __bf16* w, const float* bias, int relu, const __bf16* mask,
                void* out, int cout) {
  const int blocks = (n->g.nx / lbmnn::kTX) * (n->g.ny / lbmnn::kTY) * (n->g.nz / lbmnn::kTZ);
  hipLaunchKernelGGL((lbmnn::conv_kernel<CIN, PLANAR>), dim3(blocks), dim3(64 * lbmnn::kW), 0, n->stream, in, w, bias,
                     relu,
                     mask, out, cout, n->g, n->V);
  return hipGetLastError();
}

// forward pass of normalised x into yout (n->y if null); activations kept
// for the backward pass.  keep_input: also keep the packed input (the weight
// gradient of the first layer reads it); without it a first layer of at most
// 8 channels reads x directly.
int nn_forward(lbm_nn n, const float* x, float* yout = nullptr, bool keep_input = true) {
  if (!yout) yout = n->y;
  const bool direct = !keep_input && n->layers[0].wq && n->L > 1;
  if (!direct) {
    hipLaunchKernelGGL(lbmnn::pack_input_kernel, dim3((n->V + 255) / 256), dim3(256), 0, n->stream, x, n->ch[0],
                       n->mean, n->inv_std, n->act[0], n->V);
    NN_HIP(hipGetLastError(), "pack input");
  }
  for (int l = 0; l < n->L; ++l) {
    const Layer& ly = n->layers[l];
    const bool last = l == n->L - 1;
    const float* b = n->params + ly.b_off;
    hipError_t e;
    if (last && ly.wn) {
      const int blocks = (n->g.nx / lbmnn::kTX) * (n->g.ny / lbmnn::kTY) * (n->g.nz / lbmnn::kTZ);
      hipLaunchKernelGGL(lbmnn::conv_narrow_kernel, dim3(blocks), dim3(64 * lbmnn::kW), 0, n->stream, n->act[l], ly.wn,
                         b, yout, ly.cout, n->g, n->V);
      e = hipGetLastError();
    } else if (ly.wq) {
      const int blocks = (n->g.nx / lbmnn::kTX) * (n->g.ny / lbmnn::kTY) * (n->g.nz / lbmnn::kTZ);
      if (direct)
        hipLaunchKernelGGL((lbmnn::conv_pair_kernel<true>), dim3(blocks), dim3(64 * lbmnn::kW), 0, n->stream, nullptr,
                           0, x, n->ch[0], n->mean, n->inv_std, ly.wq, b, 1, nullptr, n->act[l + 1], ly.cout, n->g,
                           n->V);
      else
        hipLaunchKernelGGL((lbmnn::conv_pair_kernel<false>), dim3(blocks), dim3(64 * lbmnn::kW), 0, n->stream,
                           n->act[l], 16, nullptr, 0, nullptr, nullptr, ly.wq, b, 1, nullptr, n->act[l + 1], ly.cout, n->g, n->V);
      e = hipGetLastError();
    } else if (ly.cinp == 16)
      e = last ? conv<16, true>(n, n->act[l], ly.wp, b, 0, nullptr, yout, ly.cout)
               : conv<16, false>(n, n->act[l], ly.wp, b, 1, nullptr, n->act[l + 1], ly.cout);
    else
      e = last ? conv<32, true>(n, n->act[l], ly.wp, b, 0, nullptr, yout, ly.cout)
               : conv<32, false>(n, n->act[l], ly.wp, b, 1, nullptr, n->act[l + 1], ly.cout);
    NN_HIP(e, "conv forward");
  }
  return LBM_OK;
}

}  // namespace

extern "C" {

int lbm_nn_create(lbm_nn* out, int layers, const int* channels, const int64_t dims[3]) {
  if (!out) return nn_fail(LBM_EINVAL, "lbm_nn_create: out is NULL");
  *out = nullptr;
  if (layers < 1 || !channels || !dims) return nn_fail(LBM_EINVAL, "lbm_nn_create: bad layer description");
  if (channels[0] < 1 || channels[0] > 16) return nn_fail(LBM_EINVAL, "lbm_nn_create: input channels must be 1..16");
  for (int l = 1; l < layers; ++l)
    if (channels[l] != 32) return nn_fail(LBM_EINVAL, "lbm_nn_create: hidden widths must be 32");
  if (channels[layers] < 1 || channels[layers] > 32)
    return nn_fail(LBM_EINVAL, "lbm_nn_create: output channels must be 1..32");
  for (int a = 0; a < 3; ++a)
    if (dims[a] < 1 || dims[a] > 4096) return nn_fail(LBM_EINVAL, "lbm_nn_create: dims out of range");
  const int64_t V = dims[0] * dims[1] * dims[2];
  if (dims[0] % lbmnn::kTX || dims[1] % lbmnn::kTY || dims[2] % lbmnn::kTZ || V > (1 << 26))
    return nn_fail(LBM_EINVAL, "lbm_nn_create: nx must be a multiple of 32, ny and nz of 4 (at most 2^26 nodes)");
  lbm_nn n = new (std::nothrow) lbm_nn_ctx();
  if (!n) return nn_fail(LBM_ENOMEM, "lbm_nn_create: host allocation failed");
  n->L = layers;
  n->ch.assign(channels, channels + layers + 1);
  n->g = {(int)dims[0], (int)dims[1], (int)dims[2]};
  n->V = (int)V;
  long long off = 0;
  for (int l = 0; l < layers; ++l) {
    Layer ly;
    ly.cin = channels[l];
    ly.cout = channels[l + 1];
    ly.cinp = l == 0 ? 16 : 32;
    ly.w_off = off;
    off += 27LL * ly.cin * ly.cout;
    ly.b_off = off;
    off += ly.cout;
    n->layers.push_back(ly);
  }
  n->nparam = off;
  int rc = LBM_OK;
  auto alloc = [&](void** p, size_t bytes) {
    if (rc != LBM_OK) return;
    const hipError_t e = hipMalloc(p, bytes);
    if (e != hipSuccess) rc = nn_hip(e, "lbm_nn_create: hipMalloc");
  };
  hipError_t e0 = hipGetDevice(&n->device);
  if (e0 != hipSuccess) rc = nn_hip(e0, "hipGetDevice");
  const size_t P = sizeof(float) * (size_t)off;
  alloc((void**)&n->params, P);
  alloc((void**)&n->grads, P);
  alloc((void**)&n->m, P);
  alloc((void**)&n->v, P);
  alloc((void**)&n->mean, 16 * sizeof(float));
  alloc((void**)&n->inv_std, 16 * sizeof(float));
  alloc((void**)&n->out_std, 32 * sizeof(float));
  alloc((void**)&n->inv_out_std, 32 * sizeof(float));
  n->act.assign(layers, nullptr);
  for (int l = 0; l < layers; ++l) alloc((void**)&n->act[l], sizeof(__bf16) * (size_t)V * (l == 0 ? 16 : 32));
  alloc((void**)&n->dA, sizeof(__bf16) * (size_t)V * 32);
  alloc((void**)&n->dB, sizeof(__bf16) * (size_t)V * 32);
  alloc((void**)&n->y, sizeof(float) * (size_t)V * 32);
  // The partials of all layers, so that one launch adds them up, or of four wide ones at the most.
  static_assert(lbmnn::kNMaxBlocks * 8 * 32 <= lbmnn::kGMaxBlocks * 1024, "a narrow layer's are no more than a wide one's");
  for (int l = 0; l < layers; ++l) {
    const Layer& ly = n->layers[l];
    int ntiles, tpb, nblk;
    gradient_blocks(n->g, ntiles, tpb, nblk, narrow_side(*n, l) ? lbmnn::kNMaxBlocks : lbmnn::kGMaxBlocks);
    n->part_size += (size_t)28 * nblk * ly.cin * ly.cout;
  }
  n->part_size = std::min(n->part_size, (size_t)4 * 28 * lbmnn::kGMaxBlocks * 1024);
  alloc((void**)&n->part, sizeof(float) * n->part_size);
  alloc((void**)&n->lpart, sizeof(double) * (size_t)((V + 255) / 256));
  alloc((void**)&n->loss_acc, sizeof(double));
  alloc((void**)&n->fld, sizeof(float) * 16 * (size_t)V);
  for (int l = 0; l < layers; ++l) {
    Layer& ly = n->layers[l];
    alloc((void**)&ly.wp, sizeof(__bf16) * 27 * ly.cinp * 32);
    if (narrow_output(*n, l)) alloc((void**)&ly.wr, sizeof(__bf16) * 14 * 32 * 16);
    else if (l > 0) alloc((void**)&ly.wb, sizeof(__bf16) * 27 * 32 * 32);
    if (l == layers - 1 && ly.cinp == 32 && ly.cout <= 16) alloc((void**)&ly.wn, sizeof(__bf16) * 27 * 16 * 32);
    if (l == 0 && layers > 1 && ly.cin <= 8) alloc((void**)&ly.wq, sizeof(__bf16) * 14 * 32 * 16);
  }
  if (rc == LBM_OK) {
    std::vector<float> mean(16, 0.f), one(32, 1.f);
    hipError_t e = hipMemset(n->params, 0, P);
    if (e == hipSuccess) e = hipMemset(n->grads, 0, P);
    if (e == hipSuccess) e = hipMemset(n->m, 0, P);
    if (e == hipSuccess) e = hipMemset(n->v, 0, P);
    if (e == hipSuccess) e = hipMemset(n->loss_acc, 0, sizeof(double));
    if (e == hipSuccess) e = hipMemcpy(n->mean, mean.data(), 16 * sizeof(float), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(n->inv_std, one.data(), 16 * sizeof(float), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(n->out_std, one.data(), 32 * sizeof(float), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(n->inv_out_std, one.data(), 32 * sizeof(float), hipMemcpyHostToDevice);
    if (e != hipSuccess) rc = nn_hip(e, "lbm_nn_create: initialise");
  }
  if (rc == LBM_OK) rc = nn_pack_weights(n);
  if (rc == LBM_OK) {
    const hipError_t e = hipStreamSynchronize(n->stream);
    if (e != hipSuccess) rc = nn_hip(e, "hipStreamSynchronize");
  }
  if (rc != LBM_OK) {
    lbm_nn_destroy(n);
    return rc;
  }
  *out = n;
  return LBM_OK;
}

int lbm_nn_destroy(lbm_nn n) {
  if (!n) return LBM_OK;
  (void)nn_select(n);
  if (n->stream) (void)hipStreamSynchronize(n->stream);
  for (void* p : {(void*)n->params, (void*)n->grads, (void*)n->m, (void*)n->v, (void*)n->mean, (void*)n->inv_std,
                  (void*)n->out_std, (void*)n->inv_out_std, (void*)n->dA, (void*)n->dB, (void*)n->y, (void*)n->part, (void*)n->lpart,
                  (void*)n->loss_acc, (void*)n->fld})
    if (p) (void)hipFree(p);
  for (__bf16* p : n->act)
    if (p) (void)hipFree(p);
  for (Layer& ly : n->layers) {
    if (ly.wp) (void)hipFree(ly.wp);
    if (ly.wb) (void)hipFree(ly.wb);
    if (ly.wn) (void)hipFree(ly.wn);
    if (ly.wq) (void)hipFree(ly.wq);
    if (ly.wr) (void)hipFree(ly.wr);
  }
  delete n;
  return LBM_OK;
}

int lbm_nn_set_stream(lbm_nn n, void* s) {
  if (!n) return nn_fail(LBM_EINVAL, "lbm_nn_set_stream: NULL network");
  n->stream = static_cast<hipStream_t>(s);
  return LBM_OK;
}

int64_t lbm_nn_param_count(lbm_nn n) { return n ? n->nparam : -1; }

int lbm_nn_set_params(lbm_nn n, const float* params, int mem) {
  if (!n || !params) return nn_fail(LBM_EINVAL, "lbm_nn_set_params: NULL argument");
  if (mem != LBM_HOST && mem != LBM_DEVICE) return nn_fail(LBM_EINVAL, "lbm_nn_set_params: bad memory kind");
  int rc = nn_select(n);
  if (rc) return rc;
  NN_HIP(hipMemcpyAsync(n->params, params, sizeof(float) * n->nparam,
                        mem == LBM_HOST ? hipMemcpyHostToDevice : hipMemcpyDeviceToDevice, n->stream),
         "copy params");
  if ((rc = nn_pack_weights(n))) return rc;
  NN_HIP(hipStreamSynchronize(n->stream), "hipStreamSynchronize");
  return LBM_OK;
}

static int nn_copy_out(lbm_nn n, float* dst, const float* src, int mem, const char* what) {
  if (!n || !dst) return nn_fail(LBM_EINVAL, std::string(what) + ": NULL argument");
  if (mem != LBM_HOST && mem != LBM_DEVICE) return nn_fail(LBM_EINVAL, std::string(what) + ": bad memory kind");
  int rc = nn_select(n);
  if (rc) return rc;
  NN_HIP(hipMemcpyAsync(dst, src, sizeof(float) * n->nparam,
                        mem == LBM_HOST ? hipMemcpyDeviceToHost : hipMemcpyDeviceToDevice, n->stream),
         what);
  NN_HIP(hipStreamSynchronize(n->stream), "hipStreamSynchronize");
  return LBM_OK;
}

int lbm_nn_get_params(lbm_nn n, float* p, int mem) { return nn_copy_out(n, p, n ? n->params : nullptr, mem, "lbm_nn_get_params"); }
int lbm_nn_get_grads(lbm_nn n, float* g, int mem) { return nn_copy_out(n, g, n ? n->grads : nullptr, mem, "lbm_nn_get_grads"); }

int lbm_nn_zero_grad(lbm_nn n) {
  if (!n) return nn_fail(LBM_EINVAL, "lbm_nn_zero_grad: NULL network");
  int rc = nn_select(n);
  if (rc) return rc;
  NN_HIP(hipMemsetAsync(n->grads, 0, sizeof(float) * n->nparam, n->stream), "zero grads");
  return LBM_OK;
}

int lbm_nn_set_scaling(lbm_nn n, const double* mean, const double* sd, const double* out_sd) {
  if (!n || !mean || !sd) return nn_fail(LBM_EINVAL, "lbm_nn_set_scaling: NULL argument");
  std::vector<float> m(16, 0.f), is(16, 1.f), os(32, 1.f), ios(32, 1.f);
  for (int c = 0; c < n->ch[0]; ++c) {
    if (!(sd[c] > 0.0) || !std::isfinite(sd[c]) || !std::isfinite(mean[c]))
      return nn_fail(LBM_EINVAL, "lbm_nn_set_scaling: std must be finite and > 0");
    m[c] = (float)mean[c];
    is[c] = (float)(1.0 / sd[c]);
  }
  const double* o = out_sd ? out_sd : sd;
  for (int c = 0; c < n->ch[n->L]; ++c) {
    if (!(o[c] > 0.0) || !std::isfinite(o[c]))
      return nn_fail(LBM_EINVAL, "lbm_nn_set_scaling: out_std must be finite and > 0");
    os[c] = (float)o[c];
    ios[c] = (float)(1.0 / o[c]);
  }
  int rc = nn_select(n);
  if (rc) return rc;
  NN_HIP(hipMemcpyAsync(n->mean, m.data(), 16 * sizeof(float), hipMemcpyHostToDevice, n->stream), "copy mean");
  NN_HIP(hipMemcpyAsync(n->inv_std, is.data(), 16 * sizeof(float), hipMemcpyHostToDevice, n->stream), "copy std");
  NN_HIP(hipMemcpyAsync(n->out_std, os.data(), 32 * sizeof(float), hipMemcpyHostToDevice, n->stream), "copy out_std");
  NN_HIP(hipMemcpyAsync(n->inv_out_std, ios.data(), 32 * sizeof(float), hipMemcpyHostToDevice, n->stream),
         "copy out_std");
  NN_HIP(hipStreamSynchronize(n->stream), "hipStreamSynchronize");
  return LBM_OK;
}

int lbm_nn_set_output_offset(lbm_nn n, int offset) {
  if (!n) return nn_fail(LBM_EINVAL, "lbm_nn_set_output_offset: NULL network");
  if (offset < 0 || offset + n->ch[n->L] > n->ch[0])
    return nn_fail(LBM_EINVAL, "lbm_nn_set_output_offset: offset + output channels must not exceed the input channels");
  n->out_off = offset;
  return LBM_OK;
}

int lbm_nn_set_correction_limit(lbm_nn n, double limit) {
  if (!n) return nn_fail(LBM_EINVAL, "lbm_nn_set_correction_limit: NULL network");
  if (!(limit >= 0.0) || !std::isfinite(limit))
    return nn_fail(LBM_EINVAL, "lbm_nn_set_correction_limit: limit must be finite and >= 0");
  n->limit = limit;
  return LBM_OK;
}

int lbm_nn_forward(lbm_nn n, const float* x, float* y) {
  if (!n || !x || !y) return nn_fail(LBM_EINVAL, "lbm_nn_forward: NULL argument");
  int rc = nn_select(n);
  if (rc) return rc;
  // inference: the first layer reads x directly and the last writes y
  return nn_forward(n, x, y, false);
}

int lbm_nn_loss_backward(lbm_nn n, const float* x, const float* target, double* loss) {
  if (!n || !x || !target) return nn_fail(LBM_EINVAL, "lbm_nn_loss_backward: NULL argument");
  if (n->out_off + n->ch[n->L] > n->ch[0])
    return nn_fail(LBM_EINVAL, "lbm_nn_loss_backward: output fields beyond the input fields");
  int rc = nn_select(n);
  if (rc) return rc;
  if ((rc = nn_forward(n, x))) return rc;
  const int V = n->V, C = n->ch[n->L];
  const int lblocks = (V + 255) / 256;
  const bool narrow = n->layers[n->L - 1].wr != nullptr;  // its gradient has 8 channels per node
  hipLaunchKernelGGL((narrow ? lbmnn::loss_kernel<8> : lbmnn::loss_kernel<32>), dim3(lblocks), dim3(256), 0, n->stream,
                     n->y, x, target, n->inv_out_std, C, n->out_off, V, n->dA, n->lpart);
  NN_HIP(hipGetLastError(), "loss kernel");
  // dA holds the gradient with respect to the output of layer l (pre-ReLU for l < L-1)
  __bf16 *dcur = n->dA, *dnext = n->dB;
  int ntiles, tpb, tpb_narrow, nblk, nblk_narrow;
  gradient_blocks(n->g, ntiles, tpb, nblk, lbmnn::kGMaxBlocks);
  gradient_blocks(n->g, ntiles, tpb_narrow, nblk_narrow, lbmnn::kNMaxBlocks);
  lbmnn::SumTable sums;
  size_t used = 0;  // floats of the partials that wait for their sum
  auto add_up = [&]() {
    const unsigned blocks = (unsigned)(sums.blocks + (sums.lpart ? 1 : 0));
    hipLaunchKernelGGL(lbmnn::wgrad_sum_kernel, dim3(blocks), dim3(64 * lbmnn::kGRuns), 0, n->stream, sums);
    sums = lbmnn::SumTable();
    used = 0;
    return hipGetLastError();
  };
  for (int l = n->L - 1; l >= 0; --l) {
    const Layer& ly = n->layers[l];
    const bool thin = narrow_side(*n, l);
    const int blocks = thin ? nblk_narrow : nblk;
    const size_t need = (size_t)28 * blocks * ly.cin * ly.cout;
    if (sums.layers == lbmnn::kSumLayers || used + need > n->part_size) NN_HIP(add_up(), "weight gradient sums");
    float* part = n->part + used;
    used += need;
    if (ly.wr)
      hipLaunchKernelGGL((lbmnn::wgrad_narrow_kernel<false>), dim3(blocks), dim3(512), 0, n->stream, n->act[l], dcur, 8,
                         part, n->g, ntiles, tpb_narrow, ly.cin, ly.cout);
    else if (thin)
      hipLaunchKernelGGL((lbmnn::wgrad_narrow_kernel<true>), dim3(blocks), dim3(512), 0, n->stream, dcur, n->act[l], 16,
                         part, n->g, ntiles, tpb_narrow, ly.cin, ly.cout);
    else if (ly.cinp == 16)
      hipLaunchKernelGGL((lbmnn::wgrad_kernel<16>), dim3(blocks), dim3(512), 0, n->stream, n->act[l], dcur, part, n->g,
                         ntiles, tpb, ly.cin, ly.cout);
    else
      hipLaunchKernelGGL((lbmnn::wgrad_kernel<32>), dim3(blocks), dim3(512), 0, n->stream, n->act[l], dcur, part, n->g,
                         ntiles, tpb, ly.cin, ly.cout);
    NN_HIP(hipGetLastError(), "weight gradient kernel");
    sums.layer[sums.layers++] = {part, n->grads + ly.w_off, n->grads + ly.b_off, blocks, ly.cin, ly.cout, sums.blocks};
    sums.blocks += (ly.cin * ly.cout + 63) / 64 * 28;
    if (l > 0) {
      // gradient with respect to this layer's input = previous output; times the ReLU derivative
      if (ly.wr) {
        const int tiles = (n->g.nx / lbmnn::kTX) * (n->g.ny / lbmnn::kTY) * (n->g.nz / lbmnn::kTZ);
        hipLaunchKernelGGL((lbmnn::conv_pair_kernel<false>), dim3(tiles), dim3(64 * lbmnn::kW), 0, n->stream, dcur, 8,
                           nullptr, 0, nullptr, nullptr, ly.wr, nullptr, 0, n->act[l], dnext, 32, n->g, V);
        NN_HIP(hipGetLastError(), "conv backward-data");
      } else {
        NN_HIP((conv<32, false>(n, dcur, ly.wb, nullptr, 0, n->act[l], dnext, 32)), "conv backward-data");
      }
      __bf16* t = dcur;
      dcur = dnext;
      dnext = t;
    }
  }
  if (!loss) {
    sums.lpart = n->lpart;
    sums.lcount = lblocks;
    sums.lscale = 1.0 / ((double)C * V);
    sums.loss = n->loss_acc;
  }
  NN_HIP(add_up(), "weight gradient sums");
  if (loss) {
    std::vector<double> h(lblocks);
    NN_HIP(hipMemcpyAsync(h.data(), n->lpart, sizeof(double) * lblocks, hipMemcpyDeviceToHost, n->stream),
           "copy loss");
    NN_HIP(hipStreamSynchronize(n->stream), "hipStreamSynchronize");
    double s = 0.0;
    for (double x2 : h) s += x2;
    *loss = s / ((double)C * V);
  } else {
    ++n->loss_count;
  }
  return LBM_OK;
}

int lbm_nn_take_loss(lbm_nn n, double* sum, int64_t* count) {
  if (!n || !sum) return nn_fail(LBM_EINVAL, "lbm_nn_take_loss: NULL argument");
  int rc = nn_select(n);
  if (rc) return rc;
  NN_HIP(hipMemcpyAsync(sum, n->loss_acc, sizeof(double), hipMemcpyDeviceToHost, n->stream), "copy loss sum");
  NN_HIP(hipMemsetAsync(n->loss_acc, 0, sizeof(double), n->stream), "reset loss sum");
  NN_HIP(hipStreamSynchronize(n->stream), "hipStreamSynchronize");
  if (count) *count = n->loss_count;
  n->loss_count = 0;
  return LBM_OK;
}

int lbm_nn_adam_step(lbm_nn n, double lr, double beta1, double beta2, double eps, double grad_scale, int64_t t) {
  if (!n) return nn_fail(LBM_EINVAL, "lbm_nn_adam_step: NULL network");
  if (t < 1 || !(lr > 0.0) || !(beta1 >= 0.0 && beta1 < 1.0) || !(beta2 >= 0.0 && beta2 < 1.0) || !(eps > 0.0))
    return nn_fail(LBM_EINVAL, "lbm_nn_adam_step: bad hyper-parameters");
  int rc = nn_select(n);
  if (rc) return rc;
  const float c1 = (float)(1.0 / (1.0 - std::pow(beta1, (double)t)));
  const float c2 = (float)(1.0 / (1.0 - std::pow(beta2, (double)t)));
  hipLaunchKernelGGL(lbmnn::adam_kernel, dim3((unsigned)((n->nparam + 255) / 256)), dim3(256), 0, n->stream,
                     n->params, n->grads, n->m, n->v, n->nparam, (float)lr, (float)beta1, (float)beta2, (float)eps,
                     (float)grad_scale, c1, c2);
  NN_HIP(hipGetLastError(), "adam kernel");
  return nn_pack_weights(n);
}

int lbm_nn_fields_to_planes(int D, int64_t nodes, const double* rho, const double* u, const double* T, float* x,
                            void* stream) {
  if (!rho || !u || !T || !x) return nn_fail(LBM_EINVAL, "lbm_nn_fields_to_planes: NULL argument");
  if ((D != 2 && D != 3) || nodes < 1 || nodes > (1LL << 31) - 256)
    return nn_fail(LBM_EINVAL, "lbm_nn_fields_to_planes: bad lattice or node count");
  const int V = (int)nodes;
  hipLaunchKernelGGL(lbmnn::fields_to_input_kernel, dim3((V + 255) / 256), dim3(256), 0,
                     static_cast<hipStream_t>(stream), rho, u, T, D, V, x);
  NN_HIP(hipGetLastError(), "fields kernel");
  return LBM_OK;
}

int lbm_nn_correct(lbm_nn n, lbm_handle h) {
  if (!n || !h) return nn_fail(LBM_EINVAL, "lbm_nn_correct: NULL argument");
  const int D = h->lattice;
  if (n->ch[0] != D + 2 || n->out_off + n->ch[n->L] > D + 2)
    return nn_fail(LBM_EINVAL, "lbm_nn_correct: the network must read the D + 2 fields and correct fields among them");
  if (D != 3) return nn_fail(LBM_EINVAL, "lbm_nn_correct: networks are three-dimensional, the handle is not");
  if (h->n[0] != n->g.nx || h->n[1] != n->g.ny || h->n[2] != n->g.nz)
    return nn_fail(LBM_EINVAL, "lbm_nn_correct: grid of the handle differs from the network's");
  int rc = nn_select(n);
  if (rc) return rc;
  // everything on the handle's stream: planes, network, re-equilibration
  hipStream_t saved = n->stream;
  n->stream = h->stream;
  rc = lbm::corrector_planes(h, n->fld);
  if (rc == LBM_OK) rc = nn_forward(n, n->fld, nullptr, false);
  if (rc == LBM_OK)
    rc = lbm::corrector_apply(h, n->y, n->out_std, n->ch[n->L], n->out_off, (float)n->limit);
  n->stream = saved;
  return rc;
}

}  // extern "C"

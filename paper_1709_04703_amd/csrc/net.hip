// Learned warm start for the multigrid solve: a 5-layer 3x3x3 convolution
// net with 16 channels (ReLU between layers, periodic padding), BF16 weights
// and activations, FP32 accumulation on the matrix cores of gfx950.
//
// Each layer is an implicit GEMM over taps t:  Out^T (16 co x voxels) +=
// W_t^T (16 co x 16 ci) * In_t^T (16 ci x voxels).  Activations are stored
// channels-last (16 BF16 = 32 B per voxel), so a lane's B fragment (8
// channels of one voxel) is one 16-byte read and its D fragment (4 channels of
// one voxel) one 8-byte write.  MFMA lane layout (64 lanes, g = lane / 16, r =
// lane % 16), 16x16x32: A[r][8g..8g+7], B[8g..8g+7][r], D[4g..4g+3][r].
//
// The data gradient of a layer is the same kernel with the taps mirrored and
// the channel roles swapped (BACKWARD flag); the weight gradient reduces
// In^T * G over voxels on the matrix cores, per workgroup, then in a fixed
// order over workgroups (deterministic).
#include <algorithm>
#include <cmath>

#include "internal.h"

namespace sdpm {
namespace {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// 16 bytes from memory of the callers' own alignment (2 bytes for BF16
// activations, 4 for FP32 scratch)
typedef uint32_t u32x4_a2 __attribute__((ext_vector_type(4), aligned(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));

constexpr int kNC = 16;                 // channels

__device__ inline uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return 0x7fc0;       // NaN stays NaN
  u += 0x7fffu + ((u >> 16) & 1u);                           // round to nearest even
  return (uint16_t)(u >> 16);
}
__device__ inline float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ inline int64_t vox(int i, int j, int k, int n) { return ((int64_t)k * n + j) * n + i; }

// ---------------------------------------------------------------- forward
// flags: 1 ReLU, 2 FP32 output of channel 0 only, 4 backward-data (mirrored
// taps, swapped channels, no bias), 8 multiply by [mask > 0].
//
// v_mfma_f32_16x16x32_bf16 (K = 32: two taps of 16 input channels at once;
// gfx950 runs it at twice the rate of the K = 16 form).  Lane layout (g =
// lane / 16, r = lane % 16): A[r][8g .. 8g+7], B[8g .. 8g+7][r],
// D[4g .. 4g+3][r].  Taps are paired along x: one MFMA takes dx = -1 (k < 16)
// and dx = 0 (k >= 16) of an input row, a second dx = +1 (k < 16; the other
// half has zero weights).
//
// A workgroup takes a column of 64 voxels in x (its 4 waves 16 each) and kCY
// rows and marches the input planes of its zc output planes.  Only one input
// plane is needed at a time: a wave reads each of its kCY + 2 rows once and
// adds it to the up to nine output rows it feeds, in three planes of
// accumulators (the plane that starts with this input plane, the one in its
// middle, the one it completes), whose roles rotate (the loop is unrolled by
// three so that they stay in registers).  Two LDS slots take the planes in
// turn; the next plane's global loads are in flight during a plane's
// products, and one barrier per plane separates writes from reads.  The
// weights stay in registers.  A tap's contributions are added plane by plane
// and row by row, as in a block of planes held at once, so results do not
// depend on zc.
// 128^3 takes 57 us forward and 69 us backward with the mask, 256^3 346 and 428
// us (blocks of 4 planes loaded between barriers, one workgroup per CU at 128^3:
// 96, 120, 552 and 705 us).  Neither HBM nor LDS bounds it (counters at 128^3:
// 107 MB, 2.3 TB/s, half a copy's rate; LDS active 9 % of the time, no bank
// conflicts): the matrix cores are busy 41 % of the time, a quarter of it on the
// second fragment's zero half, other vector instructions issue for about 28 %,
// and a wave waits for memory or a barrier for 36 %.  With the mask the waits
// are 56 %, the matrix cores 28 %.  252 registers, two waves per SIMD; with the
// mask 215 for 4 rows, and 256 with 58 spilled for 8.
typedef short bf16x8 __attribute__((ext_vector_type(8)));
constexpr int kBX = 64 + 2;

template <int FLAGS, int kCY>
__global__ void __launch_bounds__(256, 2)
k_conv(int n, int zc, const uint16_t* __restrict__ in, const float* __restrict__ w,
       const float* __restrict__ bias, const uint16_t* __restrict__ mask, void* __restrict__ out) {
  constexpr bool RELU = FLAGS & 1, OUT0 = FLAGS & 2, BWD = FLAGS & 4, MASK = FLAGS & 8;
  constexpr int kBY = kCY + 2;
  constexpr int kBUnits = kBY * kBX * 2;           // 16-byte units of an input plane's tile
  constexpr int kBLoads = (kBUnits + 255) / 256;   // per thread
  __shared__ u32x4 blk[2][kBUnits];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int g = lane >> 4, r = lane & 15, hi = g >> 1, cg = g & 1;
  const int m = n - 1;
  const int gx = (n + 63) / 64, gy = n / kCY;
  const int b = (int)xcd_block();
  const int bx = b % gx, by = (b / gx) % gy, bz = b / (gx * gy);
  const int x0 = bx * 64, y0 = by * kCY, z0 = bz * zc;
  const int zn = min(zc, n - z0);                // output planes z0 .. z0 + zn - 1
  // this thread's units of a plane's tile (rows y0 - 1 .. y0 + kCY, voxels
  // x0 - 1 .. x0 + 64, two units per voxel): offsets within a plane
  int off[kBLoads];
#pragma unroll
  for (int u = 0; u < kBLoads; ++u) {
    const int c = tid + 256 * u, v = c >> 1;
    const int px = v % kBX, py = v / kBX;
    off[u] = (((y0 - 1 + py) & m) * n + ((x0 - 1 + px) & m)) * 2 + (c & 1);
  }
  u32x4 nxt[kBLoads];
  auto load = [&](int z) {
    const u32x4* p = (const u32x4*)(in + (int64_t)(z & m) * n * n * kNC);
#pragma unroll
    for (int u = 0; u < kBLoads; ++u)
      if (tid + 256 * u < kBUnits) nxt[u] = p[off[u]];
  };
  auto store = [&](int slot) {
#pragma unroll
    for (int u = 0; u < kBLoads; ++u)
      if (tid + 256 * u < kBUnits) blk[slot][tid + 256 * u] = nxt[u];
  };
  load(z0 - 1);
  // weight fragments per (dy, dz): a01 = taps dx = -1 (k < 16), dx = 0 (k >= 16);
  // a2 = tap dx = +1 (k < 16), zero for k >= 16.  Element j of lane (g, r):
  // input channel 8 cg + j, output channel r.
  bf16x8 a01[9], a2[9];
#pragma unroll
  for (int yz = 0; yz < 9; ++yz) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int ci = 8 * cg + j;
      const int t01 = yz * 3 + (hi ? 1 : 0), t2 = yz * 3 + 2;
      const float v01 = BWD ? w[((26 - t01) * kNC + r) * kNC + ci] : w[(t01 * kNC + ci) * kNC + r];
      const float v2 = BWD ? w[((26 - t2) * kNC + r) * kNC + ci] : w[(t2 * kNC + ci) * kNC + r];
      a01[yz][j] = (short)f2bf(v01);
      a2[yz][j] = hi ? (short)0 : (short)f2bf(v2);
    }
  }
  float bq[4] = {0.f, 0.f, 0.f, 0.f};
  if (!BWD && bias) {
#pragma unroll
    for (int q = 0; q < 4; ++q) bq[q] = bias[4 * g + q];
  }
  store(0);
  __syncthreads();
  f32x4 acc[3][kCY];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int y = 0; y < kCY; ++y) acc[a][y] = f32x4{0.f, 0.f, 0.f, 0.f};
  // output voxel x0 + 16 wave + r reads tile column 16 wave + r + 1 + dx
  const int col = 16 * wave + r + 1;
  const int x = (x0 + 16 * wave + r) & m;
  // step s takes input plane z0 - 1 + s: dz = -1 of output plane s (which it
  // starts), dz = 0 of s - 1, dz = +1 of s - 2 (which it completes)
  for (int s0 = 0; s0 < zn + 2; s0 += 3) {
#pragma unroll
    for (int q3 = 0; q3 < 3; ++q3) {
      const int s = s0 + q3;
      if (s >= zn + 2) break;                    // uniform
      if (s + 1 < zn + 2) load(z0 + s);
      const bool done = s >= 2;
      const int zo = z0 + s - 2;
      bf16x4 mk[MASK ? kCY : 1];
      if (MASK && done) {
#pragma unroll
        for (int y = 0; y < kCY; ++y)
          mk[y] = *(const bf16x4*)(mask + vox(x, y0 + y, zo, n) * kNC + 4 * g);
      }
#pragma unroll
      for (int y = 0; y < kCY; ++y) acc[q3][y] = f32x4{0.f, 0.f, 0.f, 0.f};
      const u32x4* tile = blk[s & 1];
#pragma unroll
      for (int py = 0; py < kBY; ++py) {
        // F01: k < 16 from x - 1, k >= 16 from x; F2: x + 1 (both halves)
        const bf16x8 f01 = *(const bf16x8*)&tile[(py * kBX + col - 1 + hi) * 2 + cg];
        const bf16x8 f2 = *(const bf16x8*)&tile[(py * kBX + col + 1) * 2 + cg];
#pragma unroll
        for (int dz = -1; dz <= 1; ++dz) {
          f32x4* ac = acc[(q3 + 3 - (dz + 1)) % 3];
#pragma unroll
          for (int dy = -1; dy <= 1; ++dy) {
            const int oy = py - 1 - dy;
            if (oy < 0 || oy >= kCY) continue;
            const int yz = (dz + 1) * 3 + (dy + 1);
            ac[oy] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a01[yz], f01, ac[oy], 0, 0, 0);
            ac[oy] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a2[yz], f2, ac[oy], 0, 0, 0);
          }
        }
      }
      if (done) {
        // D[co = 4g + q][voxel = r] of each output row
#pragma unroll
        for (int y = 0; y < kCY; ++y) {
          const int64_t v = vox(x, y0 + y, zo, n);
          float val[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            float a = acc[(q3 + 1) % 3][y][q] + bq[q];
            if (RELU) a = a > 0.f ? a : 0.f;
            val[q] = a;
          }
          if (MASK) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
              if (!(bf2f((uint16_t)mk[y][q]) > 0.f)) val[q] = 0.f;
          }
          if (OUT0) {
            if (g == 0) ((float*)out)[v] = val[0];
          } else {
            bf16x4 o;
#pragma unroll
            for (int q = 0; q < 4; ++q) o[q] = (short)f2bf(val[q]);
            *(bf16x4*)((uint16_t*)out + v * kNC + 4 * g) = o;
          }
        }
      }
      if (s + 1 < zn + 2) store((s + 1) & 1);
      __syncthreads();
    }
  }
}

// ---------------------------------------------------------- weight gradient
// dW[t][ci][co] = sum_v in[v + off_t][ci] g[v][co]; db[co] = sum_v g[v][co].
// On the matrix cores with the voxels of a row as the contraction index:
// D (ci x co) += A (ci x 32 voxels) * B (32 voxels x co), a lane's fragment
// being 8 consecutive voxels of one channel.  Activations are channels-last,
// so both operands are staged transposed in LDS ([row][channel][x]): a thread
// loads 8 channels of two neighbouring voxels and writes 8 dwords.
//
// A workgroup of 8 waves takes a column of kWX voxels in x and 8 rows and
// marches its planes; it owns the products whose g voxel lies in its x range
// and whose input row is one of its rows (in: one voxel of halo in x; g: one
// row and plane of halo in y and z).  Each wave owns one input row: it reads
// the row's fragment once, forms its x +- 1 shifts in registers (a fragment
// shifted by one 2-byte voxel is not aligned in LDS), and multiplies the
// three with the fragments of the nine g rows that row pairs with.  g planes
// sit in a ring of 4, input planes in a ring of 2, so one barrier per plane
// separates writes from reads, and the next plane's global loads are in
// flight during the products.  db is one more product, with A = 1.
// Bound by the matrix cores and LDS reads (10.5 KB per 28 products).  Row
// strides of 88 and 72 entries put the 16 channels of a fragment read on
// distinct banks.  At 128^3 it takes 50 us (0.58 PFLOP/s); with one
// 2-byte global load per voxel, channel and tap it took 716 us.
constexpr int kWG = 27 * kNC * kNC + kNC;   // partial size per workgroup
constexpr int kWX = 64, kWY = 8;            // voxels in x and rows of a workgroup
constexpr int kWInS = 88, kWGrS = 72;       // LDS entries per (row, channel)
constexpr int kWIn = kWY * kNC * kWInS, kWGr = (kWY + 2) * kNC * kWGrS;   // per plane
constexpr int kWLds = 2 * kWIn + 4 * kWGr;  // entries of 2 bytes

// two neighbouring voxels' 8 channels -> one dword (x, x + 1) per channel
__device__ inline void wg_store_pair(uint16_t* dst, int stride, const u32x4_a2& a, const u32x4_a2& b) {
  const uint32_t av[4] = {a.x, a.y, a.z, a.w}, bv[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    *(uint32_t*)(dst + (2 * c) * stride) = (av[c] & 0xffffu) | (bv[c] << 16);
    *(uint32_t*)(dst + (2 * c + 1) * stride) = (av[c] >> 16) | (bv[c] & 0xffff0000u);
  }
}

__global__ void __launch_bounds__(512)
k_conv_wgrad(int n, int zc, const uint16_t* __restrict__ in, const uint16_t* __restrict__ gr,
             float* __restrict__ partial) {
  __shared__ __attribute__((aligned(16))) uint16_t lds[kWLds];
  uint16_t* const lin = lds;
  uint16_t* const lgr = lds + 2 * kWIn;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int g = lane >> 4, r = lane & 15;
  const int m = n - 1;
  const int xt = n < kWX ? n : kWX, chunks = xt > 32 ? 2 : 1;
  const int gx = n / xt, gy = n / kWY;
  const int bx = blockIdx.x % gx, by = (blockIdx.x / gx) % gy, bz = blockIdx.x / (gx * gy);
  const int x0 = bx * xt, y0 = by * kWY, z0 = bz * zc;
  const int zn = min(zc, n - z0);
  // rows shorter than a product's 32 voxels: the rest of g stays zero
  if (xt < kWX)
    for (int c = tid; c < kWLds / 2; c += 512) ((uint32_t*)lds)[c] = 0u;
  // this thread's loads: one voxel pair of the input plane and up to two of
  // the g plane (640 pairs), 8 channels each; threads below 32 one halo voxel
  const int half = tid & 1, pair = (tid >> 1) & 31, row = tid >> 6;
  const bool inx = 2 * pair < xt;
  u32x4_a2 ia, ib, ga[2], gb[2], ha;
  auto load_in = [&](int z) {
    const int zz = z & m;
    if (inx) {
      const u32x4_a2* s = (const u32x4_a2*)(in + vox(x0 + 2 * pair, y0 + row, zz, n) * kNC) + half;
      ia = s[0];
      ib = s[2];
    }
    if (tid < 32) {
      const int xh = (tid & 2) ? x0 + xt : x0 - 1;
      ha = ((const u32x4_a2*)(in + vox(xh & m, y0 + (tid >> 2), zz, n) * kNC))[half];
    }
  };
  auto store_in = [&](int z) {
    uint16_t* p = lin + (z & 1) * kWIn;
    if (inx) wg_store_pair(p + (row * kNC + 8 * half) * kWInS + 8 + 2 * pair, kWInS, ia, ib);
    if (tid < 32) {
      uint16_t* q = p + ((tid >> 2) * kNC + 8 * half) * kWInS + ((tid & 2) ? 8 + xt : 7);
      const uint32_t hv[4] = {ha.x, ha.y, ha.z, ha.w};
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        q[(2 * c) * kWInS] = (uint16_t)hv[c];
        q[(2 * c + 1) * kWInS] = (uint16_t)(hv[c] >> 16);
      }
    }
  };
  auto load_gr = [&](int z) {
    const int zz = z & m;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int rw = row + 8 * u;
      if (rw < kWY + 2 && inx) {
        const u32x4_a2* s =
            (const u32x4_a2*)(gr + vox(x0 + 2 * pair, (y0 - 1 + rw) & m, zz, n) * kNC) + half;
        ga[u] = s[0];
        gb[u] = s[2];
      }
    }
  };
  auto store_gr = [&](int z) {
    uint16_t* p = lgr + ((z + 4) & 3) * kWGr;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int rw = row + 8 * u;
      if (rw < kWY + 2 && inx)
        wg_store_pair(p + (rw * kNC + 8 * half) * kWGrS + 2 * pair, kWGrS, ga[u], gb[u]);
    }
  };
  f32x4 acc[28];
#pragma unroll
  for (int t = 0; t < 28; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  bf16x8 ones;
#pragma unroll
  for (int j = 0; j < 8; ++j) ones[j] = (short)0x3f80;
  if (xt < kWX) __syncthreads();
  // planes are counted from the workgroup's first (z0): g planes -1, 0, 1
  // and input plane 0 are in LDS before the first products
  for (int z = -1; z <= 1; ++z) {
    load_gr(z0 + z);
    store_gr(z);
  }
  load_in(z0);
  store_in(0);
  __syncthreads();
  for (int z = 0; z < zn; ++z) {
    const bool more = z + 1 < zn;
    if (more) {
      load_in(z0 + z + 1);
      load_gr(z0 + z + 2);
    }
    const uint16_t* pin = lin + (z & 1) * kWIn + (wave * kNC + r) * kWInS + 8;
    for (int ch = 0; ch < chunks; ++ch) {
      const uint16_t* pi = pin + 32 * ch + 8 * g;
      uint4 f = *(const uint4*)pi;
      uint32_t before = *(const uint32_t*)(pi - 2), after = *(const uint32_t*)(pi + 8);
      // a row of 16 voxels fills half of the product: its other half, where
      // g is zero, must not multiply the halo's values (they may be infinite)
      if (8 * g >= xt) f = uint4{0u, 0u, 0u, 0u}, before = after = 0u;
      union { uint32_t u[4]; bf16x8 v; } a[3];
      a[0].u[0] = __builtin_amdgcn_alignbit(f.x, before, 16);
      a[0].u[1] = __builtin_amdgcn_alignbit(f.y, f.x, 16);
      a[0].u[2] = __builtin_amdgcn_alignbit(f.z, f.y, 16);
      a[0].u[3] = __builtin_amdgcn_alignbit(f.w, f.z, 16);
      a[1].u[0] = f.x, a[1].u[1] = f.y, a[1].u[2] = f.z, a[1].u[3] = f.w;
      a[2].u[0] = a[0].u[1], a[2].u[1] = a[0].u[2], a[2].u[2] = a[0].u[3];
      a[2].u[3] = __builtin_amdgcn_alignbit(after, f.w, 16);
      // input row y0 + wave, plane z pairs with g row y0 + wave - dy (entry
      // wave + 1 - dy of the tile) of plane z - dz for tap (dx, dy, dz)
#pragma unroll
      for (int dz = -1; dz <= 1; ++dz) {
#pragma unroll
        for (int dy = -1; dy <= 1; ++dy) {
          const bf16x8 b = *(const bf16x8*)(lgr + ((z - dz + 4) & 3) * kWGr +
                                            ((wave + 1 - dy) * kNC + r) * kWGrS + 32 * ch + 8 * g);
          const int t = (dz + 1) * 9 + (dy + 1) * 3;
#pragma unroll
          for (int q = 0; q < 3; ++q)
            acc[t + q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[q].v, b, acc[t + q], 0, 0, 0);
          if (dz == 0 && dy == 0)
            acc[27] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, b, acc[27], 0, 0, 0);
        }
      }
    }
    if (more) {
      store_in(z + 1);
      store_gr(z + 2);
    }
    __syncthreads();
  }
  // sum of the 8 waves, pairwise in a fixed order: D[ci = 4g + q][co = r]
  // (of the bias product every row ci holds the sum)
  float* red = (float*)lds;
  static_assert(4 * 28 * 256 * sizeof(float) <= sizeof(lds), "partials of four waves fit");
#pragma unroll
  for (int w = 4; w > 0; w >>= 1) {
    if (wave >= w && wave < 2 * w) {
#pragma unroll
      for (int t = 0; t < 28; ++t)
        *(f32x4*)(red + ((wave - w) * 28 + t) * 256 + 4 * lane) = acc[t];
    }
    __syncthreads();
    if (wave < w) {
#pragma unroll
      for (int t = 0; t < 28; ++t) acc[t] += *(const f32x4*)(red + (wave * 28 + t) * 256 + 4 * lane);
    }
    __syncthreads();
  }
  if (wave == 0) {
    float* dst = partial + (int64_t)blockIdx.x * kWG;
#pragma unroll
    for (int t = 0; t < 27; ++t)
#pragma unroll
      for (int q = 0; q < 4; ++q) dst[(t * kNC + 4 * g + q) * kNC + r] = acc[t][q];
    if (g == 0) dst[27 * kNC * kNC + r] = acc[27][0];
  }
}

// out[c] = sum over workgroups of partial[b][c] in a fixed order: 64 entries
// per workgroup, the partials split over its 16 groups of 16 lanes (four
// entries each), four sums in flight per lane: 4.8 us for 256 partials.  (One
// thread per entry, a serial chain of loads, took 242 us for 1024 partials.)
constexpr int kWRed = 64;
__global__ void __launch_bounds__(256)
k_wgrad_reduce(const float* __restrict__ partial, int nblocks, float* __restrict__ dw,
               float* __restrict__ db) {
  __shared__ f32x4 sh[256];
  const int tid = threadIdx.x, e = tid & 15, s = tid >> 4;
  const int c = blockIdx.x * kWRed + 4 * e;
  f32x4 v[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) v[u] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (c < kWG) {                               // kWG is a multiple of 4
    int b = s;
    for (; b + 48 < nblocks; b += 64)
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] += *(const f32x4_a4*)(partial + (int64_t)(b + 16 * u) * kWG + c);
    for (; b < nblocks; b += 16) v[0] += *(const f32x4_a4*)(partial + (int64_t)b * kWG + c);
  }
  sh[tid] = (v[0] + v[1]) + (v[2] + v[3]);
  __syncthreads();
  for (int off = 8; off > 0; off >>= 1) {
    if (s < off) sh[tid] += sh[tid + 16 * off];
    __syncthreads();
  }
  if (s == 0 && c < kWG) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (c + q < 27 * kNC * kNC)
        dw[c + q] = sh[e][q];
      else
        db[c + q - 27 * kNC * kNC] = sh[e][q];
    }
  }
}

// ------------------------------------------------------------- inputs, loss
// act0[v] = (r[v] s_r, phi[v] s_phi, kap, 0, ...) in BF16.  RT / PT: input types;
// SPLIT: r stored colour-split; with a box, r outside it counts as zero.
template <typename RT, typename PT, bool SPLIT>
__global__ void __launch_bounds__(256)
k_net_prep(int n, const RT* __restrict__ r, const PT* __restrict__ phi, float s_r, float s_phi,
           float kap, Box b, int use_box, uint16_t* __restrict__ act0) {
  const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t V = (int64_t)n * n * n;
  if (v >= V) return;
  const int i = (int)(v % n), j = (int)((v / n) % n), k = (int)(v / ((int64_t)n * n));
  float rv = 0.f;
  const bool in_box = !use_box || (i >= b.lo[0] && i <= b.hi[0] && j >= b.lo[1] && j <= b.hi[1] &&
                                   k >= b.lo[2] && k <= b.hi[2]);
  if (in_box) {
    const int64_t hc = (int64_t)n * n * (n >> 1);
    const int64_t ri = SPLIT ? ((int64_t)((i + j + k) & 1) * hc + ((int64_t)k * n + j) * (n >> 1) + (i >> 1)) : v;
    rv = (float)r[ri] * s_r;
  }
  const float pv = (float)phi[v] * s_phi;
  uint4 o0, o1;
  o0.x = (uint32_t)f2bf(rv) | ((uint32_t)f2bf(pv) << 16);
  o0.y = (uint32_t)f2bf(kap);
  o0.z = o0.w = 0u;
  o1.x = o1.y = o1.z = o1.w = 0u;
  ((uint4*)(act0 + v * kNC))[0] = o0;
  ((uint4*)(act0 + v * kNC))[1] = o1;
}

// g[v] = (2 (out - tscale target) gscale, 0, ...) in BF16; partial sum of
// (out - tscale target)^2.
__global__ void __launch_bounds__(256)
k_net_loss(int64_t V, const float* __restrict__ out, const float* __restrict__ target, float tscale,
           float gscale, uint16_t* __restrict__ g, float* __restrict__ partial) {
  __shared__ float sh[4];
  const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
  float d = 0.f;
  if (v < V) {
    d = out[v] - target[v] * tscale;
    uint4 o0, o1;
    o0.x = (uint32_t)f2bf(2.f * d * gscale);
    o0.y = o0.z = o0.w = 0u;
    o1.x = o1.y = o1.z = o1.w = 0u;
    ((uint4*)(g + v * kNC))[0] = o0;
    ((uint4*)(g + v * kNC))[1] = o1;
  }
  float s = d * d;
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) partial[blockIdx.x] = sh[0] + sh[1] + sh[2] + sh[3];
}

__global__ void __launch_bounds__(256)
k_sum_partials(const float* __restrict__ partial, int np, float scale, float* __restrict__ out) {
  __shared__ float sh[256];
  float s = 0.f;
  for (int q = threadIdx.x; q < np; q += 256) s += partial[q];
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if (threadIdx.x < off) sh[threadIdx.x] += sh[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = sh[0] * scale;
}

// Adam on the FP32 master parameters; the input channels >= 2 of layer 0 and
// the output channels >= 1 of layer 4 stay zero.
__global__ void __launch_bounds__(256)
k_adam(int np, float* __restrict__ p, const float* __restrict__ grad, float* __restrict__ m1,
       float* __restrict__ m2, float lr, float b1, float b2, float eps, float c1, float c2) {
  const int q = blockIdx.x * 256 + threadIdx.x;
  if (q >= np) return;
  const int per = 27 * kNC * kNC + kNC;
  const int l = q / per, o = q % per;
  bool frozen = false;
  if (o < 27 * kNC * kNC) {
    const int ci = (o / kNC) % kNC, co = o % kNC;
    frozen = (l == 0 && ci >= kNetInputs) || (l == 4 && co >= 1);
  } else {
    frozen = (l == 4 && o - 27 * kNC * kNC >= 1);
  }
  if (frozen) {
    p[q] = 0.f;
    return;
  }
  const float gq = grad[q];
  const float a = b1 * m1[q] + (1.f - b1) * gq;
  const float b = b2 * m2[q] + (1.f - b2) * gq * gq;
  m1[q] = a;
  m2[q] = b;
  p[q] -= lr * (a / c1) / (sqrtf(b / c2) + eps);
}

// Rows per workgroup of a layer: 8 read fewer halo rows (1.25x against 1.5x);
// with the mask their accumulators, weights and prefetched values need more
// than the 256 registers of two waves per SIMD, and 4 rows are faster where
// the grid fills the card (256^3: 428 against 535 us, 128^3: 69 against 87 us;
// 64^3: 36 against 30 us; without the mask 256^3: 356 against 346 us).
int conv_rows(int n, int flags) { return (flags & 8) && n >= 128 ? 4 : 8; }
// Output planes per workgroup: about 512 workgroups (two per CU, so that one's
// products cover the other's barriers; 1024 measured 79 against 57 us at
// 128^3), at least 2 planes each (a workgroup reads two more).
int conv_planes(int n, int rows) {
  const int columns = ((n + 63) / 64) * (n / rows);
  return std::max(2, std::min<int>(n, (int)((int64_t)n * columns / 512)));
}
// Planes per workgroup of the weight gradient: about 256 workgroups (one per
// CU: a workgroup's LDS takes most of one), at least 4 planes each (two more
// g planes are staged per workgroup, and its partial is written and summed).
int wgrad_planes(int n) {
  const int columns = (n / std::min(n, kWX)) * (n / kWY);
  return std::max(4, std::min<int>(n, (int)((int64_t)n * columns / 256)));
}
int wgrad_blocks(int n) {
  const int zc = wgrad_planes(n);
  return (n / std::min(n, kWX)) * (n / kWY) * ((n + zc - 1) / zc);
}

}  // namespace

bool net_size_ok(int n) { return n >= 16 && (n & (n - 1)) == 0; }

void launch_conv(int n, const uint16_t* in, const float* w, const float* bias, int flags,
                 const uint16_t* mask, void* out, hipStream_t st) {
  const int rows = conv_rows(n, flags), zc = conv_planes(n, rows);
  const dim3 g(((n + 63) / 64) * (n / rows) * ((n + zc - 1) / zc));
  const double V = (double)n * n * n;
  prof_begin(st, K_CONV);
  switch (flags) {
    case 1: hipLaunchKernelGGL((k_conv<1, 8>), g, dim3(256), 0, st, n, zc, in, w, bias, mask, out); break;
    case 2: hipLaunchKernelGGL((k_conv<2, 8>), g, dim3(256), 0, st, n, zc, in, w, bias, mask, out); break;
    case 4: hipLaunchKernelGGL((k_conv<4, 8>), g, dim3(256), 0, st, n, zc, in, w, bias, mask, out); break;
    case 12:
      if (rows == 4)
        hipLaunchKernelGGL((k_conv<12, 4>), g, dim3(256), 0, st, n, zc, in, w, bias, mask, out);
      else
        hipLaunchKernelGGL((k_conv<12, 8>), g, dim3(256), 0, st, n, zc, in, w, bias, mask, out);
      break;
    default: hipLaunchKernelGGL((k_conv<0, 8>), g, dim3(256), 0, st, n, zc, in, w, bias, mask, out); break;
  }
  // matrix-core work: 27 taps x 16 x 16 MACs per voxel
  prof_end(st, K_CONV, 2.0 * 27 * kNC * kNC * V);
}

// at least what the partials take; callers may have sized their scratch by
// one partial per 64 x 4 x 8 voxels, so it does not shrink with fewer of them
size_t wgrad_scratch_bytes(int n) {
  const int x = std::min(n, kWX);
  return (size_t)(n / x) * (n / 4) * (n / 8) * kWG * sizeof(float);
}

void launch_conv_wgrad(int n, const uint16_t* in, const uint16_t* g, float* dw, float* db,
                       float* scratch, hipStream_t st) {
  const int nb = wgrad_blocks(n);
  prof_begin(st, K_CONV_WGRAD);
  hipLaunchKernelGGL(k_conv_wgrad, dim3(nb), dim3(512), 0, st, n, wgrad_planes(n), in, g, scratch);
  hipLaunchKernelGGL(k_wgrad_reduce, dim3((kWG + kWRed - 1) / kWRed), dim3(256), 0, st, scratch, nb,
                     dw, db);
  prof_end(st, K_CONV_WGRAD, 2.0 * 27 * kNC * kNC * (double)n * n * n);
}

template <typename RT, typename PT, bool SPLIT>
void launch_net_prep(int n, const RT* r, const PT* phi, float s_r, float s_phi, float kap,
                     const Box* box, uint16_t* act0, hipStream_t st) {
  const int64_t V = (int64_t)n * n * n;
  Box b{};
  if (box) b = *box;
  hipLaunchKernelGGL((k_net_prep<RT, PT, SPLIT>), dim3((unsigned)((V + 255) / 256)), dim3(256), 0,
                     st, n, r, phi, s_r, s_phi, kap, b, box ? 1 : 0, act0);
}
template void launch_net_prep<float, float, false>(int, const float*, const float*, float, float,
                                                   float, const Box*, uint16_t*, hipStream_t);
template void launch_net_prep<float, double, true>(int, const float*, const double*, float, float,
                                                   float, const Box*, uint16_t*, hipStream_t);
template void launch_net_prep<double, double, true>(int, const double*, const double*, float, float,
                                                    float, const Box*, uint16_t*, hipStream_t);

// Net forward: act0 -> 4 hidden layers (ReLU, BF16) -> FP32 channel 0 in out.
void net_forward(int n, const float* params, const uint16_t* act0, uint16_t* a, uint16_t* b,
                 float* out, hipStream_t st) {
  const int per = 27 * kNC * kNC + kNC;
  const uint16_t* src = act0;
  uint16_t* bufs[2] = {a, b};
  for (int l = 0; l < 4; ++l) {
    const float* w = params + l * per;
    launch_conv(n, src, w, w + 27 * kNC * kNC, 1, nullptr, bufs[l & 1], st);
    src = bufs[l & 1];
  }
  const float* w = params + 4 * per;
  launch_conv(n, src, w, w + 27 * kNC * kNC, 2, nullptr, out, st);
}

size_t net_train_scratch_bytes(int n) {
  const size_t V = (size_t)n * n * n;
  const size_t act = V * kNC * sizeof(uint16_t);
  const size_t np = 5 * (27 * kNC * kNC + kNC);
  return 6 * act + V * sizeof(float) + wgrad_scratch_bytes(n) + np * sizeof(float) +
         ((V + 255) / 256) * sizeof(float) + 4096;
}

// One training step on one sample: forward with stored activations, MSE loss
// against target, backward through every layer, Adam.  loss_out (device):
// mean squared error of this sample.
void net_train_step(int n, float* params, float* m1, float* m2, int step, float lr,
                    const uint16_t* act0, const float* target, float target_scale, void* scratch,
                    float* loss_out, hipStream_t st) {
  const size_t V = (size_t)n * n * n;
  const int per = 27 * kNC * kNC + kNC;
  const int np = 5 * per;
  char* s = (char*)scratch;
  uint16_t* acts[5];
  acts[0] = (uint16_t*)act0;
  for (int l = 1; l < 5; ++l) {
    acts[l] = (uint16_t*)s;
    s += V * kNC * sizeof(uint16_t);
  }
  uint16_t* ga = (uint16_t*)s;
  s += V * kNC * sizeof(uint16_t);
  uint16_t* gb = (uint16_t*)s;
  s += V * kNC * sizeof(uint16_t);
  float* out = (float*)s;
  s += V * sizeof(float);
  float* wpart = (float*)s;
  s += wgrad_scratch_bytes(n);
  float* grad = (float*)s;
  s += (size_t)np * sizeof(float);
  float* lpart = (float*)s;
  for (int l = 0; l < 4; ++l) {
    const float* w = params + l * per;
    launch_conv(n, acts[l], w, w + 27 * kNC * kNC, 1, nullptr, acts[l + 1], st);
  }
  launch_conv(n, acts[4], params + 4 * per, params + 4 * per + 27 * kNC * kNC, 2, nullptr, out, st);
  const unsigned nbl = (unsigned)((V + 255) / 256);
  hipLaunchKernelGGL(k_net_loss, dim3(nbl), dim3(256), 0, st, (int64_t)V, out, target,
                     target_scale, 1.0f / (float)V, ga, lpart);
  hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(256), 0, st, lpart, (int)nbl, 1.0f / (float)V,
                     loss_out);
  uint16_t* gcur = ga;
  uint16_t* gnext = gb;
  for (int l = 4; l >= 0; --l) {
    float* dw = grad + l * per;
    launch_conv_wgrad(n, acts[l], gcur, dw, dw + 27 * kNC * kNC, wpart, st);
    if (l > 0) {
      // gradient into layer l's input, through the ReLU of layer l-1's output
      launch_conv(n, gcur, params + l * per, nullptr, 12, acts[l], gnext, st);
      uint16_t* tmp = gcur;
      gcur = gnext;
      gnext = tmp;
    }
  }
  const float b1 = 0.9f, b2 = 0.999f;
  const float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
  hipLaunchKernelGGL(k_adam, dim3((np + 255) / 256), dim3(256), 0, st, np, params, grad, m1, m2, lr,
                     b1, b2, 1e-8f, c1, c2);
}

}  // namespace sdpm

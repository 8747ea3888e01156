// Re-sort of the active particles: a 32-bit key per particle (the Morton
// code of its block of 2^shift cells per axis, then its cell row inside the
// block: z, then y), a stable LSD radix sort of (key, index) pairs with 8-bit
// digits, and a gather of the SoA particle arrays into sorted order.  Inside
// a row the particles keep their previous order.  The
// physics of a step does not depend on particle order (the deposit is exact
// integer arithmetic, every other pass is per particle, compaction is
// stable); the sort only makes neighbouring particles touch neighbouring
// cells, which the LDS-privatised deposit and the interpolation exploit.
//
// Radix pass: (1) each workgroup histograms the digit of its keys in LDS, (2)
// a device-wide exclusive scan over the digit-major table gives every (digit,
// workgroup) its output base, (3) each workgroup scatters its keys in order.
// A wavefront has 64 KPL consecutive keys, in registers: it counts its digits,
// takes its place behind the wavefronts before it, and goes through its keys by
// rounds of 64, the rank among equal digits from 8 ballots (one per digit bit)
// and the digit's next place from a counter of its own in LDS, so the pass is
// stable and its rounds need no barrier.
// Bound by the scattered stores, one digit's keys of a workgroup being a run:
// KPL = 16 makes the runs four times as long and the table four times as small
// as KPL = 4, but leaves a small sort few workgroups.  5 M keys, a pass: 17 us
// histogram, 14 scan, 32 scatter (17, 22 and 37 with rounds of 256 keys and
// four barriers each); 2 M keys: scatter 14.5 us, KPL = 4 13.3.
#include "internal.h"

namespace sdpm {
namespace {

constexpr int kDigits = 256;
// keys from which a lane takes 16 (see above)
constexpr int64_t kSortWide = 1 << 21;

__device__ inline uint32_t spread3(uint32_t v) {
  // insert two zero bits between the low 10-11 bits of v
  v &= 0x7ff;
  v = (v | (v << 16)) & 0x070000ff;
  v = (v | (v << 8)) & 0x0700f00f;
  v = (v | (v << 4)) & 0x430c30c3;
  v = (v | (v << 2)) & 0x49249249;
  return v;
}

__global__ void __launch_bounds__(256)
k_morton_keys(const double* __restrict__ x0, const double* __restrict__ x1,
              const double* __restrict__ x2, int64_t n, double inv_h, int ng, int shift,
              uint32_t* __restrict__ key) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (q >= n) return;
  int c[3];
  const double xs[3] = {x0[q], x1[q], x2[q]};
  for (int d = 0; d < 3; ++d) {
    double v = floor(xs[d] * inv_h);
    v = v < 0.0 ? 0.0 : (v > ng - 1 ? ng - 1 : v);   // NaN -> ng - 1: order only
    c[d] = (int)v;
  }
  const uint32_t in = (uint32_t)((1 << shift) - 1);
  const uint32_t block = spread3((uint32_t)(c[0] >> shift)) | (spread3((uint32_t)(c[1] >> shift)) << 1) |
                         (spread3((uint32_t)(c[2] >> shift)) << 2);
  key[q] = (block << (2 * shift)) | (((uint32_t)c[2] & in) << shift) | ((uint32_t)c[1] & in);
}

// First sorted index of each block (Morton index m): the lower bound of its
// first key m << 2 shift in the sorted keys; start[nblk] = n.
__global__ void __launch_bounds__(256)
k_block_starts(const uint32_t* __restrict__ key, int64_t n, int shift, int64_t nblk,
               int64_t* __restrict__ start) {
  const int64_t m = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (m > nblk) return;
  if (m == nblk) {
    start[m] = n;
    return;
  }
  const uint32_t target = (uint32_t)m << (2 * shift);
  int64_t lo = 0, hi = n;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (key[mid] < target)
      lo = mid + 1;
    else
      hi = mid;
  }
  start[m] = lo;
}

template <int KPL>
__global__ void __launch_bounds__(256)
k_radix_hist(const uint32_t* __restrict__ key, int64_t n, int bit, int nblocks,
             uint32_t* __restrict__ hist) {
  __shared__ uint32_t h[kDigits];
  const int tid = threadIdx.x;
  h[tid] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * (256 * KPL);
  uint32_t k[KPL];
#pragma unroll
  for (int u = 0; u < KPL; ++u) k[u] = key[min(base + u * 256 + tid, n - 1)];
#pragma unroll
  for (int u = 0; u < KPL; ++u)
    if (base + u * 256 + tid < n) atomicAdd(&h[(k[u] >> bit) & 0xff], 1u);
  __syncthreads();
  hist[(int64_t)tid * nblocks + blockIdx.x] = h[tid];
}

// val == nullptr: key q has the value q
template <int KPL>
__global__ void __launch_bounds__(256)
k_radix_scatter(const uint32_t* __restrict__ key, const uint32_t* __restrict__ val, int64_t n,
                int bit, int nblocks, const uint32_t* __restrict__ base_tab,
                uint32_t* __restrict__ key_out, uint32_t* __restrict__ val_out) {
  __shared__ uint32_t run[4][kDigits];           // each wavefront's next place per digit
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const unsigned long long lt = (1ull << lane) - 1ull;
  const int64_t base = ((int64_t)blockIdx.x * 4 + wave) * (64 * KPL) + lane;
  uint32_t k[KPL], v[KPL];
#pragma unroll
  for (int u = 0; u < KPL; ++u) {
    const int64_t q = min(base + u * 64, n - 1);
    k[u] = key[q];
    v[u] = val ? val[q] : (uint32_t)q;
  }
  uint32_t start = base_tab[(int64_t)tid * nblocks + blockIdx.x];
#pragma unroll
  for (int w = 0; w < 4; ++w) run[w][tid] = 0;
  __syncthreads();
#pragma unroll
  for (int u = 0; u < KPL; ++u)
    if (base + u * 64 < n) atomicAdd(&run[wave][(k[u] >> bit) & 0xff], 1u);
  __syncthreads();
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const uint32_t c = run[w][tid];
    run[w][tid] = start;
    start += c;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < KPL; ++u) {
    const bool valid = base + u * 64 < n;
    const uint32_t d = (k[u] >> bit) & 0xff;
    // lanes of this wave holding the same digit
    unsigned long long same = __ballot(valid);
    for (int b = 0; b < 8; ++b) {
      const unsigned long long m = __ballot((d >> b) & 1u);
      same &= ((d >> b) & 1u) ? m : ~m;
    }
    const uint32_t rank = (uint32_t)__popcll(same & lt);
    // the first of them moves the counter on for all
    uint32_t at = 0;
    if (valid && rank == 0) at = atomicAdd(&run[wave][d], (uint32_t)__popcll(same));
    at = __shfl(at, valid ? __ffsll((unsigned long long)same) - 1 : lane);
    if (valid) {
      key_out[at + rank] = k[u];
      val_out[at + rank] = v[u];
    }
  }
}

// device-wide exclusive scan of uint32 (three kernels)
constexpr int kScanSeg = 4096;

// a thread has kScanPer consecutive values, a workgroup 256 threads' worth
constexpr int kScanPer = kScanSeg / 256;

__device__ inline void scan_load(const uint32_t* a, int64_t n, int64_t q, uint32_t (&v)[kScanPer]) {
  if (q + kScanPer <= n) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4), aligned(4)));
#pragma unroll
    for (int u = 0; u < kScanPer; u += 4) {
      const u32x4 x = *(const u32x4*)(a + q + u);
      v[u] = x[0], v[u + 1] = x[1], v[u + 2] = x[2], v[u + 3] = x[3];
    }
  } else {
#pragma unroll
    for (int u = 0; u < kScanPer; ++u) v[u] = q + u < n ? a[q + u] : 0u;
  }
}

__global__ void __launch_bounds__(256)
k_scan_seg_sum(const uint32_t* __restrict__ a, int64_t n, uint32_t* __restrict__ part) {
  __shared__ uint32_t sh[4];
  const int tid = threadIdx.x;
  uint32_t v[kScanPer];
  scan_load(a, n, (int64_t)blockIdx.x * kScanSeg + tid * kScanPer, v);
  uint32_t s = 0;
#pragma unroll
  for (int u = 0; u < kScanPer; ++u) s += v[u];
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  if ((tid & 63) == 0) sh[tid >> 6] = s;
  __syncthreads();
  if (tid == 0) part[blockIdx.x] = sh[0] + sh[1] + sh[2] + sh[3];
}

__global__ void __launch_bounds__(1024) k_scan_parts(uint32_t* __restrict__ part, int64_t np) {
  __shared__ uint32_t sh[1024];
  const int tid = threadIdx.x;
  const int64_t per = (np + 1023) / 1024;
  const int64_t b0 = tid * per, b1 = min(np, b0 + per);
  uint32_t s = 0;
  for (int64_t b = b0; b < b1; ++b) s += part[b];
  sh[tid] = s;
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {
    const uint32_t v = tid >= off ? sh[tid - off] : 0u;
    __syncthreads();
    sh[tid] += v;
    __syncthreads();
  }
  uint32_t run = tid ? sh[tid - 1] : 0u;
  for (int64_t b = b0; b < b1; ++b) {
    const uint32_t v = part[b];
    part[b] = run;
    run += v;
  }
}

__global__ void __launch_bounds__(256)
k_scan_apply(uint32_t* __restrict__ a, int64_t n, const uint32_t* __restrict__ part) {
  __shared__ uint32_t wtot[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t q = (int64_t)blockIdx.x * kScanSeg + tid * kScanPer;
  uint32_t v[kScanPer], own = 0;
  scan_load(a, n, q, v);
#pragma unroll
  for (int u = 0; u < kScanPer; ++u) own += v[u];
  // inclusive wave scan of the threads' sums
  uint32_t x = own;
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t y = __shfl_up(x, off, 64);
    if (lane >= off) x += y;
  }
  if (lane == 63) wtot[wave] = x;
  __syncthreads();
  uint32_t run = part[blockIdx.x] + x - own;
  for (int w = 0; w < wave; ++w) run += wtot[w];
#pragma unroll
  for (int u = 0; u < kScanPer; ++u) {
    if (q + u < n) a[q + u] = run;
    run += v[u];
  }
}

template <typename PT>
__global__ void __launch_bounds__(256)
k_gather(ParticleArgs pa, const uint32_t* __restrict__ perm, double* __restrict__ sx0,
         double* __restrict__ sx1, double* __restrict__ sx2, PT* __restrict__ sp0,
         PT* __restrict__ sp1, PT* __restrict__ sp2, uint32_t* __restrict__ sid) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (q >= pa.n) return;
  const uint32_t s = perm[q];
  sx0[q] = pa.x[0][s];
  sx1[q] = pa.x[1][s];
  sx2[q] = pa.x[2][s];
  sp0[q] = ((const PT*)pa.p[0])[s];
  sp1[q] = ((const PT*)pa.p[1])[s];
  sp2[q] = ((const PT*)pa.p[2])[s];
  sid[q] = pa.id[s];
}

// A particle set in scratch back into its arrays, all seven in one launch (5 M
// particles: 71 us, the rate of a copy; seven copies by the runtime leave a gap
// after each).
template <typename PT>
__global__ void __launch_bounds__(256)
k_put_back(ParticleArgs pa, const double* __restrict__ sx, const PT* __restrict__ sp,
           const uint32_t* __restrict__ sid) {
  const int64_t base = (int64_t)blockIdx.x * 1024 + threadIdx.x;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int64_t q = base + 256 * u;
    if (q >= pa.n) return;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      pa.x[d][q] = __builtin_nontemporal_load(sx + d * pa.n + q);
      ((PT*)pa.p[d])[q] = __builtin_nontemporal_load(sp + d * pa.n + q);
    }
    pa.id[q] = __builtin_nontemporal_load(sid + q);
  }
}

void device_scan(uint32_t* a, int64_t n, uint32_t* part, hipStream_t st) {
  const int64_t np = (n + kScanSeg - 1) / kScanSeg;
  hipLaunchKernelGGL(k_scan_seg_sum, dim3((unsigned)np), dim3(256), 0, st, a, n, part);
  hipLaunchKernelGGL(k_scan_parts, dim3(1), dim3(1024), 0, st, part, np);
  hipLaunchKernelGGL(k_scan_apply, dim3((unsigned)np), dim3(256), 0, st, a, n, part);
}

// Sorts keys k0 with the values 0 .. n - 1 by key bits [from, to), to > from;
// the result is in k0, v0 (swapped on the way).
template <int KPL>
void radix_passes(uint32_t*& k0, uint32_t*& v0, uint32_t*& k1, uint32_t*& v1, int64_t n, int from,
                  int to, uint32_t* hist, uint32_t* part, hipStream_t st) {
  const int64_t nb = (n + 256 * KPL - 1) / (256 * KPL);
  for (int bit = from; bit < to; bit += 8) {
    hipLaunchKernelGGL(k_radix_hist<KPL>, dim3((unsigned)nb), dim3(256), 0, st, k0, n, bit, (int)nb,
                       hist);
    device_scan(hist, nb * kDigits, part, st);
    hipLaunchKernelGGL(k_radix_scatter<KPL>, dim3((unsigned)nb), dim3(256), 0, st, k0,
                       bit == from ? nullptr : v0, n, bit, (int)nb, hist, k1, v1);
    std::swap(k0, k1);
    std::swap(v0, v1);
  }
}

void radix_sort(uint32_t*& k0, uint32_t*& v0, uint32_t*& k1, uint32_t*& v1, int64_t n, int from, int to,
                uint32_t* hist, uint32_t* part, hipStream_t st) {
  if (n >= kSortWide)
    radix_passes<16>(k0, v0, k1, v1, n, from, to, hist, part, st);
  else
    radix_passes<4>(k0, v0, k1, v1, n, from, to, hist, part, st);
}

__global__ void __launch_bounds__(256)
k_far_pairs(ParticleArgs pa, double inv_h, int ng, uint32_t* __restrict__ count) {
  const int64_t q = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 64;
  bool far = false;
  if (q + 1 < pa.n)
    for (int d = 0; d < 3; ++d) {
      const double a = fabs(pa.x[d][q + 1] - pa.x[d][q]) * inv_h;
      far = far || fmin(a, ng - a) > kBlkCells;
    }
  const uint32_t c = (uint32_t)__popcll(__ballot(far));
  if ((threadIdx.x & 63) == 0 && c) atomicAdd(count, c);
}

}  // namespace

template <typename PT>
void launch_put_back(const ParticleArgs& pa, const void* scratch, hipStream_t st) {
  const double* sx = (const double*)scratch;
  const PT* sp = (const PT*)(sx + 3 * pa.n);
  hipLaunchKernelGGL(k_put_back<PT>, dim3((unsigned)((pa.n + 1023) / 1024)), dim3(256), 0, st, pa, sx,
                     sp, (const uint32_t*)(sp + 3 * pa.n));
}
template void launch_put_back<float>(const ParticleArgs&, const void*, hipStream_t);
template void launch_put_back<double>(const ParticleArgs&, const void*, hipStream_t);

void launch_far_pairs(const ParticleArgs& pa, int ng, double box, uint32_t* count, hipStream_t st) {
  const int64_t pairs = (pa.n + 63) / 64;
  hipLaunchKernelGGL(k_far_pairs, dim3((unsigned)((pairs + 255) / 256)), dim3(256), 0, st, pa,
                     (double)ng / box, ng, count);
}

size_t block_order_bytes(int64_t n, int ng) {
  const int64_t nb1 = ng >> kBlkShift;
  return sort_scratch_bytes(n) + (size_t)(nb1 * nb1 * nb1 + 1) * sizeof(int64_t);
}

void launch_block_order(const ParticleArgs& pa, int ng, double box, void* scratch,
                        const uint32_t** perm, const int64_t** block_start, hipStream_t st) {
  const int64_t n = pa.n, nb = (n + kChunk - 1) / kChunk, nb1 = ng >> kBlkShift, nblk = nb1 * nb1 * nb1;
  int64_t* start = (int64_t*)scratch;
  uint32_t* k0 = (uint32_t*)(start + nblk + 1);
  uint32_t *v0 = k0 + n, *k1 = v0 + n, *v1 = k1 + n, *hist = v1 + n, *part = hist + nb * kDigits;
  int lg = 0;
  while ((1 << lg) < nb1) ++lg;
  prof_begin(st, K_SORT);
  hipLaunchKernelGGL(k_morton_keys, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, pa.x[0],
                     pa.x[1], pa.x[2], n, (double)ng / box, ng, kBlkShift, k0);
  // the blocks alone: the order inside one is free
  radix_sort(k0, v0, k1, v1, n, 2 * kBlkShift, 2 * kBlkShift + 3 * lg, hist, part, st);
  hipLaunchKernelGGL(k_block_starts, dim3((unsigned)((nblk + 256) / 256)), dim3(256), 0, st, k0, n,
                     kBlkShift, nblk, start);
  const int passes = (3 * lg + 7) / 8;
  prof_end(st, K_SORT, (double)n * (24.0 + 8.0 + passes * (4.0 + 16.0)));
  *perm = v0;
  *block_start = start;
}

size_t sort_scratch_bytes(int64_t capacity) {
  const int64_t nb = (capacity + kChunk - 1) / kChunk + 1;
  const int64_t tab = nb * kDigits;
  const int64_t np = (tab + kScanSeg - 1) / kScanSeg + 1;
  return (size_t)(4 * capacity + tab + np) * sizeof(uint32_t) + 4 * 256;
}

template <typename PT>
void launch_morton_sort(const ParticleArgs& pa, int ng, double box, int shift, void* sort_scratch,
                        void* particle_scratch, int64_t* block_start, hipStream_t st) {
  const int64_t n = pa.n;
  if (n <= 1) return;
  const int64_t nb = (n + kChunk - 1) / kChunk;
  const int64_t tab = nb * kDigits;
  uint32_t* k0 = (uint32_t*)sort_scratch;
  uint32_t* v0 = k0 + n;
  uint32_t* k1 = v0 + n;
  uint32_t* v1 = k1 + n;
  uint32_t* hist = v1 + n;
  uint32_t* part = hist + tab;
  int lg = 0;
  while ((1 << lg) < ng) ++lg;
  const int bits = 3 * (lg - shift) + 2 * shift;
  const unsigned gp = (unsigned)((n + 255) / 256);
  prof_begin(st, K_SORT);
  hipLaunchKernelGGL(k_morton_keys, dim3(gp), dim3(256), 0, st, pa.x[0], pa.x[1], pa.x[2], n,
                     (double)ng / box, ng, shift, k0);
  radix_sort(k0, v0, k1, v1, n, 0, bits, hist, part, st);
  if (block_start) {
    const int64_t nb1 = ng >> shift, nblk = nb1 * nb1 * nb1;
    hipLaunchKernelGGL(k_block_starts, dim3((unsigned)((nblk + 256) / 256)), dim3(256), 0, st, k0, n,
                       shift, nblk, block_start);
  }
  const int passes = (bits + 7) / 8;
  prof_end(st, K_SORT, (double)n * (8.0 + passes * (4.0 + 16.0)));
  char* s = (char*)particle_scratch;
  double* sx0 = (double*)s;
  double* sx1 = sx0 + n;
  double* sx2 = sx1 + n;
  PT* sp0 = (PT*)(sx2 + n);
  PT* sp1 = sp0 + n;
  PT* sp2 = sp1 + n;
  uint32_t* sid = (uint32_t*)(sp2 + n);
  const double pbytes = (24.0 + 3.0 * sizeof(PT) + 4.0) * n;
  prof_begin(st, K_GATHER);
  hipLaunchKernelGGL(k_gather<PT>, dim3(gp), dim3(256), 0, st, pa, v0, sx0, sx1, sx2, sp0, sp1, sp2,
                     sid);
  prof_end(st, K_GATHER, 2.0 * pbytes + 4.0 * n);
  prof_begin(st, K_COPY);
  launch_put_back<PT>(pa, particle_scratch, st);
  prof_end(st, K_COPY, 2.0 * pbytes);
}
template void launch_morton_sort<float>(const ParticleArgs&, int, double, int, void*, void*,
                                        int64_t*, hipStream_t);
template void launch_morton_sort<double>(const ParticleArgs&, int, double, int, void*, void*,
                                         int64_t*, hipStream_t);

}  // namespace sdpm

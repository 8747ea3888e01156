// Power spectrum of particle positions in a periodic box: the accuracy metric
// the paper compares runs with (Sec. 3.1, Sec. 3.2: 3D spectra of the
// lightcone in a cubical box of the original size), with the discreteness
// corrections of Jing (2005) that the paper names for its spectrum tool
// (Sec. 2.4).
//
// delta = C / (nbar 2^(3B)) - 1 from the fixed-point CIC deposit (the step's
// own deposit kernel, no drift), one FP64 real-to-complex FFT, then shell
// sums over the half spectrum: a column 0 < i < n/2 stands for itself and
// its conjugate mode, the columns i = 0 and i = n/2 for themselves.  Shell
// b = rint(|f|) in 1 .. n/2, f the signed integer frequency (index n/2 is
// -n/2).  Per shell: mean |k|, modes, mean L^3 |delta_k|^2, mean of the CIC
// shot-noise alias factor C1(f) = prod_d (1 - 2/3 sin^2(pi f_d / n)); Jing's
// correction divides the shot-subtracted mean by the shell mean of
//   S(f) = sum_{m in [-2,2]^3} W^2(f + n m) (|f + n m| / |f|)^neff,
// W^2(g) = prod_d sinc^4(pi g_d / n), the local slope neff re-estimated
// three times from the corrected spectrum (central log-log differences of
// neighbouring shells, one-sided at the ends, clamped to [-4, 4], 0 where a
// neighbour is not positive).  S is even in each frequency and symmetric in
// the three (the images lie symmetrically), so its shell sums run over the
// sorted triples |f_x| >= |f_y| >= |f_z| with the number of modes each stands
// for: up to 48 times fewer evaluations than one per mode (256^3: 0.20 against
// 2.58 ms per pass; FP64 exponentials and logarithms bound it).  Shell sums
// are accumulated per workgroup in LDS and reduced over a fixed number of
// workgroups in a fixed order (7 us; a serial chain over the workgroups per
// entry took 216 us).
#include <algorithm>
#include <cmath>
#include <vector>

#include "internal.h"

namespace sdpm {
namespace {

constexpr int kPkBlocks = 1024;     // workgroups of the raw shell pass
constexpr int kPkAliasBlocks = 2048; // of the alias pass: about a pair per wave at 256^3
constexpr int kPkImages = 2;        // images per axis side in S
constexpr int kPkTab = 2 * kPkImages + 1;
constexpr int kPkIter = 3;
constexpr int kPkSums = 4;          // P_raw, C1, |f|, weight (S pass: S)

__device__ inline int freq(int idx, int n) { return idx < n / 2 ? idx : idx - n; }

__global__ void __launch_bounds__(256)
k_pk_delta(double* __restrict__ mesh, int64_t cells, double inv) {
  // counts (u64) -> delta (double) in place
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < cells;
       q += (int64_t)gridDim.x * blockDim.x) {
    const uint64_t c = ((const uint64_t*)mesh)[q];
    mesh[q] = (double)c * inv - 1.0;
  }
}

// tab[(f + n/2) * kPkTab + m + kPkImages] = sinc^4(pi (f + n m) / n),
// sq[(f + n/2) * kPkTab + ...] = (f + n m)^2
__global__ void __launch_bounds__(256)
k_pk_tables(double* __restrict__ tab, double* __restrict__ sq, int n) {
  const int q = blockIdx.x * 256 + threadIdx.x;
  if (q >= (n + 1) * kPkTab) return;
  const double g = (double)(q / kPkTab - n / 2) + (double)n * (q % kPkTab - kPkImages);
  const double xg = M_PI * g / n;
  const double sc = g == 0.0 ? 1.0 : sin(xg) / xg;
  tab[q] = sc * sc * sc * sc;
  sq[q] = g * g;
}

// per shell sums of w P_raw, w C1, w |f|, w over the half spectrum (rows of
// `pitch` values)
__global__ void __launch_bounds__(256)
k_pk_shells(const double2* __restrict__ c, int n, int pitch, double l3, double* __restrict__ partial) {
  extern __shared__ double acc[];
  const int nb = n / 2;
  for (int q = threadIdx.x; q < nb * kPkSums; q += blockDim.x) acc[q] = 0.0;
  __syncthreads();
  const int hx = n / 2 + 1;
  const int64_t total = (int64_t)n * n * hx;
  const double inv_n3 = 1.0 / ((double)n * n * n);
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < total;
       q += (int64_t)gridDim.x * blockDim.x) {
    const int i = (int)(q % hx);
    const int64_t r = q / hx;
    const int j = (int)(r % n), k = (int)(r / n);
    const int fx = i == n / 2 ? -n / 2 : i, fy = freq(j, n), fz = freq(k, n);
    const double fa = sqrt((double)fx * fx + (double)fy * fy + (double)fz * fz);
    const int shell = (int)rint(fa);
    if (shell < 1 || shell > nb) continue;
    const bool pair = i > 0 && i < n / 2;
    const double w = pair ? 2.0 : 1.0;
    const int sb = shell - 1;
    const double2 v = c[r * pitch + i];
    const double re = v.x * inv_n3, im = v.y * inv_n3;
    double c1 = 1.0;
    const int fs[3] = {fx, fy, fz};
    for (int d = 0; d < 3; ++d) {
      const double s = sin(M_PI * fs[d] / n);
      c1 *= 1.0 - (2.0 / 3.0) * s * s;
    }
    atomicAdd(&acc[sb * kPkSums + 0], w * l3 * (re * re + im * im));
    atomicAdd(&acc[sb * kPkSums + 1], w * c1);
    atomicAdd(&acc[sb * kPkSums + 2], w * fa);
    atomicAdd(&acc[sb * kPkSums + 3], w);
  }
  __syncthreads();
  for (int q = threadIdx.x; q < nb * kPkSums; q += blockDim.x)
    partial[(int64_t)blockIdx.x * nb * kPkSums + q] = acc[q];
}

// Modes of the spectrum with |frequency| v along one axis (n/2 occurs only
// as -n/2).
__device__ inline int axis_modes(int v, int n) { return v == 0 || v == n / 2 ? 1 : 2; }

// Per shell sums of S(f; neff[shell]) over the modes: a wave takes a pair
// a >= b of frequencies, its lanes the third, c <= b.
__global__ void __launch_bounds__(256)
k_pk_alias(int n, const double* __restrict__ neff, const double* __restrict__ tab,
           const double* __restrict__ sq, double* __restrict__ partial) {
  extern __shared__ double acc[];
  const int nb = n / 2;
  for (int q = threadIdx.x; q < nb; q += blockDim.x) acc[q] = 0.0;
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int pairs = (nb + 1) * (nb + 2) / 2, waves = gridDim.x * 4;
  for (int q = blockIdx.x * 4 + (threadIdx.x >> 6); q < pairs; q += waves) {
    int a = (int)((sqrt(8.0 * q + 1.0) - 1.0) * 0.5);
    while (a * (a + 1) / 2 > q) --a;
    while ((a + 1) * (a + 2) / 2 <= q) ++a;
    const int b = q - a * (a + 1) / 2;
    const int oa = (a + nb) * kPkTab, ob = (b + nb) * kPkTab;
    for (int c = lane; c <= b; c += 64) {
      const double f2 = (double)a * a + (double)b * b + (double)c * c;
      const int shell = (int)rint(sqrt(f2));
      if (shell < 1 || shell > nb) continue;
      const int perms = a == b && b == c ? 1 : (a == b || b == c ? 3 : 6);
      const double modes = perms * axis_modes(a, n) * axis_modes(b, n) * axis_modes(c, n);
      const double half = 0.5 * neff[shell - 1];
      double wc[kPkTab], gc[kPkTab];
#pragma unroll
      for (int u = 0; u < kPkTab; ++u) {
        wc[u] = tab[(c + nb) * kPkTab + u];
        gc[u] = sq[(c + nb) * kPkTab + u];
      }
      double s = 0.0;
      for (int u = 0; u < kPkTab; ++u)
        for (int v = 0; v < kPkTab; ++v) {
          const double wab = tab[oa + u] * tab[ob + v], gab = sq[oa + u] + sq[ob + v];
#pragma unroll
          for (int t = 0; t < kPkTab; ++t) {
            const double w = wab * wc[t];
            s += half == 0.0 ? w : w * exp(half * log((gab + gc[t]) / f2));
          }
        }
      atomicAdd(&acc[shell - 1], modes * s);
    }
  }
  __syncthreads();
  for (int q = threadIdx.x; q < nb; q += blockDim.x) partial[(int64_t)blockIdx.x * nb + q] = acc[q];
}

// out[q] = sum over workgroups of partial[b][q] in a fixed order: 8 entries
// per workgroup, 32 threads each
__global__ void __launch_bounds__(256)
k_pk_reduce(const double* __restrict__ partial, int nblocks, int width, double* __restrict__ out) {
  __shared__ double sh[256];
  const int e = threadIdx.x & 7, t = threadIdx.x >> 3, q = blockIdx.x * 8 + e;
  double s = 0.0;
  if (q < width) {
#pragma unroll 8
    for (int b = t; b < nblocks; b += 32) s += partial[(int64_t)b * width + q];
  }
  sh[threadIdx.x] = s;
  for (int off = 16; off > 0; off >>= 1) {
    __syncthreads();
    if (t < off) sh[threadIdx.x] += sh[threadIdx.x + 8 * off];
  }
  if (t == 0 && q < width) out[q] = sh[e];
}

struct PkLayout {
  size_t mesh, fft, sym, tab, sq, partial, sums, neff, flags, total;
};

PkLayout pk_layout(int n) {
  PkLayout l{};
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t at = off;
    off = (off + bytes + 255) & ~(size_t)255;
    return at;
  };
  const int nb = n / 2;
  l.mesh = take((size_t)n * n * n * sizeof(double));
  l.fft = take(2 * fft_complex_bytes(n));
  l.tab = take((size_t)(n + 1) * kPkTab * sizeof(double));
  l.sq = take((size_t)(n + 1) * kPkTab * sizeof(double));
  l.partial = take((size_t)kPkBlocks * nb * kPkSums * sizeof(double));
  l.sums = take((size_t)nb * kPkSums * sizeof(double));
  l.neff = take((size_t)nb * sizeof(double));
  l.flags = take(16 * sizeof(uint32_t));
  l.sym = l.partial;                           // of use to the solve only: overwritten here
  l.total = off;
  return l;
}

void slopes(const std::vector<double>& k, const std::vector<double>& p, std::vector<double>* out) {
  const int nb = (int)k.size();
  for (int b = 0; b < nb; ++b) {
    const int lo = std::max(b - 1, 0), hi = std::min(b + 1, nb - 1);
    double v = 0.0;
    if (hi != lo && p[lo] > 0.0 && p[hi] > 0.0 && k[lo] > 0.0)
      v = std::min(std::max(std::log(p[hi] / p[lo]) / std::log(k[hi] / k[lo]), -4.0), 4.0);
    (*out)[b] = v;
  }
}

constexpr int kOrderMesh = 128;
constexpr int64_t kOrderMin = 1 << 19;
// particles whose order fits a buffer
int64_t order_fit(size_t bytes, int n) {
  int64_t fit = (int64_t)(bytes / 17);
  while (fit > 0 && block_order_bytes(fit, n) > bytes) fit -= fit / 64 + 1;
  return fit;
}

}  // namespace

size_t pk_workspace_bytes(int n) { return pk_layout(n).total; }

int power_spectrum(const double* const x[3], int64_t npart, double box, int n, int flags,
                   void* ws, hipStream_t st, double* k_out, double* p_out, double* praw_out,
                   int64_t* modes_out, char* msg, size_t len) {
  const PkLayout lay = pk_layout(n);
  char* base = (char*)ws;
  double* mesh = (double*)(base + lay.mesh);
  double* tab = (double*)(base + lay.tab);
  double* sq = (double*)(base + lay.sq);
  double* partial = (double*)(base + lay.partial);
  double* sums = (double*)(base + lay.sums);
  double* neff_dev = (double*)(base + lay.neff);
  uint32_t* dflags = (uint32_t*)(base + lay.flags);
  const int nb = n / 2;
  const int frac_bits = 14;
  auto herr = [&](const char* what) {
    snprintf(msg, len, "%s", what);
    return SDPM_EHIP;
  };
  // CIC counts of the positions (periodic box, no drift)
  if (hipMemsetAsync(dflags, 0, 16 * sizeof(uint32_t), st) != hipSuccess) return herr("memset");
  Box full;
  for (int d = 0; d < 3; ++d) full.lo[d] = 0, full.hi[d] = n - 1;
  launch_fill<uint64_t>((uint64_t*)mesh, n, full, 0ull, st);
  ParticleArgs pa{};
  for (int d = 0; d < 3; ++d) pa.x[d] = const_cast<double*>(x[d]), pa.p[d] = nullptr;
  pa.id = nullptr;
  pa.n = npart;
  MeshMap mm{};
  mm.ng = n;
  mm.frac_bits = frac_bits;
  mm.periodic = 1;
  mm.box = box;
  mm.scale = (double)n * std::ldexp(1.0, frac_bits) / box;
  mm.active = full;
  // The deposit sums in LDS what lies close together; particles in no spatial
  // order would go to memory one by one (22 G atomic adds a second).  They go
  // through the order of their blocks, as many at a time as the transform's
  // buffer, unused until then, holds, when more than a quarter of the sampled
  // neighbours in memory are a block apart.  Whole call, unordered blobs: 4 M
  // on 256^3 2.82 -> 1.87 ms, 10 M on 128^3 (six parts) 4.73 -> 1.83, 1 M on
  // 128^3 1.15 -> 0.87; below kOrderMin it gains nothing (0.4 M: 0.75 ms either
  // way), and below 128^3 the parts get too small for it.  Particles in order
  // pay for the sample and the wait for it, 25 us.
  const int64_t fit = order_fit(2 * fft_complex_bytes(n), n);
  bool ordered = false;
  if (n >= kOrderMesh && std::min(npart, fit) >= kOrderMin) {
    launch_far_pairs(pa, n, box, dflags + 1, st);
    uint32_t far = 0;
    if (hipMemcpyAsync(&far, dflags + 1, sizeof(uint32_t), hipMemcpyDeviceToHost, st) != hipSuccess ||
        hipStreamSynchronize(st) != hipSuccess)
      return herr("order of the particles");
    ordered = (int64_t)far * 64 * 4 > npart;
  }
  if (ordered) {
    for (int64_t at = 0; at < npart; at += fit) {
      ParticleArgs part = pa;
      for (int d = 0; d < 3; ++d) part.x[d] += at;
      part.n = std::min(fit, npart - at);
      const uint32_t* perm;
      const int64_t* start;
      launch_block_order(part, n, box, base + lay.fft, &perm, &start, st);
      launch_order_deposit(part, mm, start, perm, (uint64_t*)mesh, dflags, st);
    }
  } else {
    launch_drift_deposit<double>(pa, 0.0, 0, mm, (uint64_t*)mesh, dflags, st);
  }
  const int64_t cells = (int64_t)n * n * n;
  const double nbar = (double)npart / (double)cells;
  hipLaunchKernelGGL(k_pk_delta, dim3(4096), dim3(256), 0, st, mesh, cells,
                     1.0 / (nbar * std::ldexp(1.0, 3 * frac_bits)));
  FftPlan plan;
  if (fft_init(&plan, n, base + lay.fft, (double*)(base + lay.sym), st) != SDPM_OK ||
      fft_forward(plan, mesh, st) != SDPM_OK)
    return herr("transform failed");
  hipLaunchKernelGGL(k_pk_tables, dim3(((n + 1) * kPkTab + 255) / 256), dim3(256), 0, st, tab, sq, n);
  // shell sums of the raw spectrum
  const double l3 = box * box * box;
  std::vector<double> raw((size_t)nb * kPkSums);
  prof_begin(st, K_PK);
  hipLaunchKernelGGL(k_pk_shells, dim3(kPkBlocks), dim3(256), (size_t)nb * kPkSums * sizeof(double),
                     st, (const double2*)plan.c, n, plan.pitch, l3, partial);
  prof_end(st, K_PK, 16.0 * (double)n * n * (n / 2 + 1));
  hipLaunchKernelGGL(k_pk_reduce, dim3((nb * kPkSums + 7) / 8), dim3(256), 0, st, partial, kPkBlocks,
                     nb * kPkSums, sums);
  uint32_t hflags = 0;
  if (hipMemcpyAsync(&hflags, dflags, sizeof(uint32_t), hipMemcpyDeviceToHost, st) != hipSuccess ||
      hipMemcpyAsync(raw.data(), sums, raw.size() * sizeof(double), hipMemcpyDeviceToHost, st) !=
          hipSuccess ||
      hipStreamSynchronize(st) != hipSuccess)
    return herr("shell sums failed");
  if (hflags) {
    snprintf(msg, len, "a position lies outside [0, box] or is not finite");
    return SDPM_EDOMAIN;
  }
  const double kf = 2.0 * M_PI / box;
  std::vector<double> kmean(nb), praw(nb), c1(nb), signal(nb), p(nb), neff(nb, 0.0), ssum(nb);
  const double shot = (flags & SDPM_PK_SHOT) ? l3 / (double)npart : 0.0;
  for (int b = 0; b < nb; ++b) {
    const double wsum = raw[b * kPkSums + 3];
    modes_out[b] = (int64_t)llround(wsum);
    const double inv = wsum > 0.0 ? 1.0 / wsum : 0.0;
    praw[b] = raw[b * kPkSums + 0] * inv;
    c1[b] = raw[b * kPkSums + 1] * inv;
    kmean[b] = raw[b * kPkSums + 2] * inv * kf;
    signal[b] = praw[b] - shot * c1[b];
    p[b] = signal[b];
  }
  if (flags & SDPM_PK_JING) {
    for (int it = 0; it <= kPkIter; ++it) {
      if (hipMemcpyAsync(neff_dev, neff.data(), nb * sizeof(double), hipMemcpyHostToDevice, st) !=
          hipSuccess)
        return herr("copy of the slopes failed");
      prof_begin(st, K_PK);
      hipLaunchKernelGGL(k_pk_alias, dim3(kPkAliasBlocks), dim3(256), (size_t)nb * sizeof(double), st,
                         n, neff_dev, tab, sq, partial);
      prof_end(st, K_PK, 0.0);
      hipLaunchKernelGGL(k_pk_reduce, dim3((nb + 7) / 8), dim3(256), 0, st, partial, kPkAliasBlocks, nb,
                         sums);
      if (hipMemcpyAsync(ssum.data(), sums, nb * sizeof(double), hipMemcpyDeviceToHost, st) !=
              hipSuccess ||
          hipStreamSynchronize(st) != hipSuccess)
        return herr("alias sums failed");
      for (int b = 0; b < nb; ++b) {
        const double wsum = raw[b * kPkSums + 3];
        p[b] = ssum[b] > 0.0 ? signal[b] / (ssum[b] / wsum) : 0.0;
      }
      if (it < kPkIter) slopes(kmean, p, &neff);
    }
  }
  for (int b = 0; b < nb; ++b) {
    k_out[b] = kmean[b];
    p_out[b] = p[b];
    if (praw_out) praw_out[b] = praw[b];
  }
  return SDPM_OK;
}

}  // namespace sdpm

// Exact periodic solve of the mesh equation (Lap_h - kappa h^2) phi = rhs by
// FFT: the standard particle-mesh Poisson solver the paper compares against
// (Sec. 2.4), here also for kappa > 0 (the implicit half sub-step of
// Sec. 2.1 Eq. 4), and the forward transform of the power spectrum.  The
// 7-point operator is diagonal in Fourier space with symbol -(s(kx) + s(ky) +
// s(kz)) - kappa h^2, s(k) = 2 - 2 cos(2 pi k / n); the k = 0 mode of the
// singular periodic Poisson problem (kappa = 0) is set to zero (zero-mean
// potential).
//
// FP64 transforms of power-of-two length in LDS, one pass over memory per
// axis.  A line of N points is held by N / 8 threads, 8 points each (b + m N /
// 8, m = 0 .. 7): radix-8 stages (the last one radix 8, 4 or 2) in Stockham
// order, each stage's results exchanged through LDS, so that the first stage
// reads global memory and the last one writes it in natural order from
// registers.  The x pass takes N real values as N / 2 complex ones and
// separates the spectrum's halves (Cooley, Lewis & Welch 1970); the y and z
// passes take C neighbouring x columns at once, so that a row of a tile is at
// least 128 bytes.  The solve's z pass transforms, divides by the symbol (and
// n^3) and transforms back without leaving the workgroup: five passes of 16
// bytes per cell where separate forward, divide and inverse passes are seven.
// Rows of the half spectrum are padded to a multiple of 128 bytes.
// Bound by HBM: at 256^3 a pass takes 43-51 us (5.3-6.2 TB/s of its 16 bytes
// per cell), the solve 232 us; seven passes of library transforms and a
// separate division took 463 us, and each power spectrum about 8 ms of host
// time for its plan.
#include <algorithm>
#include <cmath>
#include <tuple>

#include "internal.h"

namespace sdpm {
namespace {

struct alignas(16) c64 {
  double x, y;
};
__device__ inline c64 operator+(c64 a, c64 b) { return {a.x + b.x, a.y + b.y}; }
__device__ inline c64 operator-(c64 a, c64 b) { return {a.x - b.x, a.y - b.y}; }
__device__ inline c64 operator*(c64 a, c64 b) { return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x}; }
__device__ inline c64 conj(c64 a) { return {a.x, -a.y}; }
// -i a forward, +i a inverse
template <bool INV>
__device__ inline c64 quarter(c64 a) {
  return INV ? c64{-a.y, a.x} : c64{a.y, -a.x};
}

template <bool INV>
__device__ inline void fft4(c64& a, c64& b, c64& c, c64& d) {
  const c64 s = a + c, t = a - c, u = b + d, v = quarter<INV>(b - d);
  a = s + u;
  b = t + v;
  c = s - u;
  d = t - v;
}
// in natural order, out natural
template <bool INV>
__device__ inline void fft8(c64 (&v)[8]) {
  fft4<INV>(v[0], v[2], v[4], v[6]);
  fft4<INV>(v[1], v[3], v[5], v[7]);
  constexpr double h = 0.70710678118654752440;
  // odd half times the eighth roots of unity
  const c64 o1 = INV ? c64{h * (v[3].x - v[3].y), h * (v[3].x + v[3].y)}
                     : c64{h * (v[3].x + v[3].y), h * (v[3].y - v[3].x)};
  const c64 o2 = quarter<INV>(v[5]);
  const c64 o3 = INV ? c64{-h * (v[7].x + v[7].y), h * (v[7].x - v[7].y)}
                     : c64{h * (v[7].y - v[7].x), -h * (v[7].x + v[7].y)};
  const c64 e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6], o0 = v[1];
  v[0] = e0 + o0;
  v[4] = e0 - o0;
  v[1] = e1 + o1;
  v[5] = e1 - o1;
  v[2] = e2 + o2;
  v[6] = e2 - o2;
  v[3] = e3 + o3;
  v[7] = e3 - o3;
}

// exp(-2 pi i k / N) (conjugated for the inverse) from the table of step S
template <bool INV>
__device__ inline c64 root(const c64* tw, int k) {
  const c64 w = tw[k];
  return INV ? conj(w) : w;
}

// One line of N points, N / 8 threads; v[m] holds point b + m N / 8 before
// and after.  at(e): the line's LDS slot of point e.  tw: exp(-2 pi i k TS /
// (N TS)), so a table for a longer length serves with step TS.
template <int N, int TS, bool INV, typename At>
__device__ inline void fft_line(c64 (&v)[8], int b, At at, const c64* tw) {
  fft8<INV>(v);
#pragma unroll
  for (int ns = 8; ns < N; ns *= 8) {
    // exchange: the stage before (length ns / 8 runs) leaves its results at
    // (b / p) p 8 + b % p + r p
    const int p = ns / 8;
    const int to = (b / p) * ns + (b & (p - 1));
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 8; ++r) *at(to + r * p) = v[r];
    __syncthreads();
#pragma unroll
    for (int m = 0; m < 8; ++m) v[m] = *at(b + m * (N / 8));
    if (N / ns >= 8) {
      const int k = (b & (ns - 1)) * (N / (ns * 8)) * TS;
      const c64 w1 = root<INV>(tw, k), w2 = root<INV>(tw, 2 * k), w4 = root<INV>(tw, 4 * k);
      const c64 w3 = w1 * w2;
      v[1] = v[1] * w1;
      v[2] = v[2] * w2;
      v[3] = v[3] * w3;
      v[4] = v[4] * w4;
      v[5] = v[5] * (w1 * w4);
      v[6] = v[6] * (w2 * w4);
      v[7] = v[7] * (w3 * w4);
      fft8<INV>(v);
    } else if (N / ns == 4) {
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const int k = ((b + s * (N / 8)) & (ns - 1)) * TS;      // N / (ns 4) = 1
        const c64 w1 = root<INV>(tw, k), w2 = root<INV>(tw, 2 * k);
        v[s + 2] = v[s + 2] * w1;
        v[s + 4] = v[s + 4] * w2;
        v[s + 6] = v[s + 6] * (w1 * w2);
        fft4<INV>(v[s], v[s + 2], v[s + 4], v[s + 6]);
      }
    } else {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int k = ((b + s * (N / 8)) & (ns - 1)) * TS;      // N / (ns 2) = 1
        const c64 u = v[s + 4] * root<INV>(tw, k);
        v[s + 4] = v[s] - u;
        v[s] = v[s] + u;
      }
    }
  }
}

// Columns per tile of the y and z passes: 128-byte rows, and at least a wave.
constexpr int fft_cols(int n) { return n >= 2048 ? 4 : n >= 256 ? 8 : n >= 64 ? 16 : n >= 16 ? 32 : 64; }

enum { kFwd, kInv, kSolve };

// The axis of stride `stride`: columns i of outer index blockIdx.y (stride
// `outer`).  kSolve (the z axis, outer index j): forward, divide, inverse.
template <int N, int MODE>
__global__ void __launch_bounds__(N * fft_cols(N) / 8)
k_fft_cols(c64* __restrict__ data, int hx, int64_t stride, int64_t outer, const c64* __restrict__ tw,
           const double* __restrict__ sym, double kappa_h2, double inv_n3) {
  constexpr int C = fft_cols(N);
  __shared__ c64 lds[N > 8 ? N * 9 / 8 * C : 1];
  const int c = threadIdx.x % C, b = threadIdx.x / C;
  const int i = blockIdx.x * C + c;
  const bool on = i < hx;
  c64* p = data + blockIdx.y * outer + i;
  // one row of padding per 8 points: the first exchange writes rows 8 apart
  auto at = [&](int e) { return lds + (e + (e >> 3)) * C + c; };
  c64 v[8];
#pragma unroll
  for (int m = 0; m < 8; ++m) v[m] = on ? p[(b + m * (N / 8)) * stride] : c64{0.0, 0.0};
  fft_line<N, 1, MODE == kInv>(v, b, at, tw);
  if (MODE == kSolve) {
    const double sij = on ? sym[i] + sym[blockIdx.y] : 1.0;
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const double s = -(sij + sym[b + m * (N / 8)]) - kappa_h2;
      const double g = s != 0.0 ? inv_n3 / s : 0.0;
      v[m] = {v[m].x * g, v[m].y * g};
    }
    fft_line<N, 1, true>(v, b, at, tw);
  }
  if (on) {
#pragma unroll
    for (int m = 0; m < 8; ++m) p[(b + m * (N / 8)) * stride] = v[m];
  }
}

// The x axis: N real values of a row <-> its N / 2 + 1 coefficients.
template <int N>
constexpr int fft_rows() { return N >= 64 ? 4096 / N : N >= 16 ? 1024 / N : 64; }

template <int N, bool INV>
__global__ void __launch_bounds__(N >= 16 ? fft_rows<N>() * N / 16 : 64)
k_fft_rows(const double* __restrict__ real_in, c64* __restrict__ spec, double* __restrict__ real_out,
           int pitch, const c64* __restrict__ tw) {
  if constexpr (N == 8) {
    // one thread per row, as a complex line with zero imaginary part
    const int row = blockIdx.x * 64 + threadIdx.x;
    if (row >= N * N) return;
    c64 v[8];
    if (!INV) {
#pragma unroll
      for (int m = 0; m < 8; ++m) v[m] = {real_in[(int64_t)row * N + m], 0.0};
      fft8<false>(v);
#pragma unroll
      for (int m = 0; m <= 4; ++m) spec[(int64_t)row * pitch + m] = v[m];
    } else {
#pragma unroll
      for (int m = 0; m <= 4; ++m) v[m] = spec[(int64_t)row * pitch + m];
      v[0].y = v[4].y = 0.0;
#pragma unroll
      for (int m = 5; m < 8; ++m) v[m] = conj(v[8 - m]);
      fft8<true>(v);
#pragma unroll
      for (int m = 0; m < 8; ++m) real_out[(int64_t)row * N + m] = v[m].x;
    }
    return;
  } else {
    constexpr int M = N / 2, Q = M / 8, R = fft_rows<N>();
    __shared__ c64 lds[R * (M + Q)];
    const int b = threadIdx.x % Q, row = threadIdx.x / Q;
    c64* line = lds + row * (M + Q);
    auto at = [&](int e) { return line + e + (e >> 3); };
    const int64_t r = (int64_t)blockIdx.x * R + row;
    c64* s = spec + r * pitch;
    typedef double f64x2 __attribute__((ext_vector_type(2), aligned(8)));
    c64 v[8];
    if (!INV) {
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        const f64x2 x = *(const f64x2*)(real_in + r * N + 2 * (b + m * Q));
        v[m] = {x[0], x[1]};
      }
      fft_line<M, 2, false>(v, b, at, tw);
      __syncthreads();
#pragma unroll
      for (int m = 0; m < 8; ++m) *at(b + m * Q) = v[m];
      __syncthreads();
      // even and odd samples' spectra: X[k] = E + w^k O
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        const int k = b + m * Q;
        const c64 z = v[m], zc = conj(*at((M - k) & (M - 1)));
        const c64 e = {0.5 * (z.x + zc.x), 0.5 * (z.y + zc.y)};
        const c64 o = {0.5 * (z.y - zc.y), -0.5 * (z.x - zc.x)};
        s[k] = e + tw[k] * o;
        if (k == 0) s[M] = {z.x - z.y, 0.0};
      }
    } else {
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        v[m] = s[b + m * Q];
        *at(b + m * Q) = v[m];
      }
      __syncthreads();
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        const int k = b + m * Q;
        if (k == 0) {
          const double x0 = v[m].x, xm = s[M].x;
          v[m] = {x0 + xm, x0 - xm};
        } else {
          const c64 xc = conj(*at(M - k));
          const c64 d = (v[m] - xc) * conj(tw[k]);
          v[m] = {v[m].x + xc.x - d.y, v[m].y + xc.y + d.x};
        }
      }
      fft_line<M, 2, true>(v, b, at, tw);
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        f64x2 x;
        x[0] = v[m].x;
        x[1] = v[m].y;
        *(f64x2*)(real_out + r * N + 2 * (b + m * Q)) = x;
      }
    }
  }
}

__global__ void __launch_bounds__(256) k_fft_tables(c64* __restrict__ tw, double* __restrict__ sym, int n) {
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (k >= n) return;
  double s, c;
  sincospi(2.0 * k / n, &s, &c);
  tw[k] = {c, -s};
  const double h = sinpi((double)k / n);
  sym[k] = 4.0 * h * h;                        // 2 - 2 cos(2 pi k / n) without its cancellation
}

// The launches' own status: hipGetLastError would also return what another
// caller left in the thread before.
template <typename... P, typename... A>
bool launched(void (*kernel)(P...), dim3 grid, dim3 block, hipStream_t st, A... a) {
  std::tuple<P...> args(a...);
  return std::apply(
      [&](auto&... v) {
        void* at[] = {(void*)&v...};
        return hipLaunchKernel((const void*)kernel, grid, block, at, 0, st) == hipSuccess;
      },
      args);
}

template <int N, int MODE>
bool cols(const FftPlan& p, bool z, double kappa_h2, hipStream_t st) {
  constexpr int C = fft_cols(N);
  const int64_t row = p.pitch, plane = (int64_t)p.pitch * N;
  const int hx = N / 2 + 1;
  return launched(k_fft_cols<N, MODE>, dim3((hx + C - 1) / C, N), dim3(N * C / 8), st, (c64*)p.c, hx,
                  z ? plane : row, z ? row : plane, (const c64*)p.tw, p.sym, kappa_h2,
                  1.0 / ((double)N * N * N));
}
template <int N, bool INV>
bool rows(const FftPlan& p, const double* in, double* out, hipStream_t st) {
  constexpr int R = fft_rows<N>();
  return launched(k_fft_rows<N, INV>, dim3((N * N + R - 1) / R), dim3(N >= 16 ? R * N / 16 : 64), st,
                  in, (c64*)p.c, out, p.pitch, (const c64*)p.tw);
}
template <int N>
bool forward_n(const FftPlan& p, const double* in, hipStream_t st) {
  return rows<N, false>(p, in, nullptr, st) && cols<N, kFwd>(p, false, 0.0, st) &&
         cols<N, kFwd>(p, true, 0.0, st);
}
template <int N>
bool solve_n(const FftPlan& p, const double* rhs, double* phi, double kappa_h2, hipStream_t st) {
  const double cells = (double)N * N * N;
  prof_begin(st, K_FFT);
  bool ok = rows<N, false>(p, rhs, nullptr, st) && cols<N, kFwd>(p, false, 0.0, st);
  prof_end(st, K_FFT, 32.0 * cells, 2);      // rhs in, the half spectrum out, in and out
  prof_begin(st, K_FFT_DIVIDE);
  ok = ok && cols<N, kSolve>(p, true, kappa_h2, st);
  prof_end(st, K_FFT_DIVIDE, 16.0 * cells);
  prof_begin(st, K_FFT);
  ok = ok && cols<N, kInv>(p, false, 0.0, st) && rows<N, true>(p, nullptr, phi, st);
  prof_end(st, K_FFT, 32.0 * cells, 2);
  return ok;
}

// the padded half spectrum, then the root table
int fft_pitch(int n) { return n >= 32 ? n / 2 + 8 : n / 2 + 1; }

}  // namespace

size_t fft_complex_bytes(int n) { return (size_t)n * n * (n / 2 + 1) * sizeof(c64); }

// Fits 2 fft_complex_bytes(n), the size the layouts reserve: the padding takes
// at most 7 of n / 2 + 1 further columns and the table one row.
int fft_init(FftPlan* p, int n, void* buf, double* sym_dev, hipStream_t st) {
  p->n = n;
  p->pitch = fft_pitch(n);
  p->c = buf;
  p->tw = (char*)buf + (size_t)n * n * p->pitch * sizeof(c64);
  p->sym = sym_dev;
  return launched(k_fft_tables, dim3((n + 255) / 256), dim3(256), st, (c64*)p->tw, p->sym, n) ? SDPM_OK
                                                                                              : SDPM_EHIP;
}

#define FFT_SIZES(DO) \
  DO(8) DO(16) DO(32) DO(64) DO(128) DO(256) DO(512) DO(1024) DO(2048)

int fft_forward(const FftPlan& p, const double* in, hipStream_t st) {
  switch (p.n) {
#define FFT_CASE(N) case N: return forward_n<N>(p, in, st) ? SDPM_OK : SDPM_EHIP;
    FFT_SIZES(FFT_CASE)
#undef FFT_CASE
  }
  return SDPM_EINVAL;
}

int fft_solve(const FftPlan& p, const double* rhs, double* phi, double kappa_h2, hipStream_t st) {
  switch (p.n) {
#define FFT_CASE(N) case N: return solve_n<N>(p, rhs, phi, kappa_h2, st) ? SDPM_OK : SDPM_EHIP;
    FFT_SIZES(FFT_CASE)
#undef FFT_CASE
  }
  return SDPM_EINVAL;
}

}  // namespace sdpm

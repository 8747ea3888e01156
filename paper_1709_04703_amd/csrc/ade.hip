// The paper's alternating-direction explicit (ADE) integrator of the gravity
// diffusion equation (Sec. 2.1 Eq. 4, Sec. 2.3).  One Saul'yev sweep of a
// half sub-step updates every cell of the active box in place,
//   (1 + 3 lam) phi_c' = (1 - 3 lam) phi_c + lam (S6 - f_c),
// lam = 1 / (kappa h^2), f = S h^2 delta, S6 the sum of the six neighbours'
// current values, visiting the cells in lexicographic order (forward: z, y,
// x increasing; backward: all decreasing), so that a neighbour visited
// earlier contributes its new value and one visited later its old value.
// The first half sub-step of a time step sweeps forward, the second
// backward (two consecutive steps in alternate directions).
//
// Parallel form.  Number the rows (j, k) of the box by their distance from
// the sweep's starting corner, (jj, kk).  A row reads the rows (j -+ 1, k)
// and (j, k -+ 1): of these it must find (jj - 1, kk) and (jj, kk - 1) new
// and (jj + 1, kk) and (jj, kk + 1) old; at the far ends of the periodic
// mesh the wrap-around row counts by the visiting order (row ny - 1 is old
// for row 0, row 0 new for row ny - 1).  So any order that takes a row after
// its two predecessors gives the sequential sweep's result.
//
// k_ade_march: one launch per sweep.  A workgroup owns T consecutive planes
// kk, one wave each, and marches the rows jj, wave w behind wave w - 1: the
// new row (jj, kk - 1) comes through LDS from the wave before, the new row
// (jj - 1, kk) stays in registers, and the old rows (centre, kk + 1, source)
// are loaded D rows ahead into register rings.  The waves are paced by
// counters in LDS, not by barriers, so that two further waves can wait for
// memory without holding the others up: the output wave mails the last
// plane's new rows to the next workgroup through global memory, the input
// wave fetches the mail of the workgroup before.  A workgroup waits only on
// the ones before it, and draws its place in that order from a counter when it
// starts: those before it then run already or are done, and every wait ends in
// whatever order the workgroups are dispatched and whatever else is on the card
// (with the place taken from the block index, several sweeps at a time could
// fill an XCD with waiting workgroups of which each sweep's next one needs a
// compute unit there).  The sweep takes about ny + nz
// steps of one row and the mail's way (about 4 us) per workgroup, instead of
// ny + nz - 1 dependent launches: 0.18 ms per sweep at 128^3, 0.60 at 256^3,
// 3.02 at 512^3, against 0.83, 2.12 and 8.33 ms.  (Barriers per row and the rows
// published by release and acquire fences: 0.32, 1.06 and 4.4 ms; fetching
// four rows of mail at a time instead of two: 0.65 ms at 256^3.)
//
// Within a row the cell t (counted along the sweep) obeys
//   u_t = c_t + a u_{t-1},   a = lam / (1 + 3 lam),
// with c_t holding the old centre, the later x neighbour, the four row
// neighbours and the source.  Each lane computes the c_t of L consecutive
// cells, a scan of affine maps across the 64 lanes carries the recurrence,
// and each lane then forms its cells; the maps' factors are powers of a that
// do not depend on the row, so only their offsets are scanned.  On the
// periodic mesh the later x neighbour of the row's last cell is its first
// cell, already new: its c_t is corrected with the first cell's new value
// before the scan.
//
// k_ade_diag: rows of more than 512 cells, whose rings do not fit the march's
// registers, take one launch per diagonal jj + kk (all its rows are
// independent), one wave per row, workgroup g rows jj = 4 g .. 4 g + 3 so
// that a row and its neighbour of the previous diagonal share an XCD.
#include <algorithm>

#include "internal.h"

namespace sdpm {
namespace {

constexpr int kAdeRowsPerBlock = 4;   // one row per wave, 4 waves per workgroup

template <int L, bool FWD>
__global__ void __launch_bounds__(256)
k_ade_diag(double* __restrict__ phi, const double* __restrict__ f, int n, Box b, int periodic,
           double lam, int d, int g0) {
  // workgroup g handles rows jj = 4 g .. 4 g + 3 of every diagonal, so a row
  // and its neighbour of the previous diagonal share a workgroup id and
  // therefore an XCD; groups below the diagonal's first row return at once
  if ((int)blockIdx.x < g0) return;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int nx = b.hi[0] - b.lo[0] + 1, ny = b.hi[1] - b.lo[1] + 1, nz = b.hi[2] - b.lo[2] + 1;
  const int jj = (int)blockIdx.x * kAdeRowsPerBlock + wave, kk = d - jj;
  if (jj >= ny || kk < 0 || kk >= nz) return;   // uniform over the wave
  const int m = n - 1;
  const int j = FWD ? b.lo[1] + jj : b.hi[1] - jj;
  const int k = FWD ? b.lo[2] + kk : b.hi[2] - kk;
  const int jm = periodic ? (j - 1) & m : j - 1, jp = periodic ? (j + 1) & m : j + 1;
  const int km = periodic ? (k - 1) & m : k - 1, kp = periodic ? (k + 1) & m : k + 1;
  const int64_t row = ((int64_t)k * n + j) * n;
  const int64_t rjm = ((int64_t)k * n + jm) * n, rjp = ((int64_t)k * n + jp) * n;
  const int64_t rkm = ((int64_t)km * n + j) * n, rkp = ((int64_t)kp * n + j) * n;
  constexpr int dir = FWD ? 1 : -1;
  const int i_first = FWD ? b.lo[0] : b.hi[0];
  const double inv = 1.0 / (1.0 + 3.0 * lam);
  const double co = 1.0 - 3.0 * lam;
  const double a = lam * inv;
  // the value before the first cell: the frozen exterior, or on the periodic
  // mesh the row's other end (not yet visited: old)
  const int i_before = periodic ? (i_first - dir) & m : i_first - dir;
  const double u_before = phi[row + i_before];
  const double first_old = phi[row + i_first];
  double c[L];
#pragma unroll
  for (int q = 0; q < L; ++q) {
    const int t = lane * L + q;
    c[q] = 0.0;
    if (t < nx) {
      const int i = i_first + dir * t;
      const int in = periodic ? (i + dir) & m : i + dir;
      const double s = phi[row + in] + phi[rjm + i] + phi[rjp + i] + phi[rkm + i] + phi[rkp + i];
      c[q] = (co * phi[row + i] + lam * (s - f[row + i])) * inv;
    }
  }
  if (periodic) {
    // the last cell's later x neighbour is the first cell, new by now
    const double u_first = __shfl(c[0] + a * u_before, 0, 64);
#pragma unroll
    for (int q = 0; q < L; ++q)
      if (lane * L + q == nx - 1) c[q] += a * (u_first - first_old);
  }
  // this lane's cells as one affine map u_in -> A u_in + B
  double A = 1.0, B = 0.0;
#pragma unroll
  for (int q = 0; q < L; ++q)
    if (lane * L + q < nx) {
      B = a * B + c[q];
      A *= a;
    }
  // inclusive scan over the lanes: (A, B) after (A', B') is (A A', A B' + B)
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const double Ap = __shfl_up(A, off, 64), Bp = __shfl_up(B, off, 64);
    if (lane >= off) {
      B = A * Bp + B;
      A = A * Ap;
    }
  }
  double Ae = __shfl_up(A, 1, 64), Be = __shfl_up(B, 1, 64);
  if (lane == 0) Ae = 1.0, Be = 0.0;
  double u = Ae * u_before + Be;
#pragma unroll
  for (int q = 0; q < L; ++q) {
    const int t = lane * L + q;
    if (t < nx) {
      u = a * u + c[q];
      phi[row + i_first + dir * t] = u;
    }
  }
}

// x of the lane selected by a DPP control word, 0 where there is none
template <int CTRL, int ROW_MASK>
__device__ inline double dpp0(double x) {
  union { double d; int i[2]; } v, o;
  v.d = x;
  o.i[0] = __builtin_amdgcn_update_dpp(0, v.i[0], CTRL, ROW_MASK, 0xf, true);
  o.i[1] = __builtin_amdgcn_update_dpp(0, v.i[1], CTRL, ROW_MASK, 0xf, true);
  return o.d;
}
__device__ inline double pow_int(double x, int e) {
  double p = 1.0;
  for (; e > 0; e >>= 1, x *= x)
    if (e & 1) p *= x;
  return p;
}

// L doubles of a lane in sweep order from the first cell of a row
template <int L, bool FWD>
__device__ inline void store_cells(double* p, const double (&v)[L]) {
  typedef double f64x2 __attribute__((ext_vector_type(2), aligned(8)));
#pragma unroll
  for (int q = 0; q < L; q += 2) {
    f64x2 x;
    x[0] = v[FWD ? q : L - 1 - q];
    x[1] = v[FWD ? q + 1 : L - 2 - q];
    *(f64x2*)(p + q) = x;
  }
}
template <int L, bool FWD>
__device__ inline void load_cells(const double* p, double (&v)[L]) {
  // two at a time, from memory of 8-byte alignment
  typedef double f64x2 __attribute__((ext_vector_type(2), aligned(8)));
  if constexpr (L == 1) {
    v[0] = p[0];
  } else {
#pragma unroll
    for (int q = 0; q < L; q += 2) {
      const f64x2 x = *(const f64x2*)(p + q);
      v[FWD ? q : L - 1 - q] = x[0];
      v[FWD ? q + 1 : L - 2 - q] = x[1];
    }
  }
}

__device__ inline double lane_value(double x, int l) {
  union { double d; int i[2]; } v;
  v.d = x;
  v.i[0] = __builtin_amdgcn_readlane(v.i[0], l);
  v.i[1] = __builtin_amdgcn_readlane(v.i[1], l);
  return v.d;
}
// Counters in LDS, each written by one wave.  A wave's LDS operations take
// effect in order, so rows written before their count (and counts read before
// their rows) need no more than the compiler to keep that order.
__device__ inline int count_get(const int* c) {
  const int v = __hip_atomic_load(c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  asm volatile("" ::: "memory");
  return v;
}
__device__ inline void count_set(int* c, int v) {
  asm volatile("" ::: "memory");
  __hip_atomic_store(c, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Mail between workgroups: a cell is two 8-byte words, each half of the value
// and the row's number + 1 (0: not yet written).  A word is written and read
// whole, so a row is there when all its words carry its number; no fence and
// no other flag is needed, and nothing else passes between workgroups.
// A row's words lie lane by lane for each cell of a lane and each half
// (`lanes` lanes have cells), so a wave's accesses are contiguous.
template <int L>
__device__ inline void mail_put(uint64_t* row, int lanes, int lane, const double (&x)[L], uint32_t tag) {
  const uint64_t t = (uint64_t)tag << 32;
  if (lane < lanes) {
#pragma unroll
    for (int q = 0; q < L; ++q) {
      const uint64_t v = (uint64_t)__double_as_longlong(x[q]);
      __hip_atomic_store(row + 2 * q * lanes + lane, t | (v & 0xffffffffull), __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(row + (2 * q + 1) * lanes + lane, t | (v >> 32), __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}
// Moves all rows of a mail box into an LDS ring of R rows as they arrive,
// up to P at a time; made counts the rows put into the ring, taken those read
// from it.  Run by one wave.
template <int L, int P, int R>
__device__ inline void mail_to_ring(const uint64_t* box, int lanes, int ny, int lane, double* ring,
                                    int* made, const int* taken) {
  const int at = min(lane, lanes - 1);
  for (int have = 0; have < ny;) {
    uint64_t lo[P][L], hi[P][L];
#pragma unroll
    for (int u = 0; u < P; ++u) {
      const uint64_t* p = box + (int64_t)min(have + u, ny - 1) * (2 * L * lanes) + at;
#pragma unroll
      for (int q = 0; q < L; ++q) {
        lo[u][q] = __hip_atomic_load(p + 2 * q * lanes, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        hi[u][q] = __hip_atomic_load(p + (2 * q + 1) * lanes, __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    while (count_get(taken) < have + P - R) __builtin_amdgcn_s_sleep(1);
    int put = have;
#pragma unroll
    for (int u = 0; u < P; ++u) {
      const uint32_t tag = (uint32_t)(have + u + 1);   // of no row when past the last
      bool ok = put == have + u;                       // and all rows before it are there
#pragma unroll
      for (int q = 0; q < L; ++q)
        ok = ok && (uint32_t)(lo[u][q] >> 32) == tag && (uint32_t)(hi[u][q] >> 32) == tag;
      if (__all(ok)) {
#pragma unroll
        for (int q = 0; q < L; ++q)
          ring[((have + u) % R * L + q) * 64 + lane] =
              __longlong_as_double((long long)((hi[u][q] << 32) | (lo[u][q] & 0xffffffffull)));
        ++put;
      }
    }
    have = put;
    if (lane == 0) count_set(made, have);
  }
}

constexpr int kAdeR = 2;        // rows of the rings between a workgroup's waves

template <int L, int T, int D, bool FWD, bool PER>
__global__ void __launch_bounds__(64 * (T + 2))
k_ade_march(double* phi, const double* f, int n, Box b, double lam, uint64_t* mail,
            unsigned int* ticket) {
  // stage 0 is fed by the input wave with the rows of the plane before this
  // workgroup's first, stage w + 1 by wave w; cell q of lane l at [q][l].  made[s] and
  // taken[s] count the rows put into stage s and read from it.
  constexpr int kAdeIn = 8;                      // rows of the rings from and to other workgroups
  constexpr int kAdeGet = L > 4 ? 1 : 2;         // rows fetched at once
  constexpr int kRow = L * 64;
  __shared__ double rows[(2 * kAdeIn + (T - 1) * kAdeR) * kRow];
  constexpr int kOut = kAdeIn * kRow, kInner = 2 * kOut;   // after the input ring
  __shared__ int made[T + 1], taken[T + 1], place;
  constexpr int dir = FWD ? 1 : -1;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int nx = b.hi[0] - b.lo[0] + 1, ny = b.hi[1] - b.lo[1] + 1, nz = b.hi[2] - b.lo[2] + 1;
  const int m = n - 1;
  if (threadIdx.x <= T) made[threadIdx.x] = taken[threadIdx.x] = 0;
  if (threadIdx.x == 0) place = gridDim.x > 1 ? (int)atomicAdd(ticket, 1u) : 0;
  __syncthreads();
  const int group = __builtin_amdgcn_readfirstlane(place);   // this workgroup's place in the sweep
  const int k0 = group * T, kk = k0 + w;         // this wave's plane, counted along the sweep
  const int last = min(T, nz - k0) - 1;          // this workgroup's last wave with a plane
  const bool next = group + 1 < (int)gridDim.x;  // then all T waves have one
  const int i_first = FWD ? b.lo[0] : b.hi[0];
  // offsets of plane kr and, in a plane, of row jr, wrapped if periodic
  auto plane_at = [&](int kr) -> int64_t {
    int k = FWD ? b.lo[2] + kr : b.hi[2] - kr;
    if (PER) k &= m;
    return (int64_t)k * n * n;
  };
  auto row_at = [&](int jr) -> int64_t {
    int j = FWD ? b.lo[1] + jr : b.hi[1] - jr;
    if (PER) j &= m;
    return (int64_t)j * n;
  };
  // this lane's cells of a row: on the periodic mesh all in the row (lanes
  // past a row shorter than a wave repeat its last cell); in a box cell by
  // cell, those past the row's end repeating its last one
  int idx[L];
#pragma unroll
  for (int q = 0; q < L; ++q) idx[q] = i_first + dir * min(lane * L + q, nx - 1);
  const int vec = FWD ? min(lane * L, n - L) : max(n - (lane + 1) * L, 0);
  auto cells = [&](const double* p, double (&v)[L]) {
    if constexpr (PER) {
      load_cells<L, FWD>(p + vec, v);
    } else {
#pragma unroll
      for (int q = 0; q < L; ++q) v[q] = p[idx[q]];
    }
  };
  auto put_cells = [&](double* p, const double (&v)[L]) {
    if constexpr (PER && L > 1) {
      store_cells<L, FWD>(p + vec, v);
    } else {
#pragma unroll
      for (int q = 0; q < L; ++q)
        if (lane * L + q < nx) p[idx[q]] = v[q];
    }
  };

  // mail: on the periodic mesh first a box with the rows of plane 0 (for the
  // wrap-around of the last plane), then one per workgroup with a next one,
  // its last plane's; a box holds all rows, so no writer waits for a reader
  const int lane_last = (nx - 1) / L, row_words = 2 * L * (lane_last + 1);
  const int64_t box_words = (int64_t)ny * row_words;
  uint64_t* const mail1 = mail + (PER ? box_words : 0);
  if (w == T) {
    // input: plane k0 - 1, new, from the workgroup before's mail (workgroup 0:
    // the exterior, or on the periodic mesh plane nz - 1, old until the last
    // workgroup, which comes after this one, writes it)
    if (group > 0) {
      mail_to_ring<L, kAdeGet, kAdeIn>(mail1 + ((int64_t)group - 1) * box_words, lane_last + 1, ny,
                                       lane, rows, &made[0], &taken[0]);
      return;
    }
    const double* p = phi + plane_at(k0 - 1);
    for (int have = 0; have < ny; have += kAdeGet) {
      double v[kAdeGet][L];
#pragma unroll
      for (int u = 0; u < kAdeGet; ++u) cells(p + row_at(min(have + u, ny - 1)), v[u]);
      while (count_get(&taken[0]) < have + kAdeGet - kAdeIn) __builtin_amdgcn_s_sleep(1);
#pragma unroll
      for (int u = 0; u < kAdeGet; ++u)
#pragma unroll
        for (int q = 0; q < L; ++q) rows[((have + u) % kAdeIn * L + q) * 64 + lane] = v[u][q];
      if (lane == 0) count_set(&made[0], min(have + kAdeGet, ny));
    }
    return;
  }
  if (w == T + 1 && next) {
    // output: mails wave T - 1's rows
    uint64_t* box = mail1 + (int64_t)group * box_words;
    for (int k = 0; k < ny; ++k) {
      while (count_get(&made[T]) <= k) __builtin_amdgcn_s_sleep(1);
      double v[L];
#pragma unroll
      for (int q = 0; q < L; ++q) v[q] = rows[kOut + (k % kAdeIn * L + q) * 64 + lane];
      mail_put<L>(box + (int64_t)k * row_words, lane_last + 1, lane, v, k + 1);
      if (lane == 0) count_set(&taken[T], k + 1);
    }
    return;
  }
  if (w == T + 1) {
    // the last workgroup: plane 0, new, for the wrap-around of its last plane
    if (PER)
      mail_to_ring<L, kAdeGet, kAdeIn>(mail, lane_last + 1, ny, lane, rows + kOut, &made[T], &taken[T]);
    return;
  }
  if (w > last) return;

  const double inv = 1.0 / (1.0 + 3.0 * lam);
  const double co = 1.0 - 3.0 * lam;
  const double a = lam * inv;
  // factors of the scan over lanes: windows of 1, 2, 4, 8 lanes, then the
  // lanes up to this one in its row of 16, then in its half
  const double a1 = pow_int(a, L), a2 = a1 * a1, a4 = a2 * a2, a8 = a4 * a4;
  const double a16 = pow_int(a1, (lane & 15) + 1), a32 = pow_int(a1, (lane & 31) + 1);
  // lane 0: the cell before the row; other lanes: the cell after it
  const int i_edge = lane == 0 ? i_first - dir : i_first + dir * nx;
  const int64_t rc = plane_at(kk), rn = plane_at(kk + 1);
  // plane kk + 1 of the last plane is plane 0 on the periodic mesh, new: it
  // comes by mail through the output ring
  const bool wraps = PER && kk == nz - 1;
  double cen[D][L], jp[D][L], src[D][L], edge[D];
  double un[L];                                  // the new row jj - 1
  // entry s of the rings <- row jj: its centre (jj up to ny: the row after
  // the last, new on the periodic mesh by then), plane kk + 1 and source.
  // Rows past the last are clamped and left unused: with a fixed number of
  // memory operations per row the compiler's waits are for the entry in use,
  // not for all in flight.
  auto load = [&](int s, int jj) {
    const int64_t kc = row_at(min(jj, ny)), kr = row_at(min(jj, ny - 1));
    cells(phi + rc + kc, cen[s]);
    cells(phi + rn + kr, jp[s]);
    cells(f + rc + kr, src[s]);
    if (!PER) edge[s] = phi[rc + kr + i_edge];
  };
  cells(phi + rc + row_at(-1), un);
#pragma unroll
  for (int s = 0; s < D; ++s) load(s, s);
  for (int t0 = 0; t0 < ny; t0 += D) {
#pragma unroll
    for (int s = 0; s < D; ++s) {
      const int jj = t0 + s;
      if (jj >= ny) break;                       // uniform
      const double ub = PER ? lane_value(cen[s][L - 1], lane_last) : lane_value(edge[s], 0);
      // the cell after the row (periodic: its first cell, old), and the later
      // x neighbour of the lane's last cell (wave_shl:1)
      const double x_after = PER ? lane_value(cen[s][0], 0) : lane_value(edge[s], 1);
      const double xn = dpp0<0x130, 0xf>(cen[s][0]);
      if (wraps) {
        for (;;) {
          const int have = count_get(&made[T]);
#pragma unroll
          for (int q = 0; q < L; ++q) jp[s][q] = rows[kOut + (jj % kAdeIn * L + q) * 64 + lane];
          if (have > jj) break;
        }
        if (lane == 0) count_set(&taken[T], jj + 1);
      }
      double c[L];
#pragma unroll
      for (int q = 0; q < L; ++q) {
        double xq = q < L - 1 ? cen[s][q < L - 1 ? q + 1 : 0] : xn;
        if (lane * L + q == nx - 1) xq = x_after;
        const double s4 = (xq + jp[s][q]) + (un[q] + cen[(s + 1) % D][q]);
        c[q] = s4 - src[s][q];
      }
      // the new row of plane kk - 1
      const int before = w == 0 ? jj % kAdeIn * kRow : kInner + ((w - 1) * kAdeR + jj % kAdeR) * kRow;
      double v[L];
      for (;;) {
        const int have = count_get(&made[w]);
#pragma unroll
        for (int q = 0; q < L; ++q) v[q] = rows[before + q * 64 + lane];
        if (have > jj) break;
      }
      if (lane == 0) count_set(&taken[w], jj + 1);
      // one sum and one factor for all of c, as in k_ade_diag: with a factor a of
      // its own for v a smooth field's error was a third larger at lam = 1000
      // (co cen, the largest term for small lam, enters unrounded)
#pragma unroll
      for (int q = 0; q < L; ++q) c[q] = __builtin_fma(co, cen[s][q], lam * (c[q] + v[q])) * inv;
      if (PER) {
        // the last cell's later x neighbour is the first cell, new by now
        const double u_first = lane_value(c[0] + a * ub, 0);
#pragma unroll
        for (int q = 0; q < L; ++q)
          if (lane * L + q == nx - 1) c[q] += a * (u_first - x_after);
      }
      double B = lane == 0 ? ub : 0.0;
#pragma unroll
      for (int q = 0; q < L; ++q) B = a * B + c[q];
      B += a1 * dpp0<0x111, 0xf>(B);             // row_shr:1, 2, 4, 8
      B += a2 * dpp0<0x112, 0xf>(B);
      B += a4 * dpp0<0x114, 0xf>(B);
      B += a8 * dpp0<0x118, 0xf>(B);
      B += a16 * dpp0<0x142, 0xa>(B);            // row_bcast:15 into rows 1 and 3
      B += a32 * dpp0<0x143, 0xc>(B);            // row_bcast:31 into rows 2 and 3
      double u = dpp0<0x138, 0xf>(B);            // wave_shr:1
      if (lane == 0) u = ub;
#pragma unroll
      for (int q = 0; q < L; ++q) un[q] = u = a * u + c[q];
      if (w < last || next) {
        const bool out = w == T - 1;
        while (count_get(&taken[w + 1]) < jj + 1 - (out ? kAdeIn : kAdeR)) __builtin_amdgcn_s_sleep(0);
        const int to = out ? kOut + jj % kAdeIn * kRow : kInner + (w * kAdeR + jj % kAdeR) * kRow;
#pragma unroll
        for (int q = 0; q < L; ++q) rows[to + q * 64 + lane] = un[q];
        if (lane == 0) count_set(&made[w + 1], jj + 1);
      }
      put_cells(phi + rc + row_at(jj), un);
      if (PER && kk == 0) mail_put<L>(mail + (int64_t)jj * row_words, lane_last + 1, lane, un, jj + 1);
      load(s, jj + D);
    }
  }
}

__global__ void __launch_bounds__(256)
k_ade_clear(uint64_t* mail, int64_t words, unsigned int* ticket) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *ticket = 0u;
  for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < words; q += (int64_t)gridDim.x * 256)
    mail[q] = 0u;
}

template <int L, int T, int D>
void ade_march(double* phi, const double* f, int n, const Box& b, int periodic, double lam,
               bool forward, uint64_t* mail, unsigned int* ticket, hipStream_t st) {
  const int64_t nx = b.hi[0] - b.lo[0] + 1, ny = b.hi[1] - b.lo[1] + 1, nz = b.hi[2] - b.lo[2] + 1;
  const dim3 grid((unsigned)((nz + T - 1) / T)), block(64 * (T + 2));
  const int64_t words = 2 * ((nx + L - 1) / L * L) * ny * ((int64_t)grid.x - (periodic ? 0 : 1));
  if (words > 0)
    hipLaunchKernelGGL(k_ade_clear, dim3((unsigned)std::min<int64_t>((words + 255) / 256, 2048)),
                       dim3(256), 0, st, mail, words, ticket);
  if (periodic && forward)
    hipLaunchKernelGGL((k_ade_march<L, T, D, true, true>), grid, block, 0, st, phi, f, n, b, lam, mail,
                       ticket);
  else if (periodic)
    hipLaunchKernelGGL((k_ade_march<L, T, D, false, true>), grid, block, 0, st, phi, f, n, b, lam, mail,
                       ticket);
  else if (forward)
    hipLaunchKernelGGL((k_ade_march<L, T, D, true, false>), grid, block, 0, st, phi, f, n, b, lam, mail,
                       ticket);
  else
    hipLaunchKernelGGL((k_ade_march<L, T, D, false, false>), grid, block, 0, st, phi, f, n, b, lam, mail,
                       ticket);
}

template <int L>
void ade_diagonals(double* phi, const double* f, int n, const Box& b, int periodic, double lam,
                   bool forward, hipStream_t st) {
  const int ny = b.hi[1] - b.lo[1] + 1, nz = b.hi[2] - b.lo[2] + 1;
  for (int d = 0; d <= ny + nz - 2; ++d) {
    const int jlo = std::max(0, d - nz + 1), jhi = std::min(d, ny - 1);
    const unsigned grid = (unsigned)(jhi / kAdeRowsPerBlock + 1);
    const int g0 = jlo / kAdeRowsPerBlock;
    if (forward)
      hipLaunchKernelGGL((k_ade_diag<L, true>), dim3(grid), dim3(256), 0, st, phi, f, n, b,
                         periodic, lam, d, g0);
    else
      hipLaunchKernelGGL((k_ade_diag<L, false>), dim3(grid), dim3(256), 0, st, phi, f, n, b,
                         periodic, lam, d, g0);
  }
}

}  // namespace

void launch_ade_sweep(double* phi, const double* f, int n, const Box& b, bool periodic, double lam,
                      bool forward, void* scratch, unsigned int* ticket, hipStream_t st) {
  const int nx = b.hi[0] - b.lo[0] + 1;
  const int per = periodic ? 1 : 0;
  prof_begin(st, K_ADE);
  // T planes per workgroup (with the input and the output wave 8 waves, two per
  // SIMD, 256 registers each) and D rows of prefetch, as many as these take on
  // the periodic mesh.  In a box, where every cell has an index of its own, rows
  // of more than 128 cells spill (6 registers, 45 of more than 256 cells): boxes
  // of 108^3, 210^3 and 466^3 take 0.15, 0.59 and 4.9 ms (by diagonals 0.70,
  // 1.65 and 7.1)
  if (nx <= 64)
    ade_march<1, 6, 6>(phi, f, n, b, per, lam, forward, (uint64_t*)scratch, ticket, st);
  else if (nx <= 128)
    ade_march<2, 6, 6>(phi, f, n, b, per, lam, forward, (uint64_t*)scratch, ticket, st);
  else if (nx <= 256)
    ade_march<4, 6, 4>(phi, f, n, b, per, lam, forward, (uint64_t*)scratch, ticket, st);
  else if (nx <= 512)
    ade_march<8, 6, 2>(phi, f, n, b, per, lam, forward, (uint64_t*)scratch, ticket, st);
  else if (nx <= 1024)
    ade_diagonals<16>(phi, f, n, b, per, lam, forward, st);
  else
    ade_diagonals<32>(phi, f, n, b, per, lam, forward, st);
  // read phi and f, write phi once per cell
  prof_end(st, K_ADE, 24.0 * box_cells(b));
}

}  // namespace sdpm

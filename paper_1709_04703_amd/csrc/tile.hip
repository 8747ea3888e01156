// The passes of a V(2,2) cycle on its smaller levels, each level's way down
// and way up in one launch.  On levels of 128^3 cells and fewer a separate
// half sweep moves 1-12 MB and takes the 3-7 us of a dependent launch whatever
// its size, and a level takes eleven of them per cycle.
//
// A workgroup takes TS^3 cells with a halo of 5 (6) on each side into LDS (colour
// split), runs the passes there and writes its own cells: each half sweep is
// right one cell less far from the region's faces, and 5 cells are what the
// restriction of the residual after two red-black sweeps from zero reaches
// (red 5, black 4, red 3, black 2, residual 1; 6 from a given correction), or
// the six half sweeps of a coarsest level.  Every thread keeps its cells' right-hand side in registers.
// The halo is computed several times over (4.3 times a tile's cells for TS =
// 16, 11 for TS = 8), which costs less than the launches it replaces:
//   down: red, black, red, black from zero (or from the level's correction),
//         the red residual and its full weighting onto the next level;
//   up:   the next level's correction prolonged onto the black cells, then
//         red, black, red, black;
//   plain: up to six half sweeps from zero, or four, on a coarsest level.
// The workgroups read their neighbours' cells, so a pass never writes the
// array it reads: the way down leaves the black values in the black half of
// t (the residual scratch, whose red half alone the other kernels use), the
// way up reads them there and writes e.
// The arithmetic of every cell is that of the separate kernels (k_smooth_color
// and its 4-cell form, k_resid_red, k_restrict, k_prolong, whose 4-cell forms
// add in another order: V4), so results are bit-identical.
// Bound by LDS reads and barriers at 128^3, by latency below.
// @TILEFIG@
#include "internal.h"

namespace sdpm {
namespace {


template <typename T>
struct TileArgs {
  const T* black;    // black half of the start, or null: from zero
  const T* coarse;   // next level's correction (up)
  const T* r;        // right-hand side, both colours
  T* red_out;        // red half of the result, or null
  T* black_out;      // black half of the result
  T* rc;             // next level's right-hand side (down)
  int n, nc;         // cells a side, of this level and the next
  Box b, bc;         // boxes of both
  int periodic, nhalf;
  T scale, inv_diag, inv_scale, kappa;
};

enum { kPlain, kDown, kDownFrom, kUp };

template <typename T, int TS, int NT, int MODE, bool V4>
__global__ void __launch_bounds__(NT)
k_tile(TileArgs<T> a) {
  constexpr bool DOWN = MODE == kDown || MODE == kDownFrom;
  constexpr int kHalo = MODE == kDownFrom ? 6 : 5;
  constexpr int W = TS + 2 * kHalo, HX = W / 2, NQ = W * W * HX, U = (NQ + NT - 1) / NT;
  __shared__ T E[2][NQ];                         // red, black: (k, j, i >> 1) of the region
  const int n = a.n, m = n - 1, hn = n >> 1;
  const int64_t hc = half_cells(n);
  // tile origin (even in the mesh), region origin
  const int bx = a.b.lo[0] & ~1, by = a.b.lo[1] & ~1, bz = a.b.lo[2] & ~1;
  const int gx = (a.b.hi[0] - bx + TS) / TS, gy = (a.b.hi[1] - by + TS) / TS;
  const int id = (int)xcd_block();
  const int ox = bx + id % gx * TS, oy = by + id / gx % gy * TS, oz = bz + id / (gx * gy) * TS;
  const int rx = ox - kHalo, ry = oy - kHalo, rz = oz - kHalo;
  const int p0 = (rx + ry + rz) & 1;
  // Region pair (k, j, h): its red cell at i = 2 h + s, its black one at
  // 2 h + 1 - s.  Flags per pair: 1 red, 2 black updated (in the box, off the
  // region's faces); 4 s; 8 red, 16 black in this tile (and box).
  int fl[U];
  T rr[2][U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int q = threadIdx.x + u * NT;
    fl[u] = 0;
    rr[0][u] = rr[1][u] = 0;
    if (q >= NQ) continue;
    const int h = q % HX, j = q / HX % W, k = q / (HX * W);
    const int s = (p0 + j + k) & 1;
    const int gj = ry + j, gk = rz + k;
    const bool in_jk = a.periodic || (gj >= a.b.lo[1] && gj <= a.b.hi[1] && gk >= a.b.lo[2] &&
                                      gk <= a.b.hi[2]);
    const bool off_jk = j > 0 && j < W - 1 && k > 0 && k < W - 1;
    const bool tile_jk = j >= kHalo && j < W - kHalo && k >= kHalo && k < W - kHalo;
    const int64_t row = ((int64_t)(gk & m) * n + (gj & m)) * hn;
    int f = s << 2;
    T e[2] = {0, 0};
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int i = 2 * h + (c ? 1 - s : s), gi = rx + i;
      if (!in_jk || !(a.periodic || (gi >= a.b.lo[0] && gi <= a.b.hi[0]))) continue;
      if (off_jk && i > 0 && i < W - 1) f |= 1 << c;
      if (tile_jk && i >= kHalo && i < W - kHalo) f |= 8 << c;
      const int64_t at = row + ((gi & m) >> 1);
      rr[c][u] = a.r[c * hc + at];
      if (c == 0) {
        if (!a.black) e[0] = -a.scale * rr[0][u] * a.inv_diag;
      } else if (a.black) {
        e[1] = a.black[at];
        if constexpr (MODE == kUp) {
          // trilinear: the mean of coarse cells v >> 1 and (v >> 1) + (v & 1)
          // per axis (they coincide for even v)
          const int mc = a.nc - 1, x = gi & m, y = gj & m, z = gk & m;
          const int X[2] = {x >> 1, ((x >> 1) + (x & 1)) & mc};
          const int Y[2] = {y >> 1, ((y >> 1) + (y & 1)) & mc};
          const int Z[2] = {z >> 1, ((z >> 1) + (z & 1)) & mc};
          if constexpr (V4) {
            const int ny = 1 + (y & 1), nz = 1 + (z & 1);
            T l[2] = {0, 0};
            for (int zz = 0; zz < nz; ++zz)
              for (int yy = 0; yy < ny; ++yy) {
                l[0] += a.coarse[sidx(X[0], Y[yy], Z[zz], a.nc)];
                l[1] += a.coarse[sidx(X[1], Y[yy], Z[zz], a.nc)];
              }
            const T w = (T)0.125 * (T)((3 - ny) * (3 - nz));
            e[1] = e[1] + w * (l[0] + l[1]);
          } else {
            T v[8];
#pragma unroll
            for (int t = 0; t < 8; ++t)
              v[t] = a.coarse[sidx(X[t & 1], Y[(t >> 1) & 1], Z[t >> 2], a.nc)];
            const T sum = v[0] + v[1] + v[2] + v[3] + v[4] + v[5] + v[6] + v[7];
            e[1] += (T)0.125 * sum;
          }
        }
      }
    }
    fl[u] = f;
    E[0][q] = e[0];
    E[1][q] = e[1];
  }
  __syncthreads();
  auto neighbours = [&](const T* o, int q, int s) -> T {
    return o[q - 1 + s] + o[q + s] + o[q - HX] + o[q + HX] + o[q - HX * W] + o[q + HX * W];
  };
  for (int c = a.black ? 0 : 1, left = a.black ? a.nhalf : a.nhalf - 1; left > 0; c ^= 1, --left) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int q = threadIdx.x + u * NT;
      if (!(fl[u] & (1 << c))) continue;
      // s of this cell: which of the pair's two places it has
      const int s = ((fl[u] >> 2) & 1) ^ c;
      const T nb = neighbours(E[c ^ 1], q, s);
      E[c][q] = (nb - a.scale * (c ? rr[1][u] : rr[0][u])) * a.inv_diag;
    }
    __syncthreads();
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int q = threadIdx.x + u * NT;
    if (!(fl[u] & 24)) continue;
    const int h = q % HX, j = q / HX % W, k = q / (HX * W), s = (fl[u] >> 2) & 1;
    const int64_t row = ((int64_t)((rz + k) & m) * n + ((ry + j) & m)) * hn;
    if (!DOWN && (fl[u] & 8) && a.red_out)
      a.red_out[row + (((rx + 2 * h + s) & m) >> 1)] = E[0][q];
    if (fl[u] & 16) a.black_out[row + (((rx + 2 * h + 1 - s) & m) >> 1)] = E[1][q];
  }
  if constexpr (DOWN) {
    // the red residual in place of the red cells (no other reads them now)
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int q = threadIdx.x + u * NT;
      if (!(fl[u] & 1)) continue;
      const T ctr = E[0][q];
      const T nb = neighbours(E[1], q, (fl[u] >> 2) & 1);
      E[0][q] = rr[0][u] - (nb - (T)6 * ctr) * a.inv_scale + a.kappa * ctr;
    }
    __syncthreads();
    constexpr int TC = TS / 2;
    for (int q = threadIdx.x; q < TC * TC * TC; q += NT) {
      const int x = q % TC, y = q / TC % TC, z = q / (TC * TC);
      const int I = ox / 2 + x, J = oy / 2 + y, K = oz / 2 + z;
      if (I < a.bc.lo[0] || I > a.bc.hi[0] || J < a.bc.lo[1] || J > a.bc.hi[1] || K < a.bc.lo[2] ||
          K > a.bc.hi[2])
        continue;
      const int i = kHalo + 2 * x, j = kHalo + 2 * y, k = kHalo + 2 * z;
      auto R = [&](int di, int dj, int dk) -> T {
        return E[0][((k + dk) * W + j + dj) * HX + ((i + di) >> 1)];
      };
      const T centre = R(0, 0, 0);
      T edges;
      if constexpr (V4) {
        edges = 0;
        edges += R(-1, -1, 0) + R(1, -1, 0);
        edges += R(-1, 1, 0) + R(1, 1, 0);
        edges += R(-1, 0, -1) + R(1, 0, -1);
        edges += R(-1, 0, 1) + R(1, 0, 1);
        edges += R(0, -1, -1);
        edges += R(0, 1, -1);
        edges += R(0, -1, 1);
        edges += R(0, 1, 1);
      } else {
        edges = R(-1, -1, 0) + R(1, -1, 0) + R(-1, 1, 0) + R(1, 1, 0) +
                R(-1, 0, -1) + R(1, 0, -1) + R(-1, 0, 1) + R(1, 0, 1) +
                R(0, -1, -1) + R(0, 1, -1) + R(0, -1, 1) + R(0, 1, 1);
      }
      a.rc[sidx(I, J, K, a.nc)] = (T)0.125 * centre + (T)0.03125 * edges;
    }
  }
}

template <typename T, int TS, int NT>
void launch(const TileArgs<T>& a, int mode, bool v4, hipStream_t st) {
  unsigned g = 1;
  for (int d = 0; d < 3; ++d) g *= (unsigned)((a.b.hi[d] - (a.b.lo[d] & ~1) + TS) / TS);
  if (mode == kPlain)
    hipLaunchKernelGGL((k_tile<T, TS, NT, kPlain, false>), dim3(g), dim3(NT), 0, st, a);
  else if (mode == kDown && v4)
    hipLaunchKernelGGL((k_tile<T, TS, NT, kDown, sizeof(T) == 4>), dim3(g), dim3(NT), 0, st, a);
  else if (mode == kDown)
    hipLaunchKernelGGL((k_tile<T, TS, NT, kDown, false>), dim3(g), dim3(NT), 0, st, a);
  else if (mode == kDownFrom && v4)
    hipLaunchKernelGGL((k_tile<T, TS, NT, kDownFrom, sizeof(T) == 4>), dim3(g), dim3(NT), 0, st, a);
  else if (mode == kDownFrom)
    hipLaunchKernelGGL((k_tile<T, TS, NT, kDownFrom, false>), dim3(g), dim3(NT), 0, st, a);
  else if (v4)
    hipLaunchKernelGGL((k_tile<T, TS, NT, kUp, sizeof(T) == 4>), dim3(g), dim3(NT), 0, st, a);
  else
    hipLaunchKernelGGL((k_tile<T, TS, NT, kUp, false>), dim3(g), dim3(NT), 0, st, a);
}
template <typename T>
void dispatch(const TileArgs<T>& a, int mode, bool v4, hipStream_t st) {
  launch<T, 8, 512>(a, mode, v4, st);
}

template <typename T>
TileArgs<T> args(const Level& L, int l, double kappa, bool periodic, int nhalf) {
  TileArgs<T> a{};
  a.r = (const T*)L.r;
  a.n = L.n;
  a.b = L.box;
  a.periodic = periodic ? 1 : 0;
  a.nhalf = nhalf;
  const double s = (double)(1ll << (2 * l));
  a.scale = (T)s;
  a.inv_diag = (T)(1.0 / (6.0 + s * kappa));
  a.inv_scale = (T)(1.0 / s);
  a.kappa = (T)kappa;
  return a;
}

}  // namespace

template <typename T>
void launch_tile_down(const Level& L, const Level& C, int l, double kappa, bool periodic, bool zero,
                      bool v4, hipStream_t st) {
  TileArgs<T> a = args<T>(L, l, kappa, periodic, 4);
  const int64_t hc = half_cells(L.n);
  a.black = zero ? nullptr : (const T*)L.e + hc;
  a.black_out = (T*)L.t + hc;
  a.rc = (T*)C.r;
  a.nc = C.n;
  a.bc = C.box;
  dispatch<T>(a, zero ? kDown : kDownFrom, v4, st);
}

template <typename T>
void launch_tile_up(const Level& L, const Level& C, int l, double kappa, bool periodic, bool v4,
                    hipStream_t st) {
  TileArgs<T> a = args<T>(L, l, kappa, periodic, 4);
  const int64_t hc = half_cells(L.n);
  a.black = (const T*)L.t + hc;
  a.coarse = (const T*)C.e;
  a.nc = C.n;
  a.red_out = (T*)L.e;
  a.black_out = (T*)L.e + hc;
  dispatch<T>(a, kUp, v4, st);
}

template <typename T>
void launch_tile_sweeps(const Level& L, int l, double kappa, bool periodic, int sweeps,
                        hipStream_t st) {
  const int64_t hc = half_cells(L.n);
  // 6 half sweeps from zero, then 4 a launch, the black values passed on
  // between e and t so that the last launch writes e
  const int first = sweeps < 3 ? sweeps : 3;
  int launches = 1 + (sweeps - first + 1) / 2;
  const T* from = nullptr;
  for (int left = sweeps; left > 0; --launches) {
    const int now = from ? (left < 2 ? left : 2) : first;
    left -= now;
    TileArgs<T> a = args<T>(L, l, kappa, periodic, 2 * now);
    a.black = from;
    a.black_out = (launches & 1 ? (T*)L.e : (T*)L.t) + hc;
    a.red_out = left == 0 ? (T*)L.e : nullptr;
    dispatch<T>(a, kPlain, false, st);
    from = a.black_out;
  }
}

#define INSTANTIATE(T)                                                                             \
  template void launch_tile_down<T>(const Level&, const Level&, int, double, bool, bool, bool,     \
                                    hipStream_t);                                                  \
  template void launch_tile_up<T>(const Level&, const Level&, int, double, bool, bool, hipStream_t); \
  template void launch_tile_sweeps<T>(const Level&, int, double, bool, int, hipStream_t);
INSTANTIATE(float)
INSTANTIATE(double)

}  // namespace sdpm

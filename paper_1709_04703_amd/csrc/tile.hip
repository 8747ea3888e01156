// The passes of a V(2,2) cycle on its smaller levels, each level's way down
// and way up in one launch.  On levels of 64^3 cells and fewer a separate
// half sweep moves a few MB at most and takes the 3-7 us of a dependent launch
// whatever its size, and a level takes eleven of them per cycle.
//
// A workgroup takes TS^3 cells with a halo of 5 (6) on each side into LDS (colour
// split), runs the passes there and writes its own cells: each half sweep is
// right one cell less far from the region's faces, and 5 cells are what the
// restriction of the residual after two red-black sweeps from zero reaches
// (red 5, black 4, red 3, black 2, residual 1; 6 from a given correction), or
// the six half sweeps of a coarsest level.  Every thread keeps its cells'
// right-hand side in registers.
// The halo is computed several times over (11 times a tile's cells for TS =
// 8), which costs less than the launches it replaces:
//   down: red, black, red, black from zero (or from the level's correction),
//         the red residual and its full weighting onto the next level;
//   up:   the next level's correction prolonged onto the black cells, then
//         red, black, red, black;
//   plain: up to six half sweeps from zero, or four, on a coarsest level.
// The workgroups read their neighbours' cells, so a pass never writes the
// array it reads: the way down leaves the black values in the black half of
// t (the residual scratch, whose red half alone the other kernels use), the
// way up reads them there and writes e.
// Every cell's operations and their order are those of the separate kernels
// (k_smooth_color and its 4-cell form, k_resid_restrict, k_prolong, whose 4-cell
// forms add in another order: V4); solves in FP32 on 8^3 to 128^3 meshes and
// their boxes, and in FP64 on boxes, had the same bits either way.
// Bound by latency: all loads of a thread go out before the first is used, and
// a half sweep's LDS reads before its writes (the other colour is not written
// meanwhile).  64^3 level in FP32: 9.5 us down, 12.3 us up (27 and 23 us in
// separate launches), 32^3: 6 and 9 (42 and 26); FP64 32^3: 8 and 10 (47 and
// 29).  512 threads a workgroup: 10.5 and 15.0 us at 64^3; TS = 16 there: 17.6
// and 20.6 us, and at 128^3 31 and 46 us, more than the separate launches (25
// and 22 us), which the 128^3 level keeps.
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

template <int V>
struct Int {
  static constexpr int value = V;
};

template <typename T, int TS, int NT, int MODE, bool V4>
__global__ void __launch_bounds__(NT)
k_tile(TileArgs<T> a) {
  constexpr bool DOWN = MODE == kDown || MODE == kDownFrom;
  constexpr int kHalo = MODE == kDownFrom ? 6 : 5;
  constexpr int W = TS + 2 * kHalo, HX = W / 2, NQ = W * W * HX, U = (NQ + NT - 1) / NT;
  // coarse cells a side that the region's prolongation draws on
  constexpr int CW = MODE == kUp ? TS / 2 + 7 : 1;
  __shared__ T E[2][NQ];                         // red, black: (k, j, i >> 1) of the region
  __shared__ T P[CW * CW * CW];
  const int n = a.n, m = n - 1, hn = n >> 1, hc = n * n * hn;    // n <= kTileMax
  const unsigned tid = threadIdx.x;
  // tile origin (even in the mesh), region origin
  const int bx = a.b.lo[0] & ~1, by = a.b.lo[1] & ~1, bz = a.b.lo[2] & ~1;
  const unsigned gx = (a.b.hi[0] - bx + TS) / TS, gy = (a.b.hi[1] - by + TS) / TS;
  const unsigned id = (unsigned)xcd_block();
  const int ox = bx + (int)(id % gx) * TS, oy = by + (int)(id / gx % gy) * TS,
            oz = bz + (int)(id / (gx * gy)) * TS;
  const int rx = ox - kHalo, ry = oy - kHalo, rz = oz - kHalo;
  const int p0 = (rx + ry + rz) & 1;
  // Region pair (k, j, h): its red cell at i = 2 h + s, its black one at
  // 2 h + 1 - s.  All loads go out before the first is used; cells outside
  // the box load some cell of the mesh and are masked.
  const bool given = MODE == kUp || MODE == kDownFrom || (MODE == kPlain && a.black);
  int at[2][U];
  T rr[2][U], start[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const unsigned q = tid + u * NT;
    const int h = q % HX, j = q / HX % W, k = q / (HX * W), s = (p0 + j + k) & 1;
    const int row = (((rz + k) & m) * n + ((ry + j) & m)) * hn;
    at[0][u] = row + (((rx + 2 * h + s) & m) >> 1);
    at[1][u] = row + (((rx + 2 * h + 1 - s) & m) >> 1);
    rr[0][u] = a.r[at[0][u]];
    rr[1][u] = a.r[hc + at[1][u]];
    start[u] = given ? a.black[at[1][u]] : (T)0;
  }
  const int cx = (ox >> 1) - 3, cy = (oy >> 1) - 3, cz = (oz >> 1) - 3;
  if constexpr (MODE == kUp) {
    const int mc = a.nc - 1;
#pragma unroll
    for (int u = 0; u < (CW * CW * CW + NT - 1) / NT; ++u) {
      const unsigned q = tid + u * NT;
      if (q < CW * CW * CW) {
        const int x = (cx + (int)(q % CW)) & mc, y = (cy + (int)(q / CW % CW)) & mc,
                  z = (cz + (int)(q / (CW * CW))) & mc;
        P[q] = a.coarse[(int)sidx(x, y, z, a.nc)];
      }
    }
    __syncthreads();
  }
  // Flags per pair: 1 red, 2 black updated (in the box, off the region's
  // faces); 4 s; 8 red, 16 black in this tile (and box).
  int fl[U], qs[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const unsigned q = tid + u * NT;
    const int h = q % HX, j = q / HX % W, k = q / (HX * W), s = (p0 + j + k) & 1;
    const int gj = ry + j, gk = rz + k;
    const bool in_jk = q < NQ && (a.periodic || (gj >= a.b.lo[1] && gj <= a.b.hi[1] &&
                                                 gk >= a.b.lo[2] && gk <= a.b.hi[2]));
    const bool off_jk = j > 0 && j < W - 1 && k > 0 && k < W - 1;
    const bool tile_jk = j >= kHalo && j < W - kHalo && k >= kHalo && k < W - kHalo;
    int f = s << 2;
    bool in[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int i = 2 * h + (c ? 1 - s : s), gi = rx + i;
      in[c] = in_jk && (a.periodic || (gi >= a.b.lo[0] && gi <= a.b.hi[0]));
      if (in[c] && off_jk && i > 0 && i < W - 1) f |= 1 << c;
      if (in[c] && tile_jk && i >= kHalo && i < W - kHalo) f |= 8 << c;
    }
    fl[u] = f;
    // pairs on a face (never updated) read around some inner pair
    qs[u] = off_jk && q < NQ ? (int)q : (W + 1) * HX + 1;
    T red = 0, black = 0;
    if (!given) red = -a.scale * rr[0][u] * a.inv_diag;
    if (given) black = start[u];
    if constexpr (MODE == kUp) {
      // trilinear: the mean of coarse cells v >> 1 and (v >> 1) + (v & 1) per
      // axis (they coincide for even v)
      const int x = rx + 2 * h + 1 - s;
      // region cells may lie below 0: >> rounds down, as the coarse cells do
      const int X = (x >> 1) - cx, Y = (gj >> 1) - cy, Z = (gk >> 1) - cz;
      const int dx = x & 1, dy = gj & 1, dz = gk & 1;
      auto C = [&](int i, int j2, int k2) -> T {
        // pairs past the region's end read entry 0
        return P[q < NQ ? ((Z + k2) * CW + Y + j2) * CW + X + i : 0];
      };
      if constexpr (V4) {
        T l[2] = {0, 0};
        for (int zz = 0; zz <= dz; ++zz)
          for (int yy = 0; yy <= dy; ++yy) {
            l[0] += C(0, yy, zz);
            l[1] += C(dx, yy, zz);
          }
        const T w = (T)0.125 * (T)((2 - dy) * (2 - dz));
        black = black + w * (l[0] + l[1]);
      } else {
        const T sum = C(0, 0, 0) + C(dx, 0, 0) + C(0, dy, 0) + C(dx, dy, 0) +
                      C(0, 0, dz) + C(dx, 0, dz) + C(0, dy, dz) + C(dx, dy, dz);
        black += (T)0.125 * sum;
      }
    }
    if (q < NQ) {
      E[0][q] = in[0] ? red : (T)0;
      E[1][q] = in[1] ? black : (T)0;
    }
  }
  __syncthreads();
  auto neighbours = [&](const T* o, int q, int s) -> T {
    return o[q - 1 + s] + o[q + s] + o[q - HX] + o[q + HX] + o[q - HX * W] + o[q + HX * W];
  };
  auto half_sweep = [&](auto colour) {
    constexpr int c = decltype(colour)::value;
    // the other colour alone is read: all of a thread's reads may go out first
    T v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      // which of the pair's two places this colour's cell has
      const int s = ((fl[u] >> 2) & 1) ^ c;
      const T nb = neighbours(E[c ^ 1], qs[u], s);
      v[u] = (nb - a.scale * rr[c][u]) * a.inv_diag;
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (fl[u] & (1 << c)) E[c][tid + u * NT] = v[u];
    __syncthreads();
  };
  for (int left = a.nhalf; left > 0; left -= 2) {
    if (given || left < a.nhalf) half_sweep(Int<0>{});
    half_sweep(Int<1>{});
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const unsigned q = tid + u * NT;
    if (!DOWN && (fl[u] & 8) && a.red_out) a.red_out[at[0][u]] = E[0][q];
    if (fl[u] & 16) a.black_out[at[1][u]] = E[1][q];
  }
  if constexpr (DOWN) {
    // the red residual in place of the red cells (no other reads them now)
    T v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const T ctr = E[0][qs[u]];
      const T nb = neighbours(E[1], qs[u], (fl[u] >> 2) & 1);
      v[u] = rr[0][u] - (nb - (T)6 * ctr) * a.inv_scale + a.kappa * ctr;
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (fl[u] & 1) E[0][tid + u * NT] = v[u];
    __syncthreads();
    constexpr int TC = TS / 2;
#pragma unroll
    for (int u = 0; u < (TC * TC * TC + NT - 1) / NT; ++u) {
      const unsigned q = tid + u * NT;
      const int x = q % TC, y = q / TC % TC, z = q / (TC * TC);
      const int I = ox / 2 + x, J = oy / 2 + y, K = oz / 2 + z;
      if (q >= TC * TC * TC || I < a.bc.lo[0] || I > a.bc.hi[0] || J < a.bc.lo[1] ||
          J > a.bc.hi[1] || K < a.bc.lo[2] || K > a.bc.hi[2])
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
      a.rc[(int)sidx(I, J, K, a.nc)] = (T)0.125 * centre + (T)0.03125 * edges;
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
  launch<T, 8, 1024>(a, mode, v4, st);
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

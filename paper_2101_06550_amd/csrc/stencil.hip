// stencil.hip -- cuSten-style 2D xy stencil (thesis Ch.3 "Software API",
// "Software Architecture"): blocks of the field plus their halos are staged in
// LDS, each thread writes its own outputs, input and output are separate
// buffers.  Weights of up to 9 x 9 arrive by value in the kernel arguments;
// premap 1 applies the stencil to v^3 - v (the non-linear Cahn-Hilliard term).
// FP64 or FP32 arrays (the arithmetic in the arrays' type).
//
// One workgroup (4 waves) owns a tile 64 vectors wide: 64 lanes of 16 bytes by
// 16 rows where the rows divide into aligned vectors and are wide enough for
// them (the rule is at launch_class), 64 columns by 16 (FP64) or 32 rows
// otherwise.  The tile and its halo are loaded once into LDS (premap applied
// on the way in), the tile's own columns a vector per lane and the few halo
// columns by as many threads as there are; each thread then computes the
// outputs of its columns in its wave's rows, walking down the input rows and
// adding each row's values into all the outputs whose stencil that row falls
// in, so a value is read from LDS once per group of outputs instead of once
// per weight.
// The extents are rounded up to a class (0, 1, 2 or 4 per direction), the
// weights padded with zeros; each class is its own instantiation with the
// loops fully unrolled.  Tiles are numbered so that the tiles one XCD runs
// (blocks go to the XCDs round robin) form a contiguous band of the field, the
// up to seven tiles past eight equal bands last,
// so the halo rows two tiles share meet in one L2 (measured at 8192^2, single
// columns: the 5-point stencil 0.223 ms banded, 0.255 ms in plain order; 3333 x
// 6000, whose tiles are no multiple of eight, 44.8 us against 57.9); the
// outputs are written with non-temporal stores (plain stores: 0.226 ms).
// Memory bounds it: 8192^2 5-point FP64 moves 1.07 GB in 0.183 ms, 5.9 TB/s.
// A second load of every row for the halo columns had cost as many requests
// as the first (0.210 ms; 0.203 with single columns and the halo apart).
#include <hip/hip_runtime.h>

#include <cstdint>

#include "common.hpp"
#include "launch.hpp"

namespace chx {

namespace {

constexpr int kMaxExt = 4;
// Rows per wave, ms at 8191 x 8192 (single columns) and 8192^2 (vectors):
// single columns in FP64 4 (5-point 0.216 against 0.223 at 8, 9 x 9 0.361
// against 0.368), in FP32 8 (5 x 5 at 4095 x 4000 0.0313 against 0.0342 at
// 4); vectors 4 (5-point 0.183 and 9 x 9 0.292 against 0.183 and 0.296 at 8).
// Either way 9 to 26 KB of LDS, six or more workgroups per CU.
template <typename T>
constexpr int kRows = sizeof(T) == 8 ? 4 : 8;
constexpr int kRowsWide = 4;

template <typename T>
struct StencilW {
  T w[(2 * kMaxExt + 1) * (2 * kMaxExt + 1)];
};

// Index of a periodic neighbour.  mode 1: one wrap (the caller guarantees
// n >= the extent), indices past the last one any stencil reads are clamped
// (their values are never used); mode 2: full modulo (tiny fields).
__device__ __forceinline__ int wrap_index(int g, int n, int mode) {
  if (mode == 2) {
    g %= n;
    return g < 0 ? g + n : g;
  }
  g = g < 0 ? g + n : g;
  g = g >= n ? g - n : g;
  return g < n ? g : n - 1;
}

template <int EX, int EY, int VX, int R, typename T>
__global__ __launch_bounds__(256) void stencil2d_tiled(const T* __restrict__ in,
                                                       T* __restrict__ out, int nx, int ny,
                                                       long ld, StencilW<T> W, int ntx,
                                                       int per_xcd, int wrap, int premap,
                                                       int left, int right, int top,
                                                       int bottom) {
  constexpr int TX = 64 * VX, TY = 4 * R;
  constexpr int PX = (TX + 2 * EX + VX - 1) / VX * VX, HY = TY + 2 * EY, WX = 2 * EX + 1;
  constexpr int NV = VX + 2 * EX;
  typedef T Vec __attribute__((ext_vector_type(VX)));
  __shared__ __attribute__((aligned(16))) T tile[HY * PX];
  const int b = blockIdx.x;
  const int t = b < 8 * per_xcd ? (b & 7) * per_xcd + (b >> 3) : b;
  const int by = t / ntx, bx = t - by * ntx;
  const int i0 = bx * TX, j0 = by * TY;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;

  // Every load of the thread is in flight at once: the tile's own columns a
  // vector at a time, then its share of the halo columns; all from in-bounds
  // addresses, values outside the field replaced afterwards.  A last tile
  // past the field's end holds the wrapped columns in its own.
  const auto row = [&](int ly, bool& ok) {
    const int gj = j0 - EY + ly;
    ok = wrap || (gj >= 0 && gj < ny);
    return (long)(wrap ? wrap_index(gj, ny, wrap) : min(max(gj, 0), ny - 1)) * ld;
  };
  constexpr int NK = (HY + 3) / 4;
  const int ci = i0 + VX * lane;
  const bool cin = ci < nx;
  const int cs = cin ? ci : (VX == 1 && wrap == 2 ? ci % nx : min(ci - nx, nx - VX));
  Vec val[NK];
  bool rok[NK];
#pragma unroll
  for (int k = 0; k < NK; ++k) {
    const long r = row(wv + 4 * k, rok[k]);
    val[k] = *reinterpret_cast<const Vec*>(in + r + cs);
  }
  constexpr int NHALO = 2 * EX * HY, NH = (NHALO + 255) / 256;
  T hv[NH > 0 ? NH : 1];
  bool hok[NH > 0 ? NH : 1];
#pragma unroll
  for (int h = 0; h < NH; ++h) {
    const int e = min((int)threadIdx.x + 256 * h, NHALO - 1);
    const int hy = e % HY, hx = e / HY;
    const long r = row(hy, hok[h]);
    const int gi = hx < EX ? i0 - EX + hx : i0 + TX + hx - EX;
    hok[h] = hok[h] && (wrap || (gi >= 0 && gi < nx));
    hv[h] = in[r + (wrap ? wrap_index(gi, nx, wrap) : min(max(gi, 0), nx - 1))];
  }
#pragma unroll
  for (int k = 0; k < NK; ++k) {
    const int ly = wv + 4 * k;
    if (ly < HY) {
#pragma unroll
      for (int u = 0; u < VX; ++u) {
        T v = (rok[k] && (cin || wrap)) ? val[k][u] : T(0);
        if (premap) v = v * v * v - v;
        tile[ly * PX + EX + VX * lane + u] = v;
      }
    }
  }
#pragma unroll
  for (int h = 0; h < NH; ++h) {
    const int e = (int)threadIdx.x + 256 * h;
    if (e < NHALO) {
      const int hy = e % HY, hx = e / HY;
      T v = hok[h] ? hv[h] : T(0);
      if (premap) v = v * v * v - v;
      tile[hy * PX + (hx < EX ? hx : TX + hx)] = v;
    }
  }
  __syncthreads();
  if (!cin || (!wrap && (ci + VX - 1 < left || ci + right >= nx))) return;  // no outputs

  T acc[R][VX];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int u = 0; u < VX; ++u) acc[r][u] = T(0);
  const T* col = tile + wv * R * PX + VX * lane;
#pragma unroll
  for (int k = 0; k < R + 2 * EY; ++k) {
    T v[NV];
#pragma unroll
    for (int p = 0; p < NV; ++p) v[p] = col[k * PX + p];
#pragma unroll
    for (int q = 0; q <= 2 * EY; ++q) {
      const int r = k - q;
      if (r < 0 || r >= R) continue;
#pragma unroll
      for (int p = 0; p < WX; ++p)
#pragma unroll
        for (int u = 0; u < VX; ++u) acc[r][u] = fma(W.w[q * WX + p], v[p + u], acc[r][u]);
    }
    // one input row at a time: the sums this row fed are complete before the
    // next row's values are read, so only one row's worth of values is live
#pragma unroll
    for (int q = 0; q <= 2 * EY; ++q) {
      const int r = k - q;
      if (r >= 0 && r < R)
#pragma unroll
        for (int u = 0; u < VX; ++u) asm volatile("" : "+v"(acc[r][u])::"memory");
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int j = j0 + wv * R + r;
    if (j >= ny) break;
    if (!wrap && (j - top < 0 || j + bottom >= ny)) continue;
    Vec o;
#pragma unroll
    for (int u = 0; u < VX; ++u) o[u] = acc[r][u];
    if (wrap || (ci >= left && ci + VX - 1 + right < nx)) {
      __builtin_nontemporal_store(o, reinterpret_cast<Vec*>(out + (long)j * ld + ci));
    } else {
#pragma unroll
      for (int u = 0; u < VX; ++u)
        if (ci + u >= left && ci + u + right < nx) out[(long)j * ld + ci + u] = o[u];
    }
  }
}

long tiles(int n, int t) { return ((long)n + t - 1) / t; }

int ext_class(int e) { return e <= 2 ? e : kMaxExt; }

template <int EX, int EY, int VX, int R, typename T>
void launch_tiles(hipStream_t st, const T* in, T* out, int nx, int ny, long ld,
                  const StencilW<T>& W, int wrap, int premap, int left, int right, int top,
                  int bottom) {
  const long ntx = tiles(nx, 64 * VX), ntiles = ntx * tiles(ny, 4 * R);
  hipLaunchKernelGGL((stencil2d_tiled<EX, EY, VX, R, T>), dim3((unsigned)ntiles), dim3(256), 0, st,
                     in, out, nx, ny, ld, W, (int)ntx, (int)(ntiles / 8), wrap,
                     premap, left, right, top, bottom);
}

// Vectors of 16 bytes where the rows are whole aligned vectors (and the field
// at least as large as the stencil's reach), and where the tiles of vectors, 64
// of them wide, are not much wider than the row: a third more columns than
// the tiles of 64 single ones cover, a fifth more for the widest stencils,
// whose idle columns cost most, and twice as many in FP32 for stencils of one
// column.
// us, 16-byte vectors against single columns: 8192^2 5-point FP64 183 / 203,
// FP32 92 / 113, 9 x 9 FP64 292 / 380, FP32 176 / 232; 1000 x 3000 5 x 5 FP32
// 7.2 / 8.9; 66 x 8000 9 x 9 FP64 10.2 / 14.7; 512^2 5-point 6.7 / 6.7.  Fields
// of 2^24 points in rows of 64 FP32 columns (a tile of vectors covers 256): 9 x
// 9 2.73 to 2.92 times as long with vectors, 5-point 1.69 to 2.07; of 260 (1.6
// times the columns) 9 x 9 1.37, 5 x 5 1.07; of 132 (1.33) 9 x 9 1.33, 5-point
// 0.73 to 0.89; of 400 (1.14) 0.90 and 0.75.  FP64 rows of 64 (128) 1.22 to
// 1.27 and 1.07 to 1.40, of 192 (1.33) 0.97 and 1.00; 1 x 5 FP32 rows of 68
// (twice) 0.94.
template <int EX, int EY, typename T>
void launch_class(hipStream_t st, const T* in, T* out, int nx, int ny, long ld,
                  const StencilW<T>& W, int wrap, int premap, int left, int right, int top,
                  int bottom) {
  constexpr int VX = 16 / (int)sizeof(T);
  constexpr int kCover = EX == kMaxExt ? 18 : (EX == 0 && VX == 4 ? 30 : 20);  // fifteenths
  if (nx % VX == 0 && ld % VX == 0 && wrap != 2 &&
      15 * VX * tiles(nx, 64 * VX) <= kCover * tiles(nx, 64) &&
      ((reinterpret_cast<uintptr_t>(in) | reinterpret_cast<uintptr_t>(out)) & 15) == 0)
    launch_tiles<EX, EY, VX, kRowsWide>(st, in, out, nx, ny, ld, W, wrap, premap, left, right, top,
                                        bottom);
  else
    launch_tiles<EX, EY, 1, kRows<T>>(st, in, out, nx, ny, ld, W, wrap, premap, left, right, top,
                                   bottom);
}

template <int EX, typename T>
void launch_ey(int ey, hipStream_t st, const T* in, T* out, int nx, int ny, long ld,
               const StencilW<T>& W, int wrap, int premap, int left,
               int right, int top, int bottom) {
  switch (ey) {
    case 0: launch_class<EX, 0, T>(st, in, out, nx, ny, ld, W, wrap, premap, left, right, top, bottom); break;
    case 1: launch_class<EX, 1, T>(st, in, out, nx, ny, ld, W, wrap, premap, left, right, top, bottom); break;
    case 2: launch_class<EX, 2, T>(st, in, out, nx, ny, ld, W, wrap, premap, left, right, top, bottom); break;
    default: launch_class<EX, 4, T>(st, in, out, nx, ny, ld, W, wrap, premap, left, right, top, bottom); break;
  }
}

template <typename T>
hipError_t launch_stencil2d_t(const T* in, T* out, int nx, int ny, long ld, const double* w,
                              int left, int right, int top, int bottom, int periodic, int premap,
                              hipStream_t st) {
  const int ex = ext_class(left > right ? left : right);
  const int ey = ext_class(top > bottom ? top : bottom);
  // the user's (top + bottom + 1) x (left + right + 1) weights placed in the
  // class's (2 ey + 1) x (2 ex + 1) rectangle, centre on centre (rounded to
  // the array type once, here)
  StencilW<T> W;
  for (T& v : W.w) v = T(0);
  const int uw = left + right + 1;
  for (int q = 0; q <= top + bottom; ++q)
    for (int p = 0; p < uw; ++p)
      W.w[(q - top + ey) * (2 * ex + 1) + (p - left + ex)] = (T)w[q * uw + p];
  const int wrap = !periodic ? 0 : (nx >= ex && ny >= ey ? 1 : 2);
  if (tiles(nx, 64) * tiles(ny, 4 * kRows<T>) > 0x7fffffffL) return hipErrorInvalidValue;
  switch (ex) {
    case 0: launch_ey<0, T>(ey, st, in, out, nx, ny, ld, W, wrap, premap, left, right, top, bottom); break;
    case 1: launch_ey<1, T>(ey, st, in, out, nx, ny, ld, W, wrap, premap, left, right, top, bottom); break;
    case 2: launch_ey<2, T>(ey, st, in, out, nx, ny, ld, W, wrap, premap, left, right, top, bottom); break;
    default: launch_ey<4, T>(ey, st, in, out, nx, ny, ld, W, wrap, premap, left, right, top, bottom); break;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_stencil2d(const double* in, double* out, int nx, int ny, long ld,
                            const double* w, int left, int right, int top, int bottom,
                            int periodic, int premap, hipStream_t st) {
  return launch_stencil2d_t<double>(in, out, nx, ny, ld, w, left, right, top, bottom, periodic,
                                    premap, st);
}

hipError_t launch_stencil2d_f32(const float* in, float* out, int nx, int ny, long ld,
                                const double* w, int left, int right, int top, int bottom,
                                int periodic, int premap, hipStream_t st) {
  return launch_stencil2d_t<float>(in, out, nx, ny, ld, w, left, right, top, bottom, periodic,
                                   premap, st);
}

}  // namespace chx

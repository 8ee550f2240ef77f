// varband.hip -- batched banded solves with one matrix per system.
//
// The thesis's cuPentBatch (Ch.4, "Implementation on GPU") solves a batch of
// pentadiagonal systems, each with its own five diagonals, one thread per
// system on interleaved data (entry i of every system contiguous), with the
// factorisation split from the solve so that a constant matrix is factored
// once; its "Rewrite" variant factors again at every step for matrices that
// change (Ch.4, "Performance Analysis").  Ch.5 does the same for tridiagonal
// systems (Thomas with pre-factorisation).  Here:
//
//  - factor / solve: the factors overwrite the diagonals in place (as in the
//    thesis): b <- beta, c <- 1/alpha, d <- gamma, e <- delta, with a kept as
//    epsilon; tridiagonal: b <- 1/den, c <- chat.
//  - rewrite: factor and solve in one kernel that leaves the diagonals alone;
//    the back sweep's coefficients are computed a second time from the
//    diagonals, or, for few systems and for some that are not periodic, kept
//    in the workspace (the rule and its figures are at rewrite_kind()).
//  - periodic systems: the last two unknowns are bordered off (Ch.4, Navon)
//    or the corners split off as a rank-one term (Ch.5, Sherman-Morrison),
//    both built from each system's own rows.  The correction that the thesis
//    writes with E^{-1} (h^T E^{-1} f, h^T E^{-1} k, or v.y and v.z) is
//    formed during the forward sweep: with E = L R,
//    h^T E^{-1} f = (R^{-T} h) . (L^{-1} f), and R^{-T} h is itself a forward
//    recurrence in the factors already computed.  So every solve is one
//    forward and one backward pass over the data, periodic or not.
//
// Each thread walks its system serially; rows are staged U at a time in
// registers so that U rows of loads are in flight before the recurrence
// consumes them.  Every access of a wave covers 64 consecutive systems of
// one row: 512 contiguous bytes.
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "chx.h"
#include "launch.hpp"

namespace chx_vb {

constexpr int kThreads = 256;
constexpr int kU = 8;  // rows the factor and plain rewrite kernels stage per batch of loads
// The staged loads are non-temporal: every value is used once per pass
// (measured at n = 1024, 65536 systems: factored solves 2-7 % faster).
// The solve kernels stage fewer rows: with one system per thread the batch
// gives one wave per SIMD, and at 65536 systems x 1024 both factored solves
// ran fastest at 6 (penta 1.46 ms against 1.84 ms at 8; tri 0.89 against
// 1.07).
constexpr int kUS = 6;

// ---------------------------------------------------------------------------
// Pentadiagonal.  Row i: a_i x_{i-2} + b_i x_{i-1} + c_i x_i + d_i x_{i+1} +
// e_i x_{i+2}.  Periodic: indices mod n; the leading block E is rows and
// columns 0..m-1 (m = n - 2), k the columns n-2, n-1 of those rows, h the rows
// n-2, n-1 restricted to columns 0..m-1, C22 their 2 x 2 corner.
// ---------------------------------------------------------------------------

// Forward-sweep state of one system.
struct PentaFwd {
  double gm1 = 0, gm2 = 0;  // gamma_{i-1}, gamma_{i-2}
  double dm1 = 0, dm2 = 0;  // delta_{i-1}, delta_{i-2}
  double g1 = 0, g2 = 0;    // g_{i-1}, g_{i-2}
  double p1 = 0, p2 = 0;    // (L^{-1} k0)_{i-1}, _{i-2}
  double q1 = 0, q2 = 0;    // (L^{-1} k1)_{i-1}, _{i-2}
  double u1 = 0, u2 = 0;    // (R^{-T} h0)_{i-1}, _{i-2}
  double v1 = 0, v2 = 0;    // (R^{-T} h1)_{i-1}, _{i-2}
  double s0 = 0, s1 = 0;    // h^T E^{-1} f
  double m00 = 0, m01 = 0, m10 = 0, m11 = 0;  // h^T E^{-1} k
};

// The rows n-2 and n-1 of a periodic system: their entries in h and C22.
struct PentaTail {
  double h0_0, h0_m2, h0_m1;  // row n-2: e (col 0), a (col m-2), b (col m-1)
  double h1_0, h1_1, h1_m1;   // row n-1: d (col 0), e (col 1), a (col m-1)
  double c00, c01, c10, c11;  // C22
  double f0, f1;              // right-hand side of the two rows
};

template <bool PER, bool RHS>
__device__ __forceinline__ void penta_load_tail(int n, long ld, long s, const double* a,
                                                const double* b, const double* c,
                                                const double* d, const double* e,
                                                const double* f, PentaTail& t) {
  const long r0 = (long)(n - 2) * ld + s, r1 = (long)(n - 1) * ld + s;
  t.h0_0 = e[r0];
  t.h0_m2 = a[r0];
  t.h0_m1 = b[r0];
  t.h1_0 = d[r1];
  t.h1_1 = e[r1];
  t.h1_m1 = a[r1];
  t.c00 = c[r0];
  t.c01 = d[r0];
  t.c10 = b[r1];
  t.c11 = c[r1];
  t.f0 = RHS ? f[r0] : 0.0;
  t.f1 = RHS ? f[r1] : 0.0;
}

// One row of the factorisation (and, with RHS, of L g = f) of row i of E.
// ra..re are row i's raw coefficients; the band of E keeps a_i (i >= 2),
// b_i (i >= 1), d_i (i <= m-2), e_i (i <= m-3); the entries that wrap past
// column m-1 form k.  Returns gamma_i, delta_i, 1/alpha_i, beta_i and the
// forward values through the state.
// EDGE: row i may be one of the first or last two, whose band entries, k and
// h differ from the others'; SUMS: the products with h are wanted.
template <bool PER, bool RHS, bool EDGE = true, bool SUMS = true>
__device__ __forceinline__ void penta_fwd_row(int i, int m, double ra, double rb, double rc,
                                              double rd, double re, double rf,
                                              const PentaTail& tl, PentaFwd& st,
                                              double& beta, double& inv, double& gam,
                                              double& del, double& g, double& pk0,
                                              double& pk1, double& wh0, double& wh1) {
  const double ai = (!EDGE || i >= 2) ? ra : 0.0;
  const double bi = (!EDGE || i >= 1) ? rb : 0.0;
  const double di = (!EDGE || i <= m - 2) ? rd : 0.0;
  const double ei = (!EDGE || i <= m - 3) ? re : 0.0;
  beta = bi - ai * st.gm2;
  const double alpha = rc - ai * st.dm2 - beta * st.gm1;
  inv = 1.0 / alpha;
  gam = (di - beta * st.dm1) * inv;
  del = ei * inv;
  g = RHS ? (rf - ai * st.g2 - beta * st.g1) * inv : 0.0;
  pk0 = pk1 = wh0 = wh1 = 0.0;
  if (PER) {
    // columns n-2 and n-1 of row i (k), rows n-2 and n-1 at column i (h)
    double k0 = 0.0, k1 = 0.0, h0 = 0.0, h1 = 0.0;
    if (EDGE && i == 0) {
      k0 = ra;
      k1 = rb;
      h0 = tl.h0_0;
      h1 = tl.h1_0;
    }
    if (EDGE && i == 1) {
      k1 = ra;
      h1 = tl.h1_1;
    }
    if (EDGE && i == m - 2) {
      k0 = k0 + re;
      h0 = h0 + tl.h0_m2;
    }
    if (EDGE && i == m - 1) {
      k0 = k0 + rd;
      k1 = k1 + re;
      h0 = h0 + tl.h0_m1;
      h1 = h1 + tl.h1_m1;
    }
    pk0 = (k0 - ai * st.p2 - beta * st.p1) * inv;
    pk1 = (k1 - ai * st.q2 - beta * st.q1) * inv;
    // R^T w = h: R is unit upper triangular with gamma above the diagonal
    // and delta two above
    if (SUMS) {
      wh0 = h0 - st.gm1 * st.u1 - st.dm2 * st.u2;
      wh1 = h1 - st.gm1 * st.v1 - st.dm2 * st.v2;
      if (RHS) {
        st.s0 = st.s0 + wh0 * g;
        st.s1 = st.s1 + wh1 * g;
      }
      st.m00 = st.m00 + wh0 * pk0;
      st.m01 = st.m01 + wh0 * pk1;
      st.m10 = st.m10 + wh1 * pk0;
      st.m11 = st.m11 + wh1 * pk1;
      st.u2 = st.u1;
      st.u1 = wh0;
      st.v2 = st.v1;
      st.v1 = wh1;
    }
    st.p2 = st.p1;
    st.p1 = pk0;
    st.q2 = st.q1;
    st.q1 = pk1;
  }
  st.gm2 = st.gm1;
  st.gm1 = gam;
  st.dm2 = st.dm1;
  st.dm1 = del;
  st.g2 = st.g1;
  st.g1 = g;
}

// 2 x 2 inverse of C22 - h^T E^{-1} k.
__device__ __forceinline__ void penta_minv(const PentaTail& tl, const PentaFwd& st,
                                           double (&mi)[4]) {
  const double m00 = tl.c00 - st.m00, m01 = tl.c01 - st.m01;
  const double m10 = tl.c10 - st.m10, m11 = tl.c11 - st.m11;
  const double det = m00 * m11 - m01 * m10;
  const double id = 1.0 / det;
  mi[0] = m11 * id;
  mi[1] = -m01 * id;
  mi[2] = -m10 * id;
  mi[3] = m00 * id;
}

// Back sweep R x = g - (L^{-1}k) t over rows m-1..0; x holds g on entry.
template <int U, bool PER>
__device__ __forceinline__ void penta_back(int m, long s, const double* __restrict__ gam,
                                           long ldg, const double* __restrict__ del, long ldd,
                                           const double* __restrict__ pk0,
                                           const double* __restrict__ pk1, long ldw, double t0,
                                           double t1, double* __restrict__ x, long ld) {
  double x1 = 0.0, x2 = 0.0;
  int i = m - 1;
  for (; i + 1 >= U; i -= U) {
    double vg[U], vga[U], vde[U], vp[U], vq[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long r = i - u;
      vg[u] = __builtin_nontemporal_load(&x[r * ld + s]);
      vga[u] = __builtin_nontemporal_load(&gam[r * ldg + s]);
      vde[u] = __builtin_nontemporal_load(&del[r * ldd + s]);
      if (PER) {
        vp[u] = __builtin_nontemporal_load(&pk0[r * ldw + s]);
        vq[u] = __builtin_nontemporal_load(&pk1[r * ldw + s]);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      double v = vg[u];
      if (PER) v = v - vp[u] * t0 - vq[u] * t1;
      v = v - vga[u] * x1 - vde[u] * x2;
      x[(long)(i - u) * ld + s] = v;
      x2 = x1;
      x1 = v;
    }
  }
  for (; i >= 0; --i) {
    double v = x[(long)i * ld + s];
    if (PER) v = v - pk0[(long)i * ldw + s] * t0 - pk1[(long)i * ldw + s] * t1;
    v = v - gam[(long)i * ldg + s] * x1 - del[(long)i * ldd + s] * x2;
    x[(long)i * ld + s] = v;
    x2 = x1;
    x1 = v;
  }
}

// Workspace vectors of a periodic penta batch: rows 0..m-1, stride ldw.
//   factor/solve: [w0 | w1 | pk0 | pk1] then Minv (4 x ldw)
//   rewrite:      the state of the forward sweep before every block of rows
//                 (10 x ldw), or, kept, [gamma | delta | pk0 | pk1], of which
//                 a system that is not periodic has the first two

template <bool PER>
__global__ __launch_bounds__(kThreads) void penta_batch_factor_k(
    int n, int batch, long ld, double* __restrict__ a, double* __restrict__ b,
    double* __restrict__ c, double* __restrict__ d, double* __restrict__ e,
    double* __restrict__ ws, long ldw) {
  const long s = (long)blockIdx.x * kThreads + threadIdx.x;
  if (s >= batch) return;
  const int m = PER ? n - 2 : n;
  PentaTail tl{};
  if (PER) penta_load_tail<PER, false>(n, ld, s, a, b, c, d, e, nullptr, tl);
  double* w0 = PER ? ws : nullptr;
  double* w1 = PER ? ws + (long)m * ldw : nullptr;
  double* p0 = PER ? ws + 2L * m * ldw : nullptr;
  double* p1 = PER ? ws + 3L * m * ldw : nullptr;
  PentaFwd st;
  int i = 0;
  for (; i + kU <= m; i += kU) {
    double va[kU], vb[kU], vc[kU], vd[kU], ve[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const long r = (long)(i + u) * ld + s;
      va[u] = __builtin_nontemporal_load(&a[r]);
      vb[u] = __builtin_nontemporal_load(&b[r]);
      vc[u] = __builtin_nontemporal_load(&c[r]);
      vd[u] = __builtin_nontemporal_load(&d[r]);
      ve[u] = __builtin_nontemporal_load(&e[r]);
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      double beta, inv, gam, del, g, pk0, pk1, wh0, wh1;
      penta_fwd_row<PER, false>(i + u, m, va[u], vb[u], vc[u], vd[u], ve[u], 0.0, tl, st, beta,
                                inv, gam, del, g, pk0, pk1, wh0, wh1);
      const long r = (long)(i + u) * ld + s;
      b[r] = beta;
      c[r] = inv;
      d[r] = gam;
      e[r] = del;
      if (PER) {
        const long rw = (long)(i + u) * ldw + s;
        w0[rw] = wh0;
        w1[rw] = wh1;
        p0[rw] = pk0;
        p1[rw] = pk1;
      }
    }
  }
  for (; i < m; ++i) {
    const long r = (long)i * ld + s;
    double beta, inv, gam, del, g, pk0, pk1, wh0, wh1;
    penta_fwd_row<PER, false>(i, m, a[r], b[r], c[r], d[r], e[r], 0.0, tl, st, beta, inv, gam,
                              del, g, pk0, pk1, wh0, wh1);
    b[r] = beta;
    c[r] = inv;
    d[r] = gam;
    e[r] = del;
    if (PER) {
      const long rw = (long)i * ldw + s;
      w0[rw] = wh0;
      w1[rw] = wh1;
      p0[rw] = pk0;
      p1[rw] = pk1;
    }
  }
  if (PER) {
    double mi[4];
    penta_minv(tl, st, mi);
    double* mv = ws + 4L * m * ldw;
#pragma unroll
    for (int q = 0; q < 4; ++q) mv[(long)q * ldw + s] = mi[q];
  }
}

template <bool PER>
__global__ __launch_bounds__(kThreads) void penta_batch_solve_k(
    int n, int batch, long ld, const double* __restrict__ a, const double* __restrict__ b,
    const double* __restrict__ c, const double* __restrict__ d, const double* __restrict__ e,
    const double* __restrict__ ws, long ldw, double* __restrict__ x) {
  const long s = (long)blockIdx.x * kThreads + threadIdx.x;
  if (s >= batch) return;
  const int m = PER ? n - 2 : n;
  const double* w0 = PER ? ws : nullptr;
  const double* w1 = PER ? ws + (long)m * ldw : nullptr;
  double g1 = 0.0, g2 = 0.0, s0 = 0.0, s1 = 0.0;
  int i = 0;
  for (; i + kUS <= m; i += kUS) {
    double va[kUS], vb[kUS], vc[kUS], vf[kUS], vw0[kUS], vw1[kUS];
#pragma unroll
    for (int u = 0; u < kUS; ++u) {
      const long r = (long)(i + u) * ld + s;
      va[u] = __builtin_nontemporal_load(&a[r]);
      vb[u] = __builtin_nontemporal_load(&b[r]);
      vc[u] = __builtin_nontemporal_load(&c[r]);
      vf[u] = __builtin_nontemporal_load(&x[r]);
      if (PER) {
        vw0[u] = __builtin_nontemporal_load(&w0[(long)(i + u) * ldw + s]);
        vw1[u] = __builtin_nontemporal_load(&w1[(long)(i + u) * ldw + s]);
      }
    }
#pragma unroll
    for (int u = 0; u < kUS; ++u) {
      const double eps = (i + u >= 2) ? va[u] : 0.0;
      const double g = (vf[u] - eps * g2 - vb[u] * g1) * vc[u];
      x[(long)(i + u) * ld + s] = g;
      if (PER) {
        s0 = s0 + vw0[u] * g;
        s1 = s1 + vw1[u] * g;
      }
      g2 = g1;
      g1 = g;
    }
  }
  for (; i < m; ++i) {
    const long r = (long)i * ld + s;
    const double eps = (i >= 2) ? a[r] : 0.0;
    const double g = (x[r] - eps * g2 - b[r] * g1) * c[r];
    x[r] = g;
    if (PER) {
      s0 = s0 + w0[(long)i * ldw + s] * g;
      s1 = s1 + w1[(long)i * ldw + s] * g;
    }
    g2 = g1;
    g1 = g;
  }
  double t0 = 0.0, t1 = 0.0;
  if (PER) {
    const double* mv = ws + 4L * m * ldw;
    const double r0 = x[(long)(n - 2) * ld + s] - s0;
    const double r1 = x[(long)(n - 1) * ld + s] - s1;
    t0 = mv[s] * r0 + mv[ldw + s] * r1;
    t1 = mv[2 * ldw + s] * r0 + mv[3 * ldw + s] * r1;
  }
  penta_back<kUS, PER>(m, s, d, ld, e, ld, PER ? ws + 2L * m * ldw : nullptr,
                  PER ? ws + 3L * m * ldw : nullptr, ldw, t0, t1, x, ld);
  if (PER) {
    x[(long)(n - 2) * ld + s] = t0;
    x[(long)(n - 1) * ld + s] = t1;
  }
}

// ---------------------------------------------------------------------------
// Tridiagonal.  Row i: a_i x_{i-1} + b_i x_i + c_i x_{i+1}.  Periodic: A =
// A' + u v^T with u = (-b_0, 0, .., 0, c_{n-1}), v = (1, 0, .., 0, -a_0/b_0);
// A' drops the corners and has 2 b_0 and b_{n-1} + a_0 c_{n-1} / b_0 on its
// diagonal ends (Ch.5).  A' = L R with den on L's diagonal, a below it, and
// chat above R's unit diagonal; x = R^{-1}(L^{-1} f - phi L^{-1} u) with
// phi = (w . L^{-1} f) / (1 + w . L^{-1} u), w = R^{-T} v.
// Workspace: factor/solve [zu | w] then 1/(1 + v.z); rewrite the state of the
// forward sweep before every block of rows, or, kept, [chat | zu], of which a
// system that is not periodic has the first.
// ---------------------------------------------------------------------------

struct TriFwd {
  double ch1 = 0;  // chat_{i-1}
  double y1 = 0;   // (L^{-1} f)_{i-1}
  double z1 = 0;   // (L^{-1} u)_{i-1}
  double w1 = 0;   // (R^{-T} v)_{i-1}
  double sy = 0, sz = 0;
};

// EDGE: row i may be the first or the last; SUMS: the products with w are
// wanted.
template <bool PER, bool RHS, bool EDGE = true, bool SUMS = true>
__device__ __forceinline__ void tri_fwd_row(int i, int n, double ra, double rb, double rc,
                                            double rf, double a0, double b0, double cl,
                                            TriFwd& st, double& inv, double& ch, double& y,
                                            double& z, double& w) {
  const double ai = (!EDGE || i >= 1) ? ra : 0.0;
  double bi = rb;
  if (EDGE && PER && i == 0) bi = 2.0 * b0;
  if (EDGE && PER && i == n - 1) bi = rb + a0 * cl / b0;
  const double den = bi - ai * st.ch1;
  inv = 1.0 / den;
  ch = (!EDGE || i <= n - 2) ? rc * inv : 0.0;
  y = RHS ? (rf - ai * st.y1) * inv : 0.0;
  z = w = 0.0;
  if (PER) {
    const double ui = (EDGE && i == 0) ? -b0 : ((EDGE && i == n - 1) ? cl : 0.0);
    z = (ui - ai * st.z1) * inv;
    st.z1 = z;
    if (SUMS) {
      const double vi = (EDGE && i == 0) ? 1.0 : ((EDGE && i == n - 1) ? -a0 / b0 : 0.0);
      w = vi - st.ch1 * st.w1;
      if (RHS) st.sy = st.sy + w * y;
      st.sz = st.sz + w * z;
      st.w1 = w;
    }
  }
  st.ch1 = ch;
  st.y1 = y;
}

// x_i = (y_i - phi z_i) - chat_i x_{i+1}, rows n-1..0; x holds y on entry.
template <int U, bool PER>
__device__ __forceinline__ void tri_back(int n, long s, const double* __restrict__ ch, long ldc,
                                         const double* __restrict__ zu, long ldw, double phi,
                                         double* __restrict__ x, long ld) {
  double x1 = 0.0;
  int i = n - 1;
  for (; i + 1 >= U; i -= U) {
    double vy[U], vc[U], vz[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long r = i - u;
      vy[u] = __builtin_nontemporal_load(&x[r * ld + s]);
      vc[u] = __builtin_nontemporal_load(&ch[r * ldc + s]);
      if (PER) vz[u] = __builtin_nontemporal_load(&zu[r * ldw + s]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      double v = vy[u];
      if (PER) v = v - phi * vz[u];
      v = v - vc[u] * x1;
      x[(long)(i - u) * ld + s] = v;
      x1 = v;
    }
  }
  for (; i >= 0; --i) {
    double v = x[(long)i * ld + s];
    if (PER) v = v - phi * zu[(long)i * ldw + s];
    v = v - ch[(long)i * ldc + s] * x1;
    x[(long)i * ld + s] = v;
    x1 = v;
  }
}

template <bool PER>
__global__ __launch_bounds__(kThreads) void tri_batch_factor_k(int n, int batch, long ld,
                                                               double* __restrict__ a,
                                                               double* __restrict__ b,
                                                               double* __restrict__ c,
                                                               double* __restrict__ ws,
                                                               long ldw) {
  const long s = (long)blockIdx.x * kThreads + threadIdx.x;
  if (s >= batch) return;
  const double a0 = PER ? a[s] : 0.0, b0 = PER ? b[s] : 0.0;
  const double cl = PER ? c[(long)(n - 1) * ld + s] : 0.0;
  double* zu = PER ? ws : nullptr;
  double* wv = PER ? ws + (long)n * ldw : nullptr;
  TriFwd st;
  for (int i = 0; i < n; ++i) {
    const long r = (long)i * ld + s;
    double inv, ch, y, z, w;
    tri_fwd_row<PER, false>(i, n, a[r], b[r], c[r], 0.0, a0, b0, cl, st, inv, ch, y, z, w);
    b[r] = inv;
    c[r] = ch;
    if (PER) {
      zu[(long)i * ldw + s] = z;
      wv[(long)i * ldw + s] = w;
    }
  }
  if (PER) ws[2L * n * ldw + s] = 1.0 / (1.0 + st.sz);
}

template <bool PER>
__global__ __launch_bounds__(kThreads) void tri_batch_solve_k(int n, int batch, long ld,
                                                              const double* __restrict__ a,
                                                              const double* __restrict__ b,
                                                              const double* __restrict__ c,
                                                              const double* __restrict__ ws,
                                                              long ldw, double* __restrict__ x) {
  const long s = (long)blockIdx.x * kThreads + threadIdx.x;
  if (s >= batch) return;
  const double* wv = PER ? ws + (long)n * ldw : nullptr;
  double y1 = 0.0, sy = 0.0;
  int i = 0;
  for (; i + kUS <= n; i += kUS) {
    double va[kUS], vb[kUS], vf[kUS], vw[kUS];
#pragma unroll
    for (int u = 0; u < kUS; ++u) {
      const long r = (long)(i + u) * ld + s;
      va[u] = __builtin_nontemporal_load(&a[r]);
      vb[u] = __builtin_nontemporal_load(&b[r]);
      vf[u] = __builtin_nontemporal_load(&x[r]);
      if (PER) vw[u] = __builtin_nontemporal_load(&wv[(long)(i + u) * ldw + s]);
    }
#pragma unroll
    for (int u = 0; u < kUS; ++u) {
      const double ai = (i + u >= 1) ? va[u] : 0.0;
      const double y = (vf[u] - ai * y1) * vb[u];
      x[(long)(i + u) * ld + s] = y;
      if (PER) sy = sy + vw[u] * y;
      y1 = y;
    }
  }
  for (; i < n; ++i) {
    const long r = (long)i * ld + s;
    const double ai = (i >= 1) ? a[r] : 0.0;
    const double y = (x[r] - ai * y1) * b[r];
    x[r] = y;
    if (PER) sy = sy + wv[(long)i * ldw + s] * y;
    y1 = y;
  }
  const double phi = PER ? sy * ws[2L * n * ldw + s] : 0.0;
  tri_back<kUS, PER>(n, s, c, ld, PER ? ws : nullptr, ldw, phi, x, ld);
}

// ---------------------------------------------------------------------------
// Rewrite: factor and solve in one kernel, one system per thread, one wave
// per workgroup so that few systems still spread over many CUs.
//
// A system is two serial sweeps, and a batch rarely gives more than one wave
// per SIMD, so nothing hides a wave's own waits.  Both kernels therefore hold
// two groups of U rows in registers and load one while they work on the
// other.  Past a few tens of thousands of systems the memory traffic bounds
// them: a periodic pentadiagonal row costs 136 bytes if its factors are
// written and read back (6 loads, 5 stores, 5 loads, 1 store) and 109 to 114
// if its coefficients are read a second time and only the sweep's state is
// kept every 32 or 16 rows.  Below that the recurrence bounds them (one FP64
// division and some 25 dependent operations per row).  A branch around the
// loads of a group costs more than the loads of rows that do not exist: the
// wait before the other group then covers both (1024 x 16384: 0.50 ms
// against 0.35).
// ---------------------------------------------------------------------------

constexpr int kWave = 64;

// The two matrices, as the sweeps below see them.  row(): one row of the
// factorisation from its coefficients and right-hand side q; o[0] is the
// forward value, o[1..] what the way back needs beside it (in the order of
// the workspace's vectors).  border(): the bordering's or rank-one term's
// values t from the sums of a whole sweep; free(): the forward value without
// their part.  back(): one row of the back substitution.
template <bool PER>
struct Penta {
  static constexpr int kBands = 5, kOut = PER ? 5 : 3, kBack = 2, kState = PER ? 10 : 6, kEdge = 2;
  static constexpr bool kPeriodic = PER;
  using State = PentaFwd;
  using Tail = PentaTail;
  static __device__ __forceinline__ int rows(int n) { return PER ? n - 2 : n; }
  static __device__ __forceinline__ void tail(int n, long ld, long s, const double* const* q,
                                              Tail& t) {
    if (PER) penta_load_tail<PER, true>(n, ld, s, q[0], q[1], q[2], q[3], q[4], q[5], t);
  }
  template <bool EDGE, bool SUMS>
  static __device__ __forceinline__ void row(int i, int m, const double (&q)[6], const Tail& t,
                                             State& st, double (&o)[kOut]) {
    double beta, inv, pk0, pk1, wh0, wh1;
    penta_fwd_row<PER, true, EDGE, SUMS>(i, m, q[0], q[1], q[2], q[3], q[4], q[5], t, st, beta,
                                         inv, o[1], o[2], o[0], pk0, pk1, wh0, wh1);
    if constexpr (PER) {
      o[3] = pk0;
      o[4] = pk1;
    }
  }
  static __device__ __forceinline__ void border(const Tail& tl, const State& st, double (&t)[2]) {
    if (!PER) return;
    double mi[4];
    penta_minv(tl, st, mi);
    const double r0 = tl.f0 - st.s0, r1 = tl.f1 - st.s1;
    t[0] = mi[0] * r0 + mi[1] * r1;
    t[1] = mi[2] * r0 + mi[3] * r1;
  }
  static __device__ __forceinline__ double free(const double (&o)[kOut], const double (&t)[2]) {
    if constexpr (PER) return o[0] - o[3] * t[0] - o[4] * t[1];
    return o[0];
  }
  static __device__ __forceinline__ double back(double v, double gam, double del, double x1,
                                                double x2) {
    return v - gam * x1 - del * x2;
  }
  static __device__ __forceinline__ void finish(int n, long ld, int lane, const double (&t)[2],
                                                double* x) {
    if (!PER) return;
    x[(long)(n - 2) * ld + lane] = t[0];
    x[(long)(n - 1) * ld + lane] = t[1];
  }
  static __device__ __forceinline__ void save(const State& st, double (&k)[kState]) {
    k[0] = st.gm1, k[1] = st.gm2, k[2] = st.dm1, k[3] = st.dm2, k[4] = st.g1;
    k[5] = st.g2;
    if constexpr (PER) k[6] = st.p1, k[7] = st.p2, k[8] = st.q1, k[9] = st.q2;
  }
  static __device__ __forceinline__ void restore(const double (&k)[kState], State& st) {
    st.gm1 = k[0], st.gm2 = k[1], st.dm1 = k[2], st.dm2 = k[3], st.g1 = k[4];
    st.g2 = k[5];
    if constexpr (PER) st.p1 = k[6], st.p2 = k[7], st.q1 = k[8], st.q2 = k[9];
  }
};

struct TriTail {
  double a0, b0, cl;
};

template <bool PER>
struct Tri {
  static constexpr int kBands = 3, kOut = PER ? 3 : 2, kBack = 1, kState = PER ? 3 : 2, kEdge = 1;
  static constexpr bool kPeriodic = PER;
  using State = TriFwd;
  using Tail = TriTail;
  static __device__ __forceinline__ int rows(int n) { return n; }
  static __device__ __forceinline__ void tail(int n, long ld, long s, const double* const* q,
                                              Tail& t) {
    if (!PER) return;
    t.a0 = q[0][s];
    t.b0 = q[1][s];
    t.cl = q[2][(long)(n - 1) * ld + s];
  }
  template <bool EDGE, bool SUMS>
  static __device__ __forceinline__ void row(int i, int n, const double (&q)[4], const Tail& t,
                                             State& st, double (&o)[kOut]) {
    double inv, z, w;
    tri_fwd_row<PER, true, EDGE, SUMS>(i, n, q[0], q[1], q[2], q[3], t.a0, t.b0, t.cl, st, inv,
                                       o[1], o[0], z, w);
    if constexpr (PER) o[2] = z;
  }
  static __device__ __forceinline__ void border(const Tail&, const State& st, double (&t)[2]) {
    if (PER) t[0] = st.sy / (1.0 + st.sz);
  }
  static __device__ __forceinline__ double free(const double (&o)[kOut], const double (&t)[2]) {
    if constexpr (PER) return o[0] - t[0] * o[2];
    return o[0];
  }
  static __device__ __forceinline__ double back(double v, double ch, double, double x1, double) {
    return v - ch * x1;
  }
  static __device__ __forceinline__ void finish(int, long, int, const double (&)[2], double*) {}
  static __device__ __forceinline__ void save(const State& st, double (&k)[kState]) {
    k[0] = st.ch1, k[1] = st.y1;
    if constexpr (PER) k[2] = st.z1;
  }
  static __device__ __forceinline__ void restore(const double (&k)[kState], State& st) {
    st.ch1 = k[0], st.y1 = k[1];
    if constexpr (PER) st.z1 = k[2];
  }
};

// The bands in order, then the right-hand sides.
template <int Q>
struct Columns {
  const double* p[Q];
};

// U rows of Q arrays, from row i on; rows past the last are its copies, and
// groups past it one element of it.
template <int U, int Q>
struct Group {
  double v[U][Q];
  __device__ __forceinline__ void load(const double* const* p, int i, int last, long ld,
                                       int lane) {
    const unsigned off = i <= last ? 8u * lane : 0u;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long r = (long)min(max(i + u, 0), last) * ld;
#pragma unroll
      for (int j = 0; j < Q; ++j)
        v[u][j] = __builtin_nontemporal_load(reinterpret_cast<const double*>(
            reinterpret_cast<const char*>(p[j] + r) + off));
    }
  }
};

template <class S, bool SUMS, int U, class F>
__device__ __forceinline__ void sweep_group(int i, int m, const Group<U, S::kBands + 1>& g,
                                            const typename S::Tail& tl, typename S::State& st,
                                            const F& f) {
  double o[S::kOut];
  if (i >= S::kEdge && i + U <= m - S::kEdge) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      S::template row<false, SUMS>(i + u, m, g.v[u], tl, st, o);
      f(u, o);
    }
  } else {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i + u < m) {
        S::template row<true, SUMS>(i + u, m, g.v[u], tl, st, o);
        f(u, o);
      }
  }
}

// Kept factors: the forward sweep leaves its values in x and the workspace,
// the back sweep reads them.  Systems that are not periodic only: of the
// others' factors more would have to be kept.
template <class S, int U>
__global__ __launch_bounds__(kWave, 1) void rewrite_once_k(int n, int batch, long ld,
                                                           Columns<S::kBands + 1> in, double* x,
                                                           double* ws, long ldw) {
  static_assert(!S::kPeriodic);
  const long s0 = (long)blockIdx.x * kWave;
  const int lane = threadIdx.x;
  if (s0 + lane >= batch) return;
  const int m = S::rows(n);
  const typename S::Tail tl{};
#pragma unroll
  for (int j = 0; j <= S::kBands; ++j) in.p[j] += s0;
  x += s0;
  ws += s0;
  typename S::State st;
  {
    Group<U, S::kBands + 1> A, B;
    const auto put = [&](int i) {
      return [=](int u, const double (&o)[S::kOut]) {
        x[(long)(i + u) * ld + lane] = o[0];
#pragma unroll
        for (int j = 1; j < S::kOut; ++j) ws[((long)(j - 1) * m + i + u) * ldw + lane] = o[j];
      };
    };
    A.load(in.p, 0, m - 1, ld, lane);
    for (int i = 0; i < m; i += 2 * U) {
      B.load(in.p, i + U, m - 1, ld, lane);
      sweep_group<S, false, U>(i, m, A, tl, st, put(i));
      A.load(in.p, i + 2 * U, m - 1, ld, lane);
      sweep_group<S, false, U>(i + U, m, B, tl, st, put(i + U));
    }
  }
  double x1 = 0.0, x2 = 0.0;
  struct Way {
    double v[U][S::kOut];
  };
  const auto get = [&](int i, Way& g) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = max(i - u, 0);
      g.v[u][0] = __builtin_nontemporal_load(x + (long)r * ld + lane);
#pragma unroll
      for (int j = 1; j < S::kOut; ++j)
        g.v[u][j] = __builtin_nontemporal_load(ws + ((long)(j - 1) * m + r) * ldw + lane);
    }
  };
  const auto back = [&](int i, const Way& g) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i - u >= 0) {
        const double v = S::back(g.v[u][0], g.v[u][1], S::kBack > 1 ? g.v[u][2] : 0.0, x1, x2);
        x[(long)(i - u) * ld + lane] = v;
        x2 = x1;
        x1 = v;
      }
  };
  Way A, B;
  get(m - 1, A);
  for (int i = m - 1; i >= 0; i -= 2 * U) {
    get(i - U, B);
    back(i, A);
    get(i - 2 * U, A);
    back(i - U, B);
  }
}

// Factors computed twice: the forward sweep stores only its state before
// every block of U * SUB rows; the way back takes the blocks in reverse,
// factors each again from its state and substitutes.  All groups of a block
// but the last wait for the substitution in LDS: 36 KB a wave for 32 rows of
// the pentadiagonal, so that four waves, one per SIMD, fit a CU.  The result
// is stored past the caches: 1024 x 65536 takes 1.26 ms against 1.33.
template <class S, int U, int SUB>
__global__ __launch_bounds__(kWave, 1) void rewrite_twice_k(int n, int batch, long ld,
                                                            Columns<S::kBands + 1> in, double* x,
                                                            double* ws, long ldw) {
  static_assert(SUB % 2 == 0, "groups alternate between two sets of registers");
  constexpr int kBlock = U * SUB, kVal = 1 + S::kBack;
  __shared__ double rows[(SUB - 1) * U][kVal][kWave];
  const long s0 = (long)blockIdx.x * kWave;
  const int lane = threadIdx.x;
  if (s0 + lane >= batch) return;
  const int m = S::rows(n);
  typename S::Tail tl{};
  S::tail(n, ld, s0 + lane, in.p, tl);
#pragma unroll
  for (int j = 0; j <= S::kBands; ++j) in.p[j] += s0;
  x += s0;
  ws += s0;
  const int nb = (m + kBlock - 1) / kBlock;
  typename S::State st;
  Group<U, S::kBands + 1> A, B;
  double kept[S::kState];
  A.load(in.p, 0, m - 1, ld, lane);
  for (int k = 0; k < nb; ++k) {
    if (k > 0) {
      S::save(st, kept);
#pragma unroll
      for (int j = 0; j < S::kState; ++j)
        ws[((long)(k - 1) * S::kState + j) * ldw + lane] = kept[j];
    }
#pragma unroll
    for (int g = 0; g < SUB; ++g) {
      const int i = k * kBlock + g * U;
      ((g & 1) ? A : B).load(in.p, i + U, m - 1, ld, lane);
      sweep_group<S, true, U>(i, m, (g & 1) ? B : A, tl, st,
                              [](int, const double (&)[S::kOut]) {});
    }
  }
  double t[2] = {0.0, 0.0};
  S::border(tl, st, t);

  double x1 = 0.0, x2 = 0.0;
  const auto fetch = [&](int k) {
#pragma unroll
    for (int j = 0; j < S::kState; ++j)
      kept[j] = k > 0 ? __builtin_nontemporal_load(
                            ws + ((long)(k - 1) * S::kState + j) * ldw + lane)
                      : 0.0;
  };
  fetch(nb - 1);
  A.load(in.p, (nb - 1) * kBlock, m - 1, ld, lane);
  for (int k = nb - 1; k >= 0; --k) {
    S::restore(kept, st);
    double r[U][kVal];
#pragma unroll
    for (int g = 0; g < SUB; ++g) {
      const int i = k * kBlock + g * U;
      if (g == SUB - 1) fetch(k - 1);
      ((g & 1) ? A : B).load(in.p, g < SUB - 1 ? i + U : (k - 1) * kBlock, m - 1, ld, lane);
      sweep_group<S, false, U>(i, m, (g & 1) ? B : A, tl, st,
                               [&](int u, const double (&o)[S::kOut]) {
                                 r[u][0] = S::free(o, t);
#pragma unroll
                                 for (int j = 1; j < kVal; ++j) r[u][j] = o[j];
                               });
      if (g < SUB - 1) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int j = 0; j < kVal; ++j) rows[g * U + u][j][lane] = r[u][j];
      }
    }
#pragma unroll
    for (int g = SUB - 1; g >= 0; --g) {
      if (g < SUB - 1) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int j = 0; j < kVal; ++j) r[u][j] = rows[g * U + u][j][lane];
      }
      const int i = k * kBlock + g * U;
#pragma unroll
      for (int u = U - 1; u >= 0; --u)
        if (i + u < m) {
          const double v = S::back(r[u][0], r[u][1], kVal > 2 ? r[u][2] : 0.0, x1, x2);
          __builtin_nontemporal_store(v, x + (long)(i + u) * ld + lane);
          x2 = x1;
          x1 = v;
        }
    }
  }
  S::finish(n, ld, lane, t, x);
}

// Kept factors, one group of rows loaded and worked on at a time, for
// tridiagonal systems that are not periodic: 64 bytes a row where bandwidth
// bounds, against 72 of the kernels above.
__global__ __launch_bounds__(kThreads) void tri_rewrite_plain_k(
    int n, int batch, long ld, const double* __restrict__ a, const double* __restrict__ b,
    const double* __restrict__ c, double* __restrict__ x, double* __restrict__ ws, long ldw) {
  const long s = (long)blockIdx.x * kThreads + threadIdx.x;
  if (s >= batch) return;
  TriFwd st;
  int i = 0;
  for (; i + kU <= n; i += kU) {
    double va[kU], vb[kU], vc[kU], vf[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const long r = (long)(i + u) * ld + s;
      va[u] = __builtin_nontemporal_load(&a[r]);
      vb[u] = __builtin_nontemporal_load(&b[r]);
      vc[u] = __builtin_nontemporal_load(&c[r]);
      vf[u] = __builtin_nontemporal_load(&x[r]);
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      double inv, ch, y, z, w;
      tri_fwd_row<false, true>(i + u, n, va[u], vb[u], vc[u], vf[u], 0.0, 0.0, 0.0, st, inv, ch,
                               y, z, w);
      x[(long)(i + u) * ld + s] = y;
      ws[(long)(i + u) * ldw + s] = ch;
    }
  }
  for (; i < n; ++i) {
    const long r = (long)i * ld + s;
    double inv, ch, y, z, w;
    tri_fwd_row<false, true>(i, n, a[r], b[r], c[r], x[r], 0.0, 0.0, 0.0, st, inv, ch, y, z, w);
    x[r] = y;
    ws[(long)i * ldw + s] = ch;
  }
  tri_back<kU, false>(n, s, ws, ldw, nullptr, ldw, 0.0, x, ld);
}

// ---------------------------------------------------------------------------
// Host side: argument checks, workspace layout, launches.
// ---------------------------------------------------------------------------

long ws_ld(int batch) { return ((long)batch + 31) / 32 * 32; }  // 256-byte rows

size_t penta_ws_doubles(int n, int batch, int periodic, int mode) {
  const long m = periodic ? n - 2 : n;
  const long ldw = ws_ld(batch);
  if (mode == CHX_BATCH_REWRITE) return (size_t)((periodic ? 4 : 2) * m * ldw);
  return periodic ? (size_t)((4 * m + 4) * ldw) : 0;
}

size_t tri_ws_doubles(int n, int batch, int periodic, int mode) {
  const long ldw = ws_ld(batch);
  if (mode == CHX_BATCH_REWRITE) return (size_t)((periodic ? 2 : 1) * (long)n * ldw);
  return periodic ? (size_t)((2L * n + 1) * ldw) : 0;
}

int check_common(int n, int batch, long ld, int nmin, int periodic) {
  if (batch < 0 || ld < batch || ld < 1 || (periodic != 0 && periodic != 1)) return CHX_EINVAL;
  if (n < nmin) return CHX_EUNSUPPORTED_N;
  return CHX_OK;
}

int check_ws(const void* ws, size_t ws_bytes, size_t need_doubles) {
  if (need_doubles == 0) return CHX_OK;
  if (!ws || (reinterpret_cast<uintptr_t>(ws) & 255) != 0) return CHX_EINVAL;
  if (ws_bytes < need_doubles * sizeof(double)) return CHX_ENOMEM;
  return CHX_OK;
}

dim3 grid_of(int batch) { return dim3((unsigned)((batch + kThreads - 1) / kThreads)); }

// Which kernel (ms unless us, FP64; "kept" the double set of rows unless plain):
//  - periodic: twice.  1024 x 65536: penta 1.31, tri 0.84, against 1.72 and
//    1.07 kept plain; 512 x 4096: 0.161 and 0.114 against 0.180 and 0.128.
//  - not periodic: twice only where it hides what the batch waits for, 0.317
//    against 0.349 (penta) and 0.216 against 0.297 (tri) at 1024 x 16384;
//    kept below, 0.133 against 0.135 and 0.107 against 0.107 at 512 x 4096,
//    and for short systems, whose factors stay in the last-level cache
//    (100 x 65536: 0.108 against 0.124, 0.076 against 0.078).  Tridiagonal
//    batches of more than three waves a CU are bound by bandwidth, where 72
//    bytes a row kept lose to 64 (plain up to one wave per SIMD, 512 x 50000
//    0.304 against 0.347; two groups of 8 above, 256 x 100000 0.301 against
//    0.352) until the factors pass the last-level cache (1024 x 65536 0.82
//    twice, 0.84 kept).
//    Past three waves a CU the waves hide what each waits for, so the plain
//    kernel's bytes decide past 48 rows (100 x 55000: 73 us against 77).
//  - kept factors in groups of 8 rows rather than 4 for tridiagonals from 64
//    rows on: with one wave per SIMD the loads of 4 rows are not back in time
//    (us, arrays in L2 and not: 256 x 64 45 and 46 against 46 and 59, 1000 x
//    4096 167 and 168 against 211 and 220).  Plain takes 36 and 77 at 256 x 64
//    and 240 and 294 at 1000 x 64: it has nothing in flight while it computes.
//    Shorter systems are over before it matters (56 x 64: 15.1 and 14.9
//    against 13.9 and 17.0, 8 x 200: 10.7 and 7.3 against 10.6 and 6.7);
//    past three waves a CU 4 are as good (100 x 200000: 233 against 250).
//  - few periodic systems likewise: twice 31 and 31 us, plain 24 and 47 (tri of
//    100 x 64), 39 and 39, 36 and 46 (penta).
//  - groups of 4 rows for the pentadiagonal below half a wave per SIMD, where
//    the smaller kernel keeps clear of the accumulation registers (1024 x
//    16384: 0.337 against 0.353), of 8 above (1024 x 65536: 1.31 against
//    1.37); the tridiagonal fits at 8 (1024 x 16384: 0.228 against 0.264).
//  - short systems: blocks of 16 rows up to 48 and of 8 up to 8, as a block's
//    loads are issued whether or not it has the rows; 49 to 64 rows fill the same
//    64 in blocks of 32, and more states would be stored (us, periodic, 100000
//    systems: penta of 8 rows 15.0 in blocks of 8, 22.0 of 16, 37.2 of 32, 19.3
//    plain; of 16 32.6, 30.8, 46.7; tri of 8 10.0, 13.7, 23.0, of 40 50.4 of 16
//    and 60.6 of 32).
constexpr int kTwiceBatch = 16384, kTwiceRows = 256, kWideBatch = 32768;
constexpr int kBandwidthBatch = 3 * 256 * kWave, kSimdBatch = 4 * 256 * kWave;
constexpr int kCachedRows = 768, kGroupRows = 64, kShortRows = 48, kTinyRows = 8;

enum class Rewrite { kPlain, kOnce4, kOnce8, kTwice4x2, kTwice4x4, kTwice8x4 };

template <class S>
Rewrite rewrite_kind(int n, int batch) {
  constexpr bool tri = S::kBands == 3;
  if (S::kPeriodic) {
    const int m = tri ? n : n - 2;
    if (m <= kTinyRows) return Rewrite::kTwice4x2;
    if (m <= kShortRows || (!tri && batch < kWideBatch)) return Rewrite::kTwice4x4;
    return Rewrite::kTwice8x4;
  }
  const bool kept = batch < kTwiceBatch || n < kTwiceRows;
  if (tri && n > kShortRows && batch > kBandwidthBatch && batch < kSimdBatch)
    return Rewrite::kPlain;
  if (tri && n >= kGroupRows && (batch > kBandwidthBatch ? !kept && n < kCachedRows : kept))
    return Rewrite::kOnce8;
  if (kept) return Rewrite::kOnce4;
  return !tri && batch < kWideBatch ? Rewrite::kTwice4x4 : Rewrite::kTwice8x4;
}

template <class S>
void rewrite(int n, int batch, long ld, const Columns<S::kBands + 1>& in, double* x, double* ws,
             hipStream_t st) {
  const dim3 grid((unsigned)((batch + kWave - 1) / kWave)), block(kWave);
  const long ldw = ws_ld(batch);
  switch (rewrite_kind<S>(n, batch)) {
    case Rewrite::kPlain:
      if constexpr (S::kBands == 3 && !S::kPeriodic)
        hipLaunchKernelGGL(tri_rewrite_plain_k, grid_of(batch), dim3(kThreads), 0, st, n, batch, ld,
                           in.p[0], in.p[1], in.p[2], x, ws, ldw);
      return;
    case Rewrite::kOnce4:
      if constexpr (!S::kPeriodic)
        hipLaunchKernelGGL((rewrite_once_k<S, 4>), grid, block, 0, st, n, batch, ld, in, x, ws,
                           ldw);
      return;
    case Rewrite::kOnce8:
      if constexpr (!S::kPeriodic)
        hipLaunchKernelGGL((rewrite_once_k<S, 8>), grid, block, 0, st, n, batch, ld, in, x, ws,
                           ldw);
      return;
    case Rewrite::kTwice4x2:
      hipLaunchKernelGGL((rewrite_twice_k<S, 4, 2>), grid, block, 0, st, n, batch, ld, in, x, ws,
                         ldw);
      return;
    case Rewrite::kTwice4x4:
      hipLaunchKernelGGL((rewrite_twice_k<S, 4, 4>), grid, block, 0, st, n, batch, ld, in, x, ws,
                         ldw);
      return;
    case Rewrite::kTwice8x4:
      hipLaunchKernelGGL((rewrite_twice_k<S, 8, 4>), grid, block, 0, st, n, batch, ld, in, x, ws,
                         ldw);
      return;
  }
}

int launched() { return hipGetLastError() == hipSuccess ? CHX_OK : CHX_EHIP; }

// Every entry of up to five band arrays set to that band's value.
struct FillBands {
  double* band[5];
  double value[5];
};

__global__ __launch_bounds__(kThreads) void fill_bands_k(FillBands fb, int nb, int n, int batch,
                                                         long ld) {
  const long s = (long)blockIdx.x * kThreads + threadIdx.x;
  const int i = blockIdx.y;
  if (s >= batch) return;
#pragma unroll
  for (int k = 0; k < 5; ++k)
    if (k < nb) fb.band[k][(long)i * ld + s] = fb.value[k];
}

}  // namespace chx_vb

using namespace chx_vb;

// Internal launchers for the batched 1D schemes' rewrite mode.
namespace chx {

hipError_t vb_fill_bands(int nb, double* const* bands, const double* values, int n, int batch,
                         long ld, hipStream_t st) {
  if (nb < 1 || nb > 5) return hipErrorInvalidValue;
  FillBands fb{};
  for (int k = 0; k < nb; ++k) {
    fb.band[k] = bands[k];
    fb.value[k] = values[k];
  }
  hipLaunchKernelGGL(fill_bands_k, dim3((unsigned)((batch + kThreads - 1) / kThreads), n),
                     dim3(kThreads), 0, st, fb, nb, n, batch, ld);
  return hipGetLastError();
}

size_t vb_rewrite_ws_bytes(int P, int n, int batch) {
  return P == 2 ? penta_ws_doubles(n, batch, 1, CHX_BATCH_REWRITE) * sizeof(double)
                : tri_ws_doubles(n, batch, 1, CHX_BATCH_REWRITE) * sizeof(double);
}

hipError_t vb_penta_rewrite_periodic(int n, int batch, const double* const* b, long ld, double* x,
                                     double* ws, hipStream_t st) {
  rewrite<Penta<true>>(n, batch, ld, {b[0], b[1], b[2], b[3], b[4], x}, x, ws, st);
  return hipGetLastError();
}

hipError_t vb_tri_rewrite_periodic(int n, int batch, const double* const* b, long ld, double* x,
                                   double* ws, hipStream_t st) {
  rewrite<Tri<true>>(n, batch, ld, {b[0], b[1], b[2], x}, x, ws, st);
  return hipGetLastError();
}

}  // namespace chx

extern "C" {

size_t penta_batch_ws_bytes(int n, int batch, int periodic, int mode) {
  if (n < (periodic ? 5 : 3) || batch < 0 || (mode != CHX_BATCH_FACTOR && mode != CHX_BATCH_REWRITE))
    return 0;
  return penta_ws_doubles(n, batch, periodic != 0, mode) * sizeof(double);
}

size_t tri_batch_ws_bytes(int n, int batch, int periodic, int mode) {
  if (n < (periodic ? 3 : 2) || batch < 0 || (mode != CHX_BATCH_FACTOR && mode != CHX_BATCH_REWRITE))
    return 0;
  return tri_ws_doubles(n, batch, periodic != 0, mode) * sizeof(double);
}

int penta_batch_factor(int n, int batch, int periodic, double* a, double* b, double* c, double* d,
                       double* e, long ld, void* ws, size_t ws_bytes, chx_stream s) {
  int rc = check_common(n, batch, ld, periodic ? 5 : 3, periodic);
  if (rc) return rc;
  if (!a || !b || !c || !d || !e) return CHX_EINVAL;
  rc = check_ws(ws, ws_bytes, penta_ws_doubles(n, batch, periodic, CHX_BATCH_FACTOR));
  if (rc) return rc;
  if (batch == 0) return CHX_OK;
  hipStream_t st = static_cast<hipStream_t>(s);
  double* w = static_cast<double*>(ws);
  if (periodic)
    hipLaunchKernelGGL(penta_batch_factor_k<true>, grid_of(batch), dim3(kThreads), 0, st, n,
                       batch, ld, a, b, c, d, e, w, ws_ld(batch));
  else
    hipLaunchKernelGGL(penta_batch_factor_k<false>, grid_of(batch), dim3(kThreads), 0, st, n,
                       batch, ld, a, b, c, d, e, w, ws_ld(batch));
  return launched();
}

int penta_batch_solve(int n, int batch, int periodic, const double* a, const double* b,
                      const double* c, const double* d, const double* e, long ld, const void* ws,
                      size_t ws_bytes, double* x, chx_stream s) {
  int rc = check_common(n, batch, ld, periodic ? 5 : 3, periodic);
  if (rc) return rc;
  if (!a || !b || !c || !d || !e || !x) return CHX_EINVAL;
  rc = check_ws(ws, ws_bytes, penta_ws_doubles(n, batch, periodic, CHX_BATCH_FACTOR));
  if (rc) return rc;
  if (batch == 0) return CHX_OK;
  hipStream_t st = static_cast<hipStream_t>(s);
  const double* w = static_cast<const double*>(ws);
  if (periodic)
    hipLaunchKernelGGL(penta_batch_solve_k<true>, grid_of(batch), dim3(kThreads), 0, st, n,
                       batch, ld, a, b, c, d, e, w, ws_ld(batch), x);
  else
    hipLaunchKernelGGL(penta_batch_solve_k<false>, grid_of(batch), dim3(kThreads), 0, st, n,
                       batch, ld, a, b, c, d, e, w, ws_ld(batch), x);
  return launched();
}

int penta_batch_rewrite(int n, int batch, int periodic, const double* a, const double* b,
                        const double* c, const double* d, const double* e, long ld, double* x,
                        void* ws, size_t ws_bytes, chx_stream s) {
  int rc = check_common(n, batch, ld, periodic ? 5 : 3, periodic);
  if (rc) return rc;
  if (!a || !b || !c || !d || !e || !x) return CHX_EINVAL;
  rc = check_ws(ws, ws_bytes, penta_ws_doubles(n, batch, periodic, CHX_BATCH_REWRITE));
  if (rc) return rc;
  if (batch == 0) return CHX_OK;
  hipStream_t st = static_cast<hipStream_t>(s);
  double* w = static_cast<double*>(ws);
  if (periodic)
    rewrite<Penta<true>>(n, batch, ld, {a, b, c, d, e, x}, x, w, st);
  else
    rewrite<Penta<false>>(n, batch, ld, {a, b, c, d, e, x}, x, w, st);
  return launched();
}

int tri_batch_factor(int n, int batch, int periodic, double* a, double* b, double* c, long ld,
                     void* ws, size_t ws_bytes, chx_stream s) {
  int rc = check_common(n, batch, ld, periodic ? 3 : 2, periodic);
  if (rc) return rc;
  if (!a || !b || !c) return CHX_EINVAL;
  rc = check_ws(ws, ws_bytes, tri_ws_doubles(n, batch, periodic, CHX_BATCH_FACTOR));
  if (rc) return rc;
  if (batch == 0) return CHX_OK;
  hipStream_t st = static_cast<hipStream_t>(s);
  double* w = static_cast<double*>(ws);
  if (periodic)
    hipLaunchKernelGGL(tri_batch_factor_k<true>, grid_of(batch), dim3(kThreads), 0, st, n, batch,
                       ld, a, b, c, w, ws_ld(batch));
  else
    hipLaunchKernelGGL(tri_batch_factor_k<false>, grid_of(batch), dim3(kThreads), 0, st, n, batch,
                       ld, a, b, c, w, ws_ld(batch));
  return launched();
}

int tri_batch_solve(int n, int batch, int periodic, const double* a, const double* b,
                    const double* c, long ld, const void* ws, size_t ws_bytes, double* x,
                    chx_stream s) {
  int rc = check_common(n, batch, ld, periodic ? 3 : 2, periodic);
  if (rc) return rc;
  if (!a || !b || !c || !x) return CHX_EINVAL;
  rc = check_ws(ws, ws_bytes, tri_ws_doubles(n, batch, periodic, CHX_BATCH_FACTOR));
  if (rc) return rc;
  if (batch == 0) return CHX_OK;
  hipStream_t st = static_cast<hipStream_t>(s);
  const double* w = static_cast<const double*>(ws);
  if (periodic)
    hipLaunchKernelGGL(tri_batch_solve_k<true>, grid_of(batch), dim3(kThreads), 0, st, n, batch,
                       ld, a, b, c, w, ws_ld(batch), x);
  else
    hipLaunchKernelGGL(tri_batch_solve_k<false>, grid_of(batch), dim3(kThreads), 0, st, n, batch,
                       ld, a, b, c, w, ws_ld(batch), x);
  return launched();
}

int tri_batch_rewrite(int n, int batch, int periodic, const double* a, const double* b,
                      const double* c, long ld, double* x, void* ws, size_t ws_bytes,
                      chx_stream s) {
  int rc = check_common(n, batch, ld, periodic ? 3 : 2, periodic);
  if (rc) return rc;
  if (!a || !b || !c || !x) return CHX_EINVAL;
  rc = check_ws(ws, ws_bytes, tri_ws_doubles(n, batch, periodic, CHX_BATCH_REWRITE));
  if (rc) return rc;
  if (batch == 0) return CHX_OK;
  hipStream_t st = static_cast<hipStream_t>(s);
  double* w = static_cast<double*>(ws);
  if (periodic)
    rewrite<Tri<true>>(n, batch, ld, {a, b, c, x}, x, w, st);
  else
    rewrite<Tri<false>>(n, batch, ld, {a, b, c, x}, x, w, st);
  return launched();
}

}  // extern "C"

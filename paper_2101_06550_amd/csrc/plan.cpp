// plan.cpp -- host factorisation tables (see plan.hpp).  Long double
// throughout; the results are rounded once to FP64 and FP32 for the device.
#include "plan.hpp"

#include <algorithm>
#include <cmath>

#include "chx.h"

namespace chx {
namespace {

using LD = long double;

// Entry (i, j) of the non-wrapped band matrix of size n.
LD band_entry(const Band& b, int n, int i, int j) {
  const int o = j - i;
  if (j < 0 || j >= n || i < 0 || i >= n || o < -b.P || o > b.P) return 0;
  return b.coef[o + b.P];
}

// Entry (i, j) of the cyclic matrix of size n: every band offset o whose
// wrapped column (i + o) mod n equals j contributes.
LD cyc_entry(const Band& b, int n, int i, int j) {
  LD v = 0;
  for (int o = -b.P; o <= b.P; ++o)
    if ((((i + o) % n) + n) % n == j) v += b.coef[o + b.P];
  return v;
}

// A = L R with L lower (diagonal alpha, sub-diagonals Lsub) and R unit upper
// (super-diagonals Rsup): the LR factorisation of Ch.4 "Solution of the
// pentadiagonal system" (alpha, beta, epsilon in L; gamma, delta in R) for
// any half bandwidth, and the Thomas pre-factorisation of Ch.5 for P = 1
// (alpha_i = b_i - a_i chat_{i-1}, chat in R).
struct LR {
  int n = 0, P = 0;
  std::vector<LD> alpha, Lsub, Rsup;  // Lsub[i*P + r-1] = L(i,i-r); Rsup[i*P + r-1] = R(i,i+r)
  LD Lg(int i, int j) const {
    const int r = i - j;
    return (r >= 1 && r <= P && j >= 0) ? Lsub[(size_t)i * P + r - 1] : 0;
  }
  LD Rg(int i, int j) const {
    const int r = j - i;
    return (r >= 1 && r <= P && j < n) ? Rsup[(size_t)i * P + r - 1] : 0;
  }
};

int lr_factor(const Band& b, int n, LR* f) {
  const int P = b.P;
  f->n = n;
  f->P = P;
  f->alpha.assign(n, 0);
  f->Lsub.assign((size_t)n * P, 0);
  f->Rsup.assign((size_t)n * P, 0);
  for (int i = 0; i < n; ++i) {
    for (int r = P; r >= 1; --r) {
      const int j = i - r;
      if (j < 0) continue;
      LD v = band_entry(b, n, i, j);
      for (int t = std::max(0, i - P); t < j; ++t) v -= f->Lg(i, t) * f->Rg(t, j);
      f->Lsub[(size_t)i * P + r - 1] = v;
    }
    LD al = band_entry(b, n, i, i);
    for (int t = std::max(0, i - P); t < i; ++t) al -= f->Lg(i, t) * f->Rg(t, i);
    if (!(al > 0) || !std::isfinite((double)al)) return CHX_EPIVOT;
    f->alpha[i] = al;
    for (int r = 1; r <= P; ++r) {
      const int j = i + r;
      if (j >= n) continue;
      LD v = band_entry(b, n, i, j);
      for (int t = std::max(0, j - P); t < i; ++t) v -= f->Lg(i, t) * f->Rg(t, j);
      f->Rsup[(size_t)i * P + r - 1] = v / al;
    }
  }
  return CHX_OK;
}

// x = E^{-1} f  (forward L g = f, back R x = g)
std::vector<LD> lr_solve(const LR& f, const std::vector<LD>& rhs) {
  const int n = f.n, P = f.P;
  std::vector<LD> g(n), x(n);
  for (int i = 0; i < n; ++i) {
    LD v = rhs[i];
    for (int r = 1; r <= P && i - r >= 0; ++r) v -= f.Lg(i, i - r) * g[i - r];
    g[i] = v / f.alpha[i];
  }
  for (int i = n - 1; i >= 0; --i) {
    LD v = g[i];
    for (int r = 1; r <= P && i + r < n; ++r) v -= f.Rg(i, i + r) * x[i + r];
    x[i] = v;
  }
  return x;
}

// q = E^{-T} h  (E^T = R^T L^T: forward with R^T, back with L^T)
std::vector<LD> lr_solve_transposed(const LR& f, const std::vector<LD>& rhs) {
  const int n = f.n, P = f.P;
  std::vector<LD> w(n), q(n);
  for (int i = 0; i < n; ++i) {
    LD v = rhs[i];
    for (int r = 1; r <= P && i - r >= 0; ++r) v -= f.Rg(i - r, i) * w[i - r];
    w[i] = v;
  }
  for (int i = n - 1; i >= 0; --i) {
    LD v = w[i];
    for (int r = 1; r <= P && i + r < n; ++r) v -= f.Lg(i + r, i) * q[i + r];
    q[i] = v / f.alpha[i];
  }
  return q;
}

bool invert_small(const LD* m, int P, LD* inv) {
  if (P == 1) {
    if (!(m[0] != 0)) return false;
    inv[0] = 1 / m[0];
    return std::isfinite((double)inv[0]);
  }
  const LD det = m[0] * m[3] - m[1] * m[2];
  if (!(det != 0) || !std::isfinite((double)det)) return false;
  inv[0] = m[3] / det;
  inv[1] = -m[1] / det;
  inv[2] = -m[2] / det;
  inv[3] = m[0] / det;
  return true;
}

// Bordering of the last P unknowns of the cyclic system (Navon, Ch.4):
// E (leading block), k, h^T, C22 read off the periodic pattern.
struct Bordered {
  LR E;
  std::vector<std::vector<LD>> Z, q;  // Z[a] = E^{-1} k[:,a], q[a] = E^{-T} h[a,:]
  LD minv[4] = {1, 0, 0, 1};
};

int bordered_factor(const Band& b, int n, Bordered* out) {
  const int P = b.P, mi = n - P;
  Band eb = b;
  int rc = lr_factor(eb, mi, &out->E);
  if (rc) return rc;
  out->Z.assign(P, std::vector<LD>(mi));
  out->q.assign(P, std::vector<LD>(mi));
  // the couplings are a few entries at the ends: band offset o of row i meets
  // column (i + o) mod n
  auto ring = [&](int i) { return ((i % n) + n) % n; };
  std::vector<std::vector<LD>> hrow(P, std::vector<LD>(mi, 0));
  for (int a = 0; a < P; ++a) {
    std::vector<LD> kcol(mi, 0);
    for (int o = -P; o <= P; ++o) {
      const int i = ring(mi + a - o), j = ring(mi + a + o);
      if (i < mi) kcol[i] += b.coef[o + P];
      if (j < mi) hrow[a][j] += b.coef[o + P];
    }
    out->Z[a] = lr_solve(out->E, kcol);
    out->q[a] = lr_solve_transposed(out->E, hrow[a]);
  }
  LD M[4] = {0, 0, 0, 0};
  for (int a = 0; a < P; ++a)
    for (int c = 0; c < P; ++c) {
      LD v = cyc_entry(b, n, mi + a, mi + c);
      for (int i = 0; i < mi; ++i)
        if (hrow[a][i] != 0) v -= hrow[a][i] * out->Z[c][i];
      M[a * P + c] = v;
    }
  LD inv[4];
  if (!invert_small(M, P, inv)) return CHX_EPIVOT;
  for (int t = 0; t < P * P; ++t) out->minv[t] = inv[t];
  return CHX_OK;
}

std::vector<LD> bordered_solve(const Band& b, int n, const Bordered& B,
                               const std::vector<LD>& f) {
  const int P = b.P, mi = n - P;
  std::vector<LD> fh(f.begin(), f.begin() + mi);
  LD r[2] = {0, 0}, t[2] = {0, 0};
  for (int a = 0; a < P; ++a) {
    LD s = 0;
    for (int i = 0; i < mi; ++i) s += B.q[a][i] * fh[i];
    r[a] = f[mi + a] - s;
  }
  for (int a = 0; a < P; ++a)
    for (int c = 0; c < P; ++c) t[a] += B.minv[a * P + c] * r[c];
  std::vector<LD> y = lr_solve(B.E, fh);
  std::vector<LD> x(n);
  for (int i = 0; i < mi; ++i) {
    LD v = y[i];
    for (int a = 0; a < P; ++a) v -= B.Z[a][i] * t[a];
    x[i] = v;
  }
  for (int a = 0; a < P; ++a) x[mi + a] = t[a];
  return x;
}

void fill_rec(const LR& E, int i, double* rec) {
  rec[0] = (double)(1.0L / E.alpha[i]);
  rec[1] = (double)E.Lg(i, i - 1);
  rec[2] = (double)E.Rg(i, i + 1);
  rec[3] = (E.P >= 2) ? (double)E.Rg(i, i + 2) : 0.0;
}

}  // namespace

struct CyclicFactor::Impl {
  Bordered B;
  bool have_g = false;
  std::vector<LD> g;
};
CyclicFactor::CyclicFactor() : impl(new Impl) {}
CyclicFactor::~CyclicFactor() { delete impl; }

int CyclicFactor::make(const Band& b, int size) {
  band = b;
  n = size;
  return bordered_factor(b, size, &impl->B);
}

const std::vector<long double>& CyclicFactor::inverse_column() {
  if (!impl->have_g) {
    std::vector<LD> e0(n, 0);
    e0[0] = 1;
    impl->g = bordered_solve(band, n, impl->B, e0);
    impl->have_g = true;
  }
  return impl->g;
}

int build_whole(const Band& band, int n, WholeTables* out, CyclicFactor* cyc) {
  const int P = band.P;
  out->n = n;
  out->P = P;
  if (!band.periodic) {
    LR E;
    int rc = lr_factor(band, n, &E);
    if (rc) return rc;
    out->mi = n;
    out->rec.assign((size_t)n * kRec, 0.0);
    for (int i = 0; i < n; ++i) fill_rec(E, i, &out->rec[(size_t)i * kRec]);
  } else {
    CyclicFactor own;
    if (!cyc) {
      int rc = own.make(band, n);
      if (rc) return rc;
      cyc = &own;
    }
    const Bordered& B = cyc->impl->B;
    const int mi = n - P;
    out->mi = mi;
    out->rec.assign((size_t)mi * kRec, 0.0);
    for (int i = 0; i < mi; ++i) {
      double* r = &out->rec[(size_t)i * kRec];
      fill_rec(B.E, i, r);
      for (int a = 0; a < P; ++a) {
        r[4 + a] = (double)B.q[a][i];
        r[6 + a] = (double)B.Z[a][i];
      }
    }
    for (int t = 0; t < 4; ++t) out->minv[t] = 0.0;
    for (int a = 0; a < P; ++a)
      for (int c = 0; c < P; ++c) out->minv[a * 2 + c] = (double)B.minv[a * P + c];
  }
  out->rec32.assign(out->rec.begin(), out->rec.end());
  for (int t = 0; t < 4; ++t) out->minv32[t] = (float)out->minv[t];
  return CHX_OK;
}

int build_chunk(const Band& band, int n, int m, ChunkTables* out, CyclicFactor* cyc) {
  const int P = band.P;
  if (!band.periodic || m < 3 * P || n % m != 0) return CHX_EINVAL;
  const int S = n / m, mi = m - P;
  out->n = n; out->P = P; out->m = m; out->S = S; out->mi = mi;

  // Interior block of one chunk and its spike vectors.
  LR E;
  int rc = lr_factor(band, mi, &E);
  if (rc) return rc;
  out->rec.assign((size_t)mi * kRec, 0.0);
  for (int a = 0; a < P; ++a) {
    std::vector<LD> kl(mi, 0), kr(mi, 0);
    for (int p = 0; p < mi; ++p) {
      const int ol = (a - P) - p;   // previous chunk's separator a sits at -P + a
      if (ol >= -P && ol <= P) kl[p] = band.coef[ol + P];
      const int orr = mi + a - p;   // this chunk's separator a sits at mi + a
      if (orr >= -P && orr <= P) kr[p] = band.coef[orr + P];
    }
    std::vector<LD> zl = lr_solve(E, kl), zr = lr_solve(E, kr);
    for (int p = 0; p < mi; ++p) {
      out->rec[(size_t)p * kRec + 4 + a] = (double)zl[p];
      out->rec[(size_t)p * kRec + 6 + a] = (double)zr[p];
    }
  }
  for (int p = 0; p < mi; ++p) fill_rec(E, p, &out->rec[(size_t)p * kRec]);

  // Reduced system: the separator-separator block of the circulant A^{-1}.
  CyclicFactor own;
  if (!cyc) {
    rc = own.make(band, n);
    if (rc) return rc;
    cyc = &own;
  }
  const std::vector<LD>& g = cyc->inverse_column();
  auto blk = [&](int d, int a, int c) -> LD {
    long long idx = (long long)(-(long long)d * m + a - c);
    idx %= n;
    if (idx < 0) idx += n;
    return g[(size_t)idx];
  };
  std::vector<LD> nb(S, 0);
  for (int d = 0; d < S; ++d)
    for (int a = 0; a < P; ++a)
      for (int c = 0; c < P; ++c) nb[d] = std::max(nb[d], std::fabs(blk(d, a, c)));
  const LD thresh = std::ldexp((LD)1, -60) * nb[0];
  int W = 0;
  for (;; ++W) {
    LD tail = 0;
    for (int d = 0; d < S; ++d) {
      const int dist = std::min(d, S - d);
      if (dist > W) tail += nb[d];
    }
    if (tail <= thresh || 2 * W + 1 >= S) break;
  }
  if (2 * W + 1 >= S) {
    out->dlo = -((S - 1) / 2);
    out->dcount = S;
  } else {
    out->dlo = -W;
    out->dcount = 2 * W + 1;
  }
  out->max_dropped = 0.0;
  for (int d = 0; d < S; ++d) {
    const int dist = std::min(d, S - d);
    if (out->dcount < S && dist > W) out->max_dropped = std::max(out->max_dropped, (double)nb[d]);
  }
  out->blocks.assign((size_t)out->dcount * 4, 0.0);
  for (int t = 0; t < out->dcount; ++t) {
    const int d = out->dlo + t;
    for (int a = 0; a < P; ++a)
      for (int c = 0; c < P; ++c) out->blocks[(size_t)t * 4 + a * 2 + c] = (double)blk(d, a, c);
  }
  out->rec32.assign(out->rec.begin(), out->rec.end());
  out->blocks32.assign(out->blocks.begin(), out->blocks.end());
  return CHX_OK;
}

bool ragged_split(int P, int n, int M, int* m, int* r, int* S) {
  const int rmin = 3 * P;
  if (n < rmin) return false;
  for (int s = (n + M - 1) / M; s * rmin <= n; ++s)
    for (int q = std::min(M, n); q >= rmin; --q) {
      const int rem = n - (s - 1) * q;
      if (rem > q) break;
      if (rem < rmin) continue;
      *m = q;
      *r = rem;
      *S = s;
      return true;
    }
  return false;
}

int build_ragged(const Band& band, int n, int M, RaggedTables* out, CyclicFactor* cyc) {
  const int P = band.P;
  int m, r, S;
  if (!band.periodic || !ragged_split(P, n, M, &m, &r, &S)) return CHX_EINVAL;
  const int mi = m - P;
  out->n = n; out->P = P; out->M = M; out->m = m; out->r = r; out->S = S;

  LR E;
  int rc = lr_factor(band, mi, &E);
  if (rc) return rc;
  // LR factors and, for an interior of len unknowns, its spike vectors
  auto fill = [&](int len, std::vector<double>* rec) {
    rec->assign((size_t)(M - P) * kRec, 0.0);
    LR El;
    if (lr_factor(band, len, &El)) return;  // a leading block of E: its pivots are E's
    for (int p = 0; p < len; ++p) fill_rec(El, p, &(*rec)[(size_t)p * kRec]);
    for (int a = 0; a < P; ++a) {
      std::vector<LD> kl(len, 0), kr(len, 0);
      for (int p = 0; p < len; ++p) {
        const int ol = (a - P) - p, orr = len + a - p;
        if (ol >= -P && ol <= P) kl[p] = band.coef[ol + P];
        if (orr >= -P && orr <= P) kr[p] = band.coef[orr + P];
      }
      const std::vector<LD> zl = lr_solve(El, kl), zr = lr_solve(El, kr);
      for (int p = 0; p < len; ++p) {
        (*rec)[(size_t)p * kRec + 4 + a] = (double)zl[p];
        (*rec)[(size_t)p * kRec + 6 + a] = (double)zr[p];
      }
    }
  };
  fill(mi, &out->rec);
  fill(r - P, &out->recl);

  CyclicFactor own;
  if (!cyc) {
    rc = own.make(band, n);
    if (rc) return rc;
    cyc = &own;
  }
  const std::vector<LD>& g = cyc->inverse_column();
  auto blk = [&](int fam, int d, int a, int c) -> LD {
    const int shift = fam == 0 ? 0 : fam == 1 ? m - r : r - m;
    long long idx = (long long)a - c - ((long long)d * m + shift);
    idx %= n;
    if (idx < 0) idx += n;
    return g[(size_t)idx];
  };
  // the window: every chunk, or the fewest offsets on either side beyond
  // which the blocks of all families total at most 2^-60 of the largest
  auto norm = [&](int d) {
    LD v = 0;
    for (int fam = 0; fam < 3; ++fam)
      for (int a = 0; a < P; ++a)
        for (int c = 0; c < P; ++c) v = std::max(v, std::fabs(blk(fam, d, a, c)));
    return v;
  };
  std::vector<LD> nb(S);  // by distance in chunks along the nearer way
  for (int w = 0; w < S; ++w) nb[w] = std::max(norm(w), norm(-w));
  const LD thresh = std::ldexp((LD)1, -60) * nb[0];
  int W = 0;
  for (;; ++W) {
    LD tail = 0;
    for (int w = W + 1; w <= S / 2; ++w) tail += 2 * nb[w];
    if (tail <= thresh || 2 * W + 1 >= S) break;
  }
  if (2 * W + 1 >= S) {
    out->dlo = -((S - 1) / 2);
    out->dcount = S;
  } else {
    out->dlo = -W;
    out->dcount = 2 * W + 1;
  }
  out->blocks.assign((size_t)3 * out->dcount * 4, 0.0);
  for (int fam = 0; fam < 3; ++fam)
    for (int t = 0; t < out->dcount; ++t)
      for (int a = 0; a < P; ++a)
        for (int c = 0; c < P; ++c)
          out->blocks[((size_t)fam * out->dcount + t) * 4 + a * 2 + c] =
              (double)blk(fam, out->dlo + t, a, c);
  return CHX_OK;
}

}  // namespace chx

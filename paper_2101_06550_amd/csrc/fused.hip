// fused.hip -- interleaved cyclic solves with one workgroup per group of
// systems: every chunk of L systems is held in the registers of one
// workgroup, so a batch is solved in one pass over memory (16 bytes per
// unknown) and one launch, and a batched 1D scheme takes all the steps of a
// call without going back to memory.
//
// Bound by HBM: 131072 cyclic pentadiagonal systems of 1024 take 0.437 ms, 4.9
// TB/s of the 16 bytes per unknown (0.620 ms in three passes that move 26.5);
// what is left against a copy's 6.5 TB/s is the access pattern (rows 1 MB
// apart, 256 bytes of each per workgroup: 131088 systems, whose rows fall on
// other channels, run 6 % faster) and the load and store phases of the one or
// two workgroups that a CU holds.  262144 1D Cahn-Hilliard systems of 256, four
// steps in a call: 0.30 ms (1.21 ms with a pass over memory per step); 131072
// systems of 1000, an odd length: 0.447 ms.
//
// Thread (c, k) = (tid % L, tid / L) owns chunk k of system c: it loads the
// chunk, sweeps its interior, publishes the coupling part that the previous
// chunk's separators need, forms its reduced right-hand side, publishes that,
// sums its separators over the block window and corrects its interior with
// its own and the previous chunk's separators.  The sums run in the order of
// the separator kernels in solve.hip.
//
// RAG: any system length, in chunks of m <= M unknowns with a last one of r
// (see RaggedTables).  A chunk's unknowns lie at positions 0 .. len - 1 of
// the registers; positions past its interior are masked to zero between the
// forward and the back sweep, which makes the back sweep start from the
// chunk's own last row.
#include <hip/hip_runtime.h>

#include "common.hpp"
#include "launch.hpp"

namespace chx {

namespace {

constexpr int M = kChunk;

// Family of the reduced block that takes chunk j (unwrapped) to chunk k.
__device__ __forceinline__ int rag_family(int k, int j, int S) {
  if (k == S - 1) return j <= S - 2 ? 1 : 0;
  return j <= -2 ? 1 : (j >= S - 1 ? 2 : 0);
}

// The scheme's right-hand side at the middle of five consecutive values
// (0 Crank-Nicolson hyperdiffusion, 1 Crank-Nicolson diffusion, 2 1D
// Cahn-Hilliard): the expressions of the stepwise kernels.
template <int KIND>
__device__ __forceinline__ double rhs1d(double ll, double l, double x, double r, double rr,
                                        double s, double al) {
  if (KIND == 0) return -s * ll + 4.0 * s * l + (1.0 - 6.0 * s) * x + 4.0 * s * r - s * rr;
  if (KIND == 1) return s * l + (1.0 - 2.0 * s) * x + s * r;
  const double ml = l * l * l - l, mc = x * x * x - x, mr = r * r * r - r;
  return x + al * (ml - 2.0 * mc + mr);
}

// A plan table for scalar loads (see TabD), opaque to the compiler: the
// tables are read again where they are used, in every step, instead of being
// kept in scalar registers that they overflow.
__device__ __forceinline__ TabD table(const double* p) {
  TabD t = (TabD)p;
  asm volatile("" : "+s"(t));
  return t;
}

// Masks of the ragged chunks compare a position with a length: the copy keeps
// the compiler from holding every mask of a chunk for its next use.
__device__ __forceinline__ int fresh(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// Sweep of a chunk whose interior is f[0 .. li): y in place, zero beyond; t1
// and t2 the interior's last two unknowns (y[li - 1], y[li - 2]).
template <int P>
__device__ __forceinline__ void ragged_sweep(double (&f)[M], int li, TabD rec, double eps,
                                             double& t1, double& t2) {
  constexpr int MI = M - P;
#pragma unroll
  for (int p = 0; p < MI; ++p) {
    double v = f[p];
    if (P == 2 && p >= 2) v = v - eps * f[p - 2];
    if (p >= 1) v = v - rec[p * 8 + 1] * f[p - 1];
    f[p] = v * rec[p * 8 + 0];
  }
  li = fresh(li);
#pragma unroll
  for (int p = MI - 1; p >= 0; --p) {
    double v = p < li ? f[p] : 0.0;
    if (P == 2 && p + 2 < MI) v = v - rec[p * 8 + 3] * f[p + 2];
    if (p + 1 < MI) v = v - rec[p * 8 + 2] * f[p + 1];
    f[p] = v;
    t1 = p == li - 1 ? v : t1;
    if (P == 2) t2 = p == li - 2 ? v : t2;
  }
}

// pa: the separators' reduced right-hand sides but for the next chunk's part;
// pb: this chunk's part for the previous chunk's separators (chunk_parts with
// the interior's last unknowns given).
template <int P>
__device__ __forceinline__ void ragged_parts(const double (&f)[M], const double (&fs)[P],
                                             double t1, double t2, const BandT<double>& bd,
                                             double (&pa)[P], double (&pb)[P]) {
  if constexpr (P == 2) {
    pa[0] = (fs[0] - bd.c[0] * t2) - bd.c[1] * t1;
    pa[1] = fs[1] - bd.c[0] * t1;
    pb[0] = bd.c[4] * f[0];
    pb[1] = bd.c[3] * f[0] + bd.c[4] * f[1];
  } else {
    pa[0] = fs[0] - bd.c[0] * t1;
    pb[0] = bd.c[2] * f[0];
  }
}

// x = y - Zl sp - Zr so in the interior.  A wave that holds last chunks runs both tables, each chunk's separators masked to
// zero for the other's.
template <int P>
__device__ __forceinline__ void ragged_correct(double (&f)[M], bool last, TabD rec, TabD recl,
                                               const double (&sp)[P], const double (&so)[P]) {
  constexpr int MI = M - P;
  auto correct = [&](TabD z, bool mine) {
    double u[P], w[P];
#pragma unroll
    for (int a = 0; a < P; ++a) {
      u[a] = mine ? sp[a] : 0.0;
      w[a] = mine ? so[a] : 0.0;
    }
#pragma unroll
    for (int p = 0; p < MI; ++p) {
      double v = f[p];
#pragma unroll
      for (int a = 0; a < P; ++a) v = v - z[p * 8 + 4 + a] * u[a] - z[p * 8 + 6 + a] * w[a];
      f[p] = v;
    }
  };
  if (__any(!last)) correct(rec, !last);
  if (__any(last)) correct(recl, last);
}

// LINES: every row of a tile is whole 128-byte lines that no other workgroup
// touches, so they stream past the caches in launch order.  Otherwise two
// neighbouring tiles share a line in every row: they go to one XCD (workgroups
// go to the 8 XCDs round robin) one after the other, and through its L2, where
// the halves meet (60001 systems of 1024: 595 us streamed, 297 us through the
// caches in launch order, 216 us this way; 131072 systems: 434 us streamed,
// 473 us this way).
template <bool LINES>
__device__ __forceinline__ unsigned tile_of(unsigned b, unsigned nb) {
  if constexpr (LINES) return b;
  const unsigned per = nb >> 3;
  return b < (per << 3) ? (b & 7) * per + (b >> 3) : b;
}
template <bool LINES>
__device__ __forceinline__ double load(const double* p) {
  if constexpr (LINES) return __builtin_nontemporal_load(p);
  return *p;
}
template <bool LINES>
__device__ __forceinline__ void store(double* p, double v) {
  if constexpr (LINES) __builtin_nontemporal_store(v, p);
  else *p = v;
}

struct FusedArgs {
  double* x;
  long ld;
  int batch, S, m, r, dlo, dcount;
  const double *rec, *recl, *blocks;
  BandT<double> bd;
  int nsteps;
  double s, al;
};

}  // namespace

// KIND -1: one solve of the right-hand sides in x; KIND 0 .. 2: nsteps steps of
// a 1D scheme from the state in x.  In place: a workgroup owns its systems and
// loads all of them before it stores.
template <int P, int L, bool RAG, int KIND, bool LINES>
__global__ __launch_bounds__(1024) void il_fused(const FusedArgs A) {
  constexpr int MI = M - P;
  extern __shared__ double sm[];
  const int S = A.S;
  const int c = threadIdx.x % L, kt = threadIdx.x / L;
  const bool active = kt < S;
  const int k = active ? kt : S - 1;
  const long sys = (long)tile_of<LINES>(blockIdx.x, gridDim.x) * L + c;
  const bool sv = active && sys < A.batch;
  const long sl = sys < A.batch ? sys : (long)A.batch - 1;
  double* const part = sm;              // [P][S][L]: parts for the previous chunk, then separators
  double* const rho = sm + P * S * L;   // [P][S][L]: reduced right-hand sides, then first unknowns
  const int me = k * L + c;             // this thread's element of a plane
  const int nx = (k + 1 == S ? 0 : k + 1) * L + c, pv = (k == 0 ? S - 1 : k - 1) * L + c;
  const int plane = S * L;
  const bool last = RAG && k == S - 1;
  const int len = RAG ? (last ? A.r : A.m) : M;
  const int li = len - P;  // interior length

  double f[M], fs[P];  // the chunk; its separators
  const long row0 = (long)k * (RAG ? A.m : M);
  {
    const double* p0 = A.x + row0 * A.ld + sl;
    if constexpr (RAG) {  // positions past the chunk re-read its last unknown
#pragma unroll
      for (int a = 0; a < P; ++a) fs[a] = load<LINES>(p0 + (long)(li + a) * A.ld);
#pragma unroll
      for (int p = 0; p < M; ++p) {
        f[p] = load<LINES>(p0);
        p0 += p + 1 < len ? A.ld : 0;
      }
    } else {
#pragma unroll
      for (int p = 0; p < M; ++p) f[p] = load<LINES>(p0 + (long)p * A.ld);
#pragma unroll
      for (int a = 0; a < P; ++a) fs[a] = f[MI + a];
    }
  }
  double sp[P];  // the previous chunk's separators
  if constexpr (KIND >= 0) {
    // the state's chunk ends: the previous chunk's separators (registers),
    // the next chunk's first P unknowns (published in rho)
    if (active) {
#pragma unroll
      for (int a = 0; a < P; ++a) {
        part[a * plane + me] = fs[a];
        rho[a * plane + me] = f[a];
      }
    }
    __syncthreads();
#pragma unroll
    for (int a = 0; a < P; ++a) sp[a] = part[a * plane + pv];
    __syncthreads();
  }

  for (int step = 0; step < (KIND >= 0 ? A.nsteps : 1); ++step) {
    if constexpr (KIND >= 0) {
      double nb[2] = {rho[nx], P == 2 ? rho[(P - 1) * plane + nx] : 0.0};
      double ll = P == 2 ? sp[0] : 0.0, l = sp[P - 1], x = f[0];
      double r1 = RAG ? (1 < len ? f[1] : nb[0]) : f[1];
#pragma unroll
      for (int p = 0; p < M; ++p) {
        double r2;  // position p + 2 of the chunk, or the next chunk's first unknowns
        if constexpr (RAG) {
          const double in = p + 2 < M ? f[p + 2 < M ? p + 2 : 0] : 0.0;
          r2 = p + 2 < len ? in : (p + 2 == len ? nb[0] : nb[1]);
        } else {
          r2 = p + 2 < M ? f[p + 2 < M ? p + 2 : 0] : nb[p + 2 - M < 1 ? 0 : 1];
        }
        f[p] = rhs1d<KIND < 0 ? 0 : KIND>(ll, l, x, r1, r2, A.s, A.al);
        if constexpr (RAG) {
#pragma unroll
          for (int a = 0; a < P; ++a) {
            fs[a] = p == li + a ? f[p] : fs[a];
            asm volatile("" : "+v"(fs[a]));
          }
        }
        ll = l;
        l = x;
        x = r1;
        r1 = r2;
      }
    }
    // separator right-hand sides, and the sweep of the interior
    const TabD rec = table(A.rec);
    double t1 = 0, t2 = 0;  // the interior's last two unknowns
    const double eps = A.bd.c[0];
    if constexpr (RAG) {
      ragged_sweep<P>(f, li, rec, eps, t1, t2);
    } else {
#pragma unroll
      for (int a = 0; a < P; ++a) fs[a] = f[MI + a];
      chunk_sweep<P, M, double, TabD>(f, rec, eps);
      t1 = f[MI - 1];
      t2 = f[MI - 2];
    }
    double pa[P], pb[P];
    ragged_parts<P>(f, fs, t1, t2, A.bd, pa, pb);
    if (active) {
#pragma unroll
      for (int a = 0; a < P; ++a) part[a * plane + me] = pb[a];
    }
    __syncthreads();
#pragma unroll
    for (int a = 0; a < P; ++a) pa[a] -= part[a * plane + nx];
    if (active) {
#pragma unroll
      for (int a = 0; a < P; ++a) rho[a * plane + me] = pa[a];
    }
    __syncthreads();
    double so[P];
#pragma unroll
    for (int a = 0; a < P; ++a) so[a] = 0;
    int j = k + A.dlo;
    j += j < 0 ? S : 0;
    if (j < 0) j += S;
    if (j >= S) j -= S;
    for (int t = 0; t < A.dcount; ++t) {
      double w[P];
#pragma unroll
      for (int a = 0; a < P; ++a) w[a] = rho[a * plane + j * L + c];
      auto add = [&](auto B) {
#pragma unroll
        for (int a = 0; a < P; ++a)
#pragma unroll
          for (int b = 0; b < P; ++b) so[a] = so[a] + B[a * 2 + b] * w[b];
      };
      if constexpr (RAG)
        add(A.blocks + 4 * (A.dcount * rag_family(k, k + A.dlo + t, S) + t));
      else
        add((TabD)A.blocks + 4 * t);
      j = j + 1 == S ? 0 : j + 1;
    }
    if (active) {
#pragma unroll
      for (int a = 0; a < P; ++a) part[a * plane + me] = so[a];
    }
    __syncthreads();
#pragma unroll
    for (int a = 0; a < P; ++a) sp[a] = part[a * plane + pv];
    if constexpr (RAG) {
      ragged_correct<P>(f, last, table(A.rec), table(A.recl), sp, so);
      if constexpr (KIND >= 0) {  // the state's chunk again: unknowns 0 .. len - 1
        const int lj = fresh(li);
#pragma unroll
        for (int p = 0; p < M; ++p)
#pragma unroll
          for (int a = 0; a < P; ++a) f[p] = p == lj + a ? so[a] : f[p];
      }
#pragma unroll
      for (int a = 0; a < P; ++a) fs[a] = so[a];
    } else {
      chunk_correct<P, M, double, TabD>(f, table(A.rec), sp, so);
    }
    if constexpr (KIND >= 0) {  // the next step's neighbours
      if (active) {
#pragma unroll
        for (int a = 0; a < P; ++a) rho[a * plane + me] = f[a];
      }
      __syncthreads();
    }
  }
  if (sv) {
    double* p0 = A.x + row0 * A.ld + sl;
    asm volatile("" : "+v"(p0));  // the rows' addresses again, not kept since the loads
    if constexpr (RAG) {
      const int lj = fresh(li);
#pragma unroll
      for (int p = 0; p < MI; ++p)
        if (p < lj) store<LINES>(p0 + (long)p * A.ld, f[p]);
#pragma unroll
      for (int a = 0; a < P; ++a)
        store<LINES>(p0 + (long)(lj + a) * A.ld, fs[a]);
    } else {
#pragma unroll
      for (int p = 0; p < M; ++p) store<LINES>(p0 + (long)p * A.ld, f[p]);
    }
  }
}

// Contiguous rows of any length n: a workgroup takes R rows of S chunks, one
// thread per chunk.  The rows go through LDS in both directions (slot e + e /
// 32 of element e of the group, which spreads the threads' chunks over the
// banks), so memory sees whole lines; two accesses per unknown.
// Bound by HBM and, at two workgroups of LDS per CU, by how much of its
// latency they cover: 20000 rows of 1000 points 73 us, 4.4 TB/s (79 us with a
// thread's 32 loads issued 8 at a time; one thread per row: 800 us, every lane
// on a line of its own, 32 waves of them in all).
template <int P>
__global__ __launch_bounds__(256) void rows_ragged(double* x, long ld, int rows, int n, int R,
                                                   const FusedArgs A) {
  extern __shared__ double sm[];
  const int S = A.S, T = blockDim.x, t = threadIdx.x;
  const long row0 = (long)blockIdx.x * R;
  const int nr = rows - row0 < R ? (int)(rows - row0) : R;
  const int nel = nr * n;
  double* const part = sm;           // [P][T]
  double* const rho = sm + P * T;    // [P][T]
  double* const tile = sm + 2 * P * T;
  const int rt = t / S;
  const bool active = rt < nr;
  const int r = active ? rt : nr - 1, k = active ? t - rt * S : S - 1;
  const bool last = k == S - 1;
  const int len = last ? A.r : A.m, li = len - P;
  const bool dense = ld == n;
  double* const xg = x + row0 * ld;
  auto at = [&](int e) -> long { return dense ? (long)e : (long)(e / n) * ld + e % n; };
  constexpr int U = M;  // every load of a thread in flight
  for (int e0 = t; e0 < nel; e0 += U * T) {
    double v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = e0 + u * T;
      v[u] = __builtin_nontemporal_load(xg + at(e < nel ? e : nel - 1));
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = e0 + u * T;
      if (e < nel) tile[e + (e >> 5)] = v[u];
    }
  }
  __syncthreads();
  double f[M];
  const int e0 = r * n + k * A.m;
#pragma unroll
  for (int p = 0; p < M; ++p) {
    const int e = e0 + (p < len ? p : len - 1);  // past the chunk: its last unknown
    f[p] = tile[e + (e >> 5)];
  }
  double fs[P], t1 = 0, t2 = 0, pa[P], pb[P];
#pragma unroll
  for (int a = 0; a < P; ++a) fs[a] = tile[e0 + li + a + ((e0 + li + a) >> 5)];
  ragged_sweep<P>(f, li, table(A.rec), A.bd.c[0], t1, t2);
  ragged_parts<P>(f, fs, t1, t2, A.bd, pa, pb);
  const int rs = r * S, me = rs + k;
  const int nx = rs + (k + 1 == S ? 0 : k + 1), pv = rs + (k == 0 ? S - 1 : k - 1);
  if (active) {
#pragma unroll
    for (int a = 0; a < P; ++a) part[a * T + me] = pb[a];
  }
  __syncthreads();
#pragma unroll
  for (int a = 0; a < P; ++a) pa[a] -= part[a * T + nx];
  if (active) {
#pragma unroll
    for (int a = 0; a < P; ++a) rho[a * T + me] = pa[a];
  }
  __syncthreads();
  double so[P], sp[P];
#pragma unroll
  for (int a = 0; a < P; ++a) so[a] = 0;
  int j = k + A.dlo;
  j += j < 0 ? S : 0;
  for (int q = 0; q < A.dcount; ++q) {
    double w[P];
#pragma unroll
    for (int a = 0; a < P; ++a) w[a] = rho[a * T + rs + j];
    const double* B = A.blocks + 4 * (A.dcount * rag_family(k, k + A.dlo + q, S) + q);
#pragma unroll
    for (int a = 0; a < P; ++a)
#pragma unroll
      for (int b = 0; b < P; ++b) so[a] = so[a] + B[a * 2 + b] * w[b];
    j = j + 1 == S ? 0 : j + 1;
  }
  if (active) {
#pragma unroll
    for (int a = 0; a < P; ++a) part[a * T + me] = so[a];
  }
  __syncthreads();
#pragma unroll
  for (int a = 0; a < P; ++a) sp[a] = part[a * T + pv];
  ragged_correct<P>(f, last, table(A.rec), table(A.recl), sp, so);
  if (active) {
    const int lj = fresh(li);
#pragma unroll
    for (int p = 0; p < M - P; ++p)
      if (p < lj) tile[e0 + p + ((e0 + p) >> 5)] = f[p];
#pragma unroll
    for (int a = 0; a < P; ++a) tile[e0 + lj + a + ((e0 + lj + a) >> 5)] = so[a];
  }
  __syncthreads();
  for (int e = t; e < nel; e += T) __builtin_nontemporal_store(tile[e + (e >> 5)], xg + at(e));
}

// Systems per workgroup (16, 32 or 64: whole lines of every row), or 0 where
// 16 systems need more than 1024 threads.  More systems make longer rows of a
// tile and fewer workgroups: 64 where that leaves two workgroups of 512
// threads per CU (524288 systems of 256: 395 us, 419 with 32, 455 with 16), 32
// up to 1024 threads (131072 systems of 1024: 444 us, 457 with 16; 512 points:
// 395 us, 409 with 64), as long as there are two workgroups for every CU
// (1024 systems of 1024: 9.4 us with 16, 12.3 with 32).
int il_fused_systems(int S, int batch) {
  if (S * 16 > 1024) return 0;
  if (S * 64 <= 512 && batch >= 64 * 512) return 64;
  return S * 32 <= 1024 && batch >= 32 * 512 ? 32 : 16;
}

template <int P, int L, bool RAG, int KIND>
static hipError_t fused_launch(const FusedArgs& a, hipStream_t st) {
  const dim3 grid((unsigned)((a.batch + L - 1) / L)), block(((L * a.S + 63) / 64) * 64);
  const size_t lds = (size_t)2 * P * a.S * L * sizeof(double);
  if (a.ld % 16 == 0 && (reinterpret_cast<uintptr_t>(a.x) & 127) == 0)
    hipLaunchKernelGGL((il_fused<P, L, RAG, KIND, true>), grid, block, lds, st, a);
  else
    hipLaunchKernelGGL((il_fused<P, L, RAG, KIND, false>), grid, block, lds, st, a);
  return hipGetLastError();
}

template <int P, int L, bool RAG>
static hipError_t fused_kind(int kind, const FusedArgs& a, hipStream_t st) {
  if (kind < 0) return fused_launch<P, L, RAG, -1>(a, st);
  if constexpr (P == 1) return fused_launch<P, L, RAG, 1>(a, st);
  else if (kind == 0) return fused_launch<P, L, RAG, 0>(a, st);
  else return fused_launch<P, L, RAG, 2>(a, st);
}

template <int P, bool RAG>
static hipError_t fused_any(int kind, const FusedArgs& a, hipStream_t st) {
  switch (il_fused_systems(a.S, a.batch)) {
    case 64: return fused_kind<P, 64, RAG>(kind, a, st);
    case 32: return fused_kind<P, 32, RAG>(kind, a, st);
    case 16: return fused_kind<P, 16, RAG>(kind, a, st);
    default: return hipErrorInvalidValue;
  }
}

// The kernel arguments of either plan (a chunk plan is the even split).
template <class Plan>
static FusedArgs fused_args(const Plan& c, int m, int r, const double* recl, double* x, long ld,
                            int batch) {
  FusedArgs a{};
  a.x = x;
  a.ld = ld;
  a.batch = batch;
  a.nsteps = 1;
  a.S = c.S;
  a.m = m;
  a.r = r;
  a.dlo = c.dlo;
  a.dcount = c.dcount;
  a.rec = c.rec;
  a.recl = recl;
  a.blocks = c.blocks;
  for (int i = 0; i < 5; ++i) a.bd.c[i] = c.coef[i];
  return a;
}

hipError_t launch_il_fused(const DevChunk& c, int kind, double* x, long ld, int batch, int nsteps,
                           double s, double al, hipStream_t st) {
  FusedArgs a = fused_args(c, M, M, c.rec, x, ld, batch);
  a.nsteps = nsteps;
  a.s = s;
  a.al = al;
  return c.P == 2 ? fused_any<2, false>(kind, a, st) : fused_any<1, false>(kind, a, st);
}

hipError_t launch_il_fused(const DevRagged& c, int kind, double* x, long ld, int batch, int nsteps,
                           double s, double al, hipStream_t st) {
  FusedArgs a = fused_args(c, c.m, c.r, c.recl, x, ld, batch);
  a.nsteps = nsteps;
  a.s = s;
  a.al = al;
  return c.P == 2 ? fused_any<2, true>(kind, a, st) : fused_any<1, true>(kind, a, st);
}

bool rows_ragged_fits(const DevRagged& c) { return c.S >= 1 && c.S <= 256; }

template <int P>
static hipError_t rows_ragged_launch(const DevRagged& c, double* x, long ld, int rows,
                                     hipStream_t st) {
  // rows per workgroup: at least a wave of chunks, at most 256 (128 of short
  // rows: 200000 rows of 100 74 us, 93 with 256), and in between as many as
  // leave the chip two workgroups per CU
  const int most = (c.S <= 8 ? 128 : 256) / c.S, least = c.S < 64 ? (64 + c.S - 1) / c.S : 1;
  int R = rows / 512;
  R = R < least ? least : R;
  R = R > most ? most : R;
  R = R > rows ? rows : R;
  const int T = ((R * c.S + 63) / 64) * 64;
  const int nel = R * c.n;
  const size_t lds = ((size_t)2 * P * T + nel + nel / 32 + 1) * sizeof(double);
  hipLaunchKernelGGL((rows_ragged<P>), dim3((unsigned)((rows + R - 1) / R)), dim3(T), lds, st, x,
                     ld, rows, c.n, R, fused_args(c, c.m, c.r, c.recl, x, ld, rows));
  return hipGetLastError();
}

hipError_t launch_rows_ragged(const DevRagged& c, double* x, long ld, int rows, hipStream_t st) {
  if (!rows_ragged_fits(c)) return hipErrorInvalidValue;
  return c.P == 2 ? rows_ragged_launch<2>(c, x, ld, rows, st)
                  : rows_ragged_launch<1>(c, x, ld, rows, st);
}

}  // namespace chx

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
// steps in a call: 0.27 ms (1.21 ms with a pass over memory per step); 131072
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

#include <type_traits>

#include "ch_launch.hpp"
#include "common.hpp"

namespace chx {

namespace {

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
template <int P, int M>
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
template <int P, int M>
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

// x = y - Zl sp - Zr so in the interior.  A wave that holds last chunks runs
// both tables, each chunk's separators masked to zero for the other's.
template <int P, int M>
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

// Lane l of a 16-lane row receives the value of lane l - 1 (row_shr:1), lane
// 0 of the row keeps `edge`; and the other way round.
__device__ __forceinline__ double dpp_row_from_left(double v, double edge) {
  const int lo = __builtin_amdgcn_update_dpp(__double2loint(edge), __double2loint(v), 0x111, 0xF,
                                             0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(__double2hiint(edge), __double2hiint(v), 0x111, 0xF,
                                             0xF, false);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double dpp_row_from_right(double v, double edge) {
  const int lo = __builtin_amdgcn_update_dpp(__double2loint(edge), __double2loint(v), 0x101, 0xF,
                                             0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(__double2hiint(edge), __double2hiint(v), 0x101, 0xF,
                                             0xF, false);
  return __hiloint2double(hi, lo);
}

// Lane l of a quad receives the value of its lane (SEL >> 2 l) & 3.
template <int SEL>
__device__ __forceinline__ double dpp_quad(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), SEL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), SEL, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
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

// LDS the ragged blocks take (stage_blocks), in doubles.
template <bool RAG>
__host__ __device__ __forceinline__ int blocks_lds(int dcount) {
  return RAG ? 12 * dcount : 0;
}

// The ragged blocks go to LDS (a barrier follows before they are read): their
// family differs from lane to lane, so they cannot be scalar loads.
template <bool RAG>
__device__ __forceinline__ void stage_blocks(const FusedArgs& A, double* lds) {
  if constexpr (RAG) {
    for (int e = threadIdx.x; e < 12 * A.dcount; e += blockDim.x) lds[e] = A.blocks[e];
  }
}

// The separators of chunk k from the reduced right-hand sides of its system,
// value a of chunk j at rho[a plane + j step], summed in the order of the
// separator kernels in solve.hip; four terms' loads are issued together.
template <int P, bool RAG>
__device__ __forceinline__ void separators(const FusedArgs& A, const double* blocks, int k,
                                           const double* rho, int plane, int step,
                                           double (&so)[P]) {
#pragma unroll
  for (int a = 0; a < P; ++a) so[a] = 0;
  int j = k + A.dlo, jw = j + (j < 0 ? A.S : 0);  // unwrapped and wrapped
  auto terms = [&](auto count, int t) {
    constexpr int N = decltype(count)::value;
    double w[N][P], B[N][P * P];
#pragma unroll
    for (int u = 0; u < N; ++u) {
#pragma unroll
      for (int a = 0; a < P; ++a) w[u][a] = rho[a * plane + jw * step];
      if constexpr (RAG) {
        const double* b = blocks + 4 * (A.dcount * rag_family(k, j, A.S) + t + u);
#pragma unroll
        for (int q = 0; q < P * P; ++q) B[u][q] = b[(q / P) * 2 + q % P];
      } else {
        const TabD b = (TabD)A.blocks + 4 * (t + u);
#pragma unroll
        for (int q = 0; q < P * P; ++q) B[u][q] = b[(q / P) * 2 + q % P];
      }
      ++j;
      jw = jw + 1 == A.S ? 0 : jw + 1;
    }
#pragma unroll
    for (int u = 0; u < N; ++u)
#pragma unroll
      for (int a = 0; a < P; ++a)
#pragma unroll
        for (int b = 0; b < P; ++b) so[a] = so[a] + B[u][a * P + b] * w[u][b];
  };
  int t = 0;
#pragma unroll 1
  for (; t + 4 <= A.dcount; t += 4) terms(std::integral_constant<int, 4>{}, t);
#pragma unroll 1
  for (; t < A.dcount; ++t) terms(std::integral_constant<int, 1>{}, t);
}

// Sum of two values over the workgroup in a fixed order, valid in thread 0;
// red: two doubles per wave.
__device__ __forceinline__ void group_sum2(double& m, double& e, double* red) {
  m = wave_sum(m);
  e = wave_sum(e);
  if ((threadIdx.x & 63) == 0) {
    red[2 * (threadIdx.x >> 6)] = m;
    red[2 * (threadIdx.x >> 6) + 1] = e;
  }
  __syncthreads();
  if (threadIdx.x == 0)
    for (int w = 1; w < (int)blockDim.x / 64; ++w) {
      m += red[2 * w];
      e += red[2 * w + 1];
    }
}

// The state's (mass, energy) from the n partials column_whole's workgroups
// left, by one workgroup.
__device__ __forceinline__ void diag_tail(const DiagTail& d, double* sm) {
  double m = 0.0, e = 0.0;
  for (long b = threadIdx.x; b < d.n; b += blockDim.x) {
    m += d.part[2 * b];
    e += d.part[2 * b + 1];
  }
  group_sum2(m, e, sm);
  if (threadIdx.x == 0) {
    d.out[0] = m * d.scale;
    d.out[1] = e * d.scale;
  }
}

}  // namespace

// KIND -1: one solve of the right-hand sides in x; KIND 0 .. 2: nsteps steps of
// a 1D scheme from the state in x.  In place: a workgroup owns its systems and
// loads all of them before it stores.
template <int P, int L, bool RAG, int KIND, bool LINES, int M = kChunk>
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
  double* const blk = sm + 2 * P * S * L;
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
  stage_blocks<RAG>(A, blk);
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
      ragged_sweep<P, M>(f, li, rec, eps, t1, t2);
    } else {
#pragma unroll
      for (int a = 0; a < P; ++a) fs[a] = f[MI + a];
      chunk_sweep<P, M, double, TabD>(f, rec, eps);
      t1 = f[MI - 1];
      t2 = f[MI - 2];
    }
    double pa[P], pb[P];
    ragged_parts<P, M>(f, fs, t1, t2, A.bd, pa, pb);
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
    separators<P, RAG>(A, blk, k, rho + c, plane, L, so);
    if (active) {
#pragma unroll
      for (int a = 0; a < P; ++a) part[a * plane + me] = so[a];
    }
    __syncthreads();
#pragma unroll
    for (int a = 0; a < P; ++a) sp[a] = part[a * plane + pv];
    if constexpr (RAG) {
      ragged_correct<P, M>(f, last, table(A.rec), table(A.recl), sp, so);
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
// latency they cover: 20000 rows of 1000 points 70 us, 4.6 TB/s (79 us with a
// thread's 32 loads issued 8 at a time; one thread per row: 800 us, every lane
// on a line of its own, 313 waves of them in all).
// RAG as above, else rows of S M points (bitwise what the other
// row kernels give).  From src to dst, which may be the same array.  stream:
// the stores go past the caches, each as its value leaves LDS (large solves:
// 20000 rows of 1000 70 us, 80 with all of a thread's values read first);
// otherwise all at once and through the caches (1000 rows of 500 10.0 us
// against 10.9; the step's column kernel reads the rows again: 1000 x 1000
// 21.2 us per step, 22.1 streamed).  With
// tail.out, the launch's last workgroup solves no rows: it finishes the
// (mass, energy) of the state that the column kernel before it has read.
// UPD: the solved rows v are not stored: they advance the thesis scheme's two
// states, next = (2 C - Cp) + v and, where given, next_prev = C (each element
// read before it is written: next may be Cp, or next C and next_prev Cp).
template <int P, int M, bool RAG, bool UPD = false>
__global__ __launch_bounds__(256) void rows_any(const double* src, long lds, double* dst, long ldd,
                                                int rows, int n, unsigned magic, int R,
                                                const FusedArgs A, const DiagTail tail,
                                                const bool stream, const StateUpdate up) {
  extern __shared__ double sm[];
  if (tail.out != nullptr && blockIdx.x == gridDim.x - 1) {
    diag_tail(tail, sm);
    return;
  }
  const int S = A.S, T = blockDim.x, t = threadIdx.x;
  const long row0 = (long)blockIdx.x * R;
  const int nr = rows - row0 < R ? (int)(rows - row0) : R;
  const int nel = nr * n;
  double* const part = sm;           // [P][T]
  double* const rho = sm + P * T;    // [P][T]
  double* const blk = sm + 2 * P * T;
  double* const tile = blk + blocks_lds<RAG>(A.dcount);
  const int rt = t / S;
  const bool active = rt < nr;
  const int r = active ? rt : nr - 1, k = active ? t - rt * S : S - 1;
  const bool last = k == S - 1;
  const int len = RAG ? (last ? A.r : A.m) : M, li = len - P;
  const double* const xs = src + row0 * lds;
  double* const xd = dst + row0 * ldd;
  // element e of the group is row e / n (magic = ceil(2^32 / n): exact for the
  // 13 bits of both)
  auto at = [&](int e, long ld) -> long {
    const unsigned q = __umulhi((unsigned)e, magic);
    return (long)q * ld + (e - (int)q * n);
  };
  auto slot = [](int e) { return e + e / M; };
  // a thread's at most M elements, every load in flight; pairs where the
  // group is one aligned range
  auto pairs = [&](const double* p, long ld) {
    return ld == n && (reinterpret_cast<unsigned long>(p) & 15) == 0;
  };
  {
    double v[M], odd = 0.0;
    const bool two = pairs(xs, lds);
    if (two) {
#pragma unroll
      for (int u = 0; u < M / 2; ++u) {
        const int e = 2 * (t + u * T);
        typedef double dv2 __attribute__((ext_vector_type(2)));
        // (past the last pair: the first again, not used)
        const dv2 w = __builtin_nontemporal_load(
            reinterpret_cast<const dv2*>(xs + (e + 1 < nel ? e : 0)));
        v[2 * u] = w.x;
        v[2 * u + 1] = w.y;
      }
      if (nel & 1) odd = xs[nel - 1];
    } else {
#pragma unroll
      for (int u = 0; u < M; ++u) {
        const int e = t + u * T;
        v[u] = __builtin_nontemporal_load(xs + at(e < nel ? e : nel - 1, lds));
      }
    }
    stage_blocks<RAG>(A, blk);
    warm<M - P>(A.rec);
    if (two) {
#pragma unroll
      for (int u = 0; u < M / 2; ++u) {
        const int e = 2 * (t + u * T);
        if (e + 1 < nel) {
          tile[slot(e)] = v[2 * u];
          tile[slot(e + 1)] = v[2 * u + 1];
        }
      }
      if ((nel & 1) && t == 0) tile[slot(nel - 1)] = odd;
    } else {
#pragma unroll
      for (int u = 0; u < M; ++u) {
        const int e = t + u * T;
        if (e < nel) tile[slot(e)] = v[u];
      }
    }
  }
  // the states' elements, in flight until the rows are solved
  double uc[UPD ? M : 1], upv[UPD ? M : 1];
  if constexpr (UPD) {
#pragma unroll
    for (int u = 0; u < M; ++u) {
      const int e = t + u * T < nel ? t + u * T : nel - 1;
      uc[u] = up.c[row0 * up.ldc + at(e, up.ldc)];
      upv[u] = up.cp[row0 * up.ldp + at(e, up.ldp)];
    }
  }
  __syncthreads();
  double f[M];
  const int e0 = r * n + k * (RAG ? A.m : M);
#pragma unroll
  for (int p = 0; p < M; ++p)  // past the chunk: its last unknown
    f[p] = tile[slot(e0 + (!RAG || p < len ? p : len - 1))];
  double fs[P], t1 = 0, t2 = 0, pa[P], pb[P];
  if constexpr (RAG) {
#pragma unroll
    for (int a = 0; a < P; ++a) fs[a] = tile[slot(e0 + li + a)];
    ragged_sweep<P, M>(f, li, table(A.rec), A.bd.c[0], t1, t2);
  } else {
#pragma unroll
    for (int a = 0; a < P; ++a) fs[a] = f[M - P + a];
    chunk_sweep<P, M, double, TabD>(f, table(A.rec), A.bd.c[0]);
    t1 = f[M - P - 1];
    t2 = f[M - P - 2];
  }
  ragged_parts<P, M>(f, fs, t1, t2, A.bd, pa, pb);
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
  separators<P, RAG>(A, blk, k, rho + rs, T, 1, so);
  if (active) {
#pragma unroll
    for (int a = 0; a < P; ++a) part[a * T + me] = so[a];
  }
  __syncthreads();
#pragma unroll
  for (int a = 0; a < P; ++a) sp[a] = part[a * T + pv];
  if constexpr (RAG) ragged_correct<P, M>(f, last, table(A.rec), table(A.recl), sp, so);
  else chunk_correct<P, M, double, TabD>(f, table(A.rec), sp, so);
  if (active) {
    const int lj = RAG ? fresh(li) : li;
#pragma unroll
    for (int p = 0; p < M - P; ++p)
      if (!RAG || p < lj) tile[slot(e0 + p)] = f[p];
#pragma unroll
    for (int a = 0; a < P; ++a) tile[slot(e0 + lj + a)] = so[a];
  }
  __syncthreads();
  if constexpr (UPD) {
    double v[M];
#pragma unroll
    for (int u = 0; u < M; ++u) {
      const int e = t + u * T;
      v[u] = (2.0 * uc[u] - upv[u]) + tile[slot(e < nel ? e : nel - 1)];
    }
#pragma unroll
    for (int u = 0; u < M; ++u) {
      const int e = t + u * T;
      if (e >= nel) continue;
      up.next[row0 * up.ldn + at(e, up.ldn)] = v[u];
      if (up.next_prev != nullptr) up.next_prev[row0 * up.ldn + at(e, up.ldn)] = uc[u];
    }
  } else if (stream && ldd == n) {
    for (int e = t; e < nel; e += T) __builtin_nontemporal_store(tile[slot(e)], xd + e);
  } else if (pairs(xd, ldd)) {
    double2 v[M / 2];
#pragma unroll
    for (int u = 0; u < M / 2; ++u) {
      const int e = 2 * (t + u * T), g = e + 1 < nel ? e : 0;
      v[u].x = tile[slot(g)];
      v[u].y = tile[slot(g + 1)];
    }
#pragma unroll
    for (int u = 0; u < M / 2; ++u) {
      const int e = 2 * (t + u * T);
      if (e + 1 < nel) *reinterpret_cast<double2*>(xd + e) = v[u];
    }
    if ((nel & 1) && t == 0) xd[nel - 1] = tile[slot(nel - 1)];
  } else {
    double v[M];
#pragma unroll
    for (int u = 0; u < M; ++u) {
      const int e = t + u * T;
      v[u] = tile[slot(e < nel ? e : nel - 1)];
    }
#pragma unroll
    for (int u = 0; u < M; ++u) {
      const int e = t + u * T;
      if (e < nel) __builtin_nontemporal_store(v[u], xd + at(e, ldd));
    }
  }
}

// The solve of one chunk per thread, a workgroup holding whole columns: f the
// right-hand sides in, the interior's solutions out; fs the separators'
// (RAG: given; otherwise f's last two).
template <int P, int M, int L, bool RAG>
__device__ __forceinline__ void column_solve(const FusedArgs& A, double (&f)[M], double (&fs)[P],
                                             double* part, double* rho, const double* blk, int k,
                                             int c, int me, int nxt, int prv, bool active,
                                             bool last, int li) {
  constexpr int MI = M - P;
  const int plane = A.S * L;
  const double eps = A.bd.c[0];
  double t1 = 0, t2 = 0, pa[P], pb[P];
  if constexpr (RAG) {
    ragged_sweep<P, M>(f, li, table(A.rec), eps, t1, t2);
  } else {
#pragma unroll
    for (int a = 0; a < P; ++a) fs[a] = f[MI + a];
    chunk_sweep<P, M, double, TabD>(f, table(A.rec), eps);
    t1 = f[MI - 1];
    t2 = f[MI - 2];
  }
  ragged_parts<P, M>(f, fs, t1, t2, A.bd, pa, pb);
  if (active) {
#pragma unroll
    for (int a = 0; a < P; ++a) part[a * plane + me] = pb[a];
  }
  __syncthreads();
#pragma unroll
  for (int a = 0; a < P; ++a) pa[a] -= part[a * plane + nxt];
  if (active) {
#pragma unroll
    for (int a = 0; a < P; ++a) rho[a * plane + me] = pa[a];
  }
  __syncthreads();
  double sp[P];
  separators<P, RAG>(A, blk, k, rho + c, plane, L, fs);
  if (active) {
#pragma unroll
    for (int a = 0; a < P; ++a) part[a * plane + me] = fs[a];
  }
  __syncthreads();
#pragma unroll
  for (int a = 0; a < P; ++a) sp[a] = part[a * plane + prv];
  if constexpr (RAG) ragged_correct<P, M>(f, last, table(A.rec), table(A.recl), sp, fs);
  else chunk_correct<P, M, double, TabD>(f, table(A.rec), sp, fs);
}

// A solved chunk into its column: the interior, then the separators.
template <int P, int M, bool RAG>
__device__ __forceinline__ void column_store(const double (&f)[M], const double (&fs)[P],
                                             double* p0, long ldd, int li) {
  const int lj = RAG ? fresh(li) : M - P;
#pragma unroll
  for (int p = 0; p < M - P; ++p)
    if (!RAG || p < lj) __builtin_nontemporal_store(f[p], p0 + (long)p * ldd);
#pragma unroll
  for (int a = 0; a < P; ++a) __builtin_nontemporal_store(fs[a], p0 + (long)(lj + a) * ldd);
}

// One step's right-hand side and column solves of a periodic 2D field, from
// src to dst (not the same array): a workgroup takes L columns and every
// chunk of them, so the columns leave it solved and corrected.  Small and
// odd grids: the step is this launch and the rows.
// Thread (c, k) forms r on its chunk of column c from the rows around it
// (registers) and the columns beside it (DPP lane shifts inside the tile; the
// edge lanes load the columns outside it), in the expressions of the column
// pass in ch.hip, and solves as il_fused does.  What bounds it is the chain
// load, right-hand side, sweep, separators, correction, store of one chunk,
// so every load of a thread is issued before its first row.
// DIAG: a (mass, energy) partial of src per workgroup.
template <int M, int L, bool RAG, bool DIAG>
__global__ __launch_bounds__(512) void column_whole(const double* __restrict__ src, long lds,
                                                    double* __restrict__ dst, long ldd, int nx,
                                                    int ny, const ChCoef K,
                                                    double* __restrict__ dpart,
                                                    const FusedArgs A) {
  constexpr int P = 2, MI = M - P;
  extern __shared__ double sm[];
  const int S = A.S;
  const int c = threadIdx.x % L, kt = threadIdx.x / L;
  const bool active = kt < S;
  const int k = active ? kt : S - 1;
  // the last tile starts early enough to be whole; its first columns are its
  // neighbour's
  const int t0 = (int)tile_of<false>(blockIdx.x, gridDim.x) * L;
  const int i0 = t0 + L <= nx ? t0 : nx - L, i = i0 + c;
  const bool sv = active && i >= t0;
  double* const part = sm;
  double* const rho = sm + P * S * L;
  double* const blk = sm + 2 * P * S * L;
  double* const dred = blk + blocks_lds<RAG>(A.dcount);
  const int me = k * L + c;
  const int nxt = (k + 1 == S ? 0 : k + 1) * L + c, prv = (k == 0 ? S - 1 : k - 1) * L + c;
  const bool last = k == S - 1;
  const int len = RAG ? (last ? A.r : A.m) : M;
  const int li = len - P;
  const int row0 = k * (RAG ? A.m : M);

  double X[M + 2], E[M + 2];  // rows row0 - 1 .. row0 + len of the column; of the one outside
  {
    // lane 0 also loads the column left of the tile, its last lane the one right of it
    const int ie = c == 0 ? (i == 0 ? nx - 1 : i - 1)
                          : (c == L - 1 ? (i == nx - 1 ? 0 : i + 1) : i);
    const long de = (long)ie - i;
    const double* const up = src + (long)(row0 == 0 ? ny - 1 : row0 - 1) * lds + i;
    const double* const dn = src + (long)(row0 + len == ny ? 0 : row0 + len) * lds + i;
    const double* own = src + (long)row0 * lds + i;
    X[0] = up[0];
    E[0] = up[de];
#pragma unroll
    for (int q = 1; q <= M + 1; ++q) {  // past the chunk: the row after it
      const double* const a = q <= (RAG ? len : M) ? own : dn;
      X[q] = a[0];
      E[q] = a[de];
      own += lds;
    }
  }
  stage_blocks<RAG>(A, blk);
  warm<MI>(A.rec);
  double f[M], fs[P] = {0, 0};
  double msum = 0.0, esum = 0.0;
  {
    auto left = [&](int q) {
      double v = dpp_row_from_left(X[q], E[q]);
      return L < 16 && c == 0 ? E[q] : v;
    };
    auto right = [&](int q) {
      double v = dpp_row_from_right(X[q], E[q]);
      return L < 16 && c == L - 1 ? E[q] : v;
    };
    double xc_m = X[0], xl_m = left(0), xr_m = right(0);
    double xc_c = X[1], xl_c = left(1), xr_c = right(1);
#pragma unroll
    for (int p = 0; p < M; ++p) {
      const double xc_p = X[p + 2], xl_p = left(p + 2), xr_p = right(p + 2);
      const double mu_c = xc_c * xc_c * xc_c - xc_c;
      const double mu_l = xl_c * xl_c * xl_c - xl_c;
      const double mu_r = xr_c * xr_c * xr_c - xr_c;
      const double mu_s = xc_m * xc_m * xc_m - xc_m;
      const double mu_n = xc_p * xc_p * xc_p - xc_p;
      const double lap = K.cx * (mu_r + mu_l - 2.0 * mu_c) + K.cy * (mu_n + mu_s - 2.0 * mu_c);
      const double dyy_w = xl_p + xl_m - 2.0 * xl_c;
      const double dyy_c = xc_p + xc_m - 2.0 * xc_c;
      const double dyy_e = xr_p + xr_m - 2.0 * xr_c;
      double r = xc_c + lap - K.ccross * (dyy_e + dyy_w - 2.0 * dyy_c);
      if (DIAG) {
        const double w = xc_c * xc_c - 1.0;
        const double gx = (xr_c - xc_c) * K.inv_dx, gy = (xc_p - xc_c) * K.inv_dy;
        const bool in = !RAG || p < len;
        msum += in ? xc_c : 0.0;
        const double ee = 0.25 * w * w + K.half_gamma * (gx * gx + gy * gy);
        esum += in ? ee : 0.0;
      }
      f[p] = r;
      if constexpr (RAG) {
#pragma unroll
        for (int a = 0; a < P; ++a) {
          fs[a] = p == li + a ? r : fs[a];
          asm volatile("" : "+v"(fs[a]));
        }
      }
      xl_m = xl_c; xc_m = xc_c; xr_m = xr_c;
      xl_c = xl_p; xc_c = xc_p; xr_c = xr_p;
    }
  }
  column_solve<P, M, L, RAG>(A, f, fs, part, rho, blk, k, c, me, nxt, prv, active, last, li);
  if (sv) column_store<P, M, RAG>(f, fs, dst + (long)row0 * ldd + i, ldd, li);
  // the diagnostics' sums, while the stores drain
  if (DIAG) {
    msum = sv ? msum : 0.0;
    esum = sv ? esum : 0.0;
    group_sum2(msum, esum, dred);
    if (threadIdx.x == 0) {
      dpart[2 * blockIdx.x] = msum;
      dpart[2 * blockIdx.x + 1] = esum;
    }
  }
}

// The thesis scheme's step in the same form: r from the two states C and Cp
// (the expressions of ch2_rhs in ch.hip) and the column solves.  Tiles of four
// columns: each lane holds its own column and one of the four outside the
// tile (two on either side), and the neighbours at distance one and two come
// from the quad's lanes.
template <int M, bool RAG, bool DIAG>
__global__ __launch_bounds__(512) void column_whole2(const double* __restrict__ C, long ldc,
                                                     const double* __restrict__ Cp, long ldp,
                                                     double* __restrict__ dst, long ldd, int nx,
                                                     int ny, const Ch2Coef K, const ChCoef D,
                                                     double* __restrict__ dpart,
                                                     const FusedArgs A) {
  constexpr int P = 2, MI = M - P, L = 4, Q = M + 4;
  extern __shared__ double sm[];
  const int S = A.S;
  const int c = threadIdx.x % L, kt = threadIdx.x / L;
  const bool active = kt < S;
  const int k = active ? kt : S - 1;
  const int t0 = (int)tile_of<false>(blockIdx.x, gridDim.x) * L;
  const int i0 = t0 + L <= nx ? t0 : nx - L, i = i0 + c;
  const bool sv = active && i >= t0;
  double* const part = sm;
  double* const rho = sm + P * S * L;
  double* const blk = sm + 2 * P * S * L;
  double* const dred = blk + blocks_lds<RAG>(A.dcount);
  const int me = k * L + c;
  const int nxt = (k + 1 == S ? 0 : k + 1) * L + c, prv = (k == 0 ? S - 1 : k - 1) * L + c;
  const bool last = k == S - 1;
  const int len = RAG ? (last ? A.r : A.m) : M;
  const int li = len - P;
  const int row0 = k * (RAG ? A.m : M);

  // own column and the one outside, rows row0 - 2 .. row0 + len + 1
  double xc[Q], xp[Q], hc[Q], hp[Q];
  {
    int ih = c < 2 ? i0 - 2 + c : i0 + 2 + c;
    ih += ih < 0 ? nx : 0;
    ih -= ih >= nx ? nx : 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      int j = row0 - 2 + (q < (RAG ? len : M) + 4 ? q : 0);
      j += j < 0 ? ny : 0;
      j -= j >= ny ? ny : 0;
      const double* const a = C + (long)j * ldc;
      const double* const b = Cp + (long)j * ldp;
      xc[q] = a[i];
      hc[q] = a[ih];
      xp[q] = b[i];
      hp[q] = b[ih];
    }
  }
  stage_blocks<RAG>(A, blk);
  warm<MI>(A.rec);
  double f[M], fs[P] = {0, 0};
  double msum = 0.0, esum = 0.0;
  {
    // lane l of a quad takes lane ((sel >> 2 l) & 3)'s value
    auto left1 = [&](double own, double out) {  // columns c - 1
      const double a = dpp_quad<0x90>(own), b = dpp_quad<0x01>(out);
      return c == 0 ? b : a;
    };
    auto right1 = [&](double own, double out) {  // c + 1
      const double a = dpp_quad<0xF9>(own), b = dpp_quad<0x80>(out);
      return c == 3 ? b : a;
    };
    auto left2 = [&](double own, double out) {  // c - 2: the lanes outside hold them in order
      const double a = dpp_quad<0x40>(own);
      return c < 2 ? out : a;
    };
    auto right2 = [&](double own, double out) {  // c + 2
      const double a = dpp_quad<0x0E>(own);
      return c >= 2 ? out : a;
    };
    double B[Q], U[Q], BL[Q], BR[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      B[q] = 2.0 * xc[q] - xp[q];
      U[q] = xc[q] * xc[q] * xc[q] - xc[q];
      const double H = 2.0 * hc[q] - hp[q];
      BL[q] = left1(B[q], H);
      BR[q] = right1(B[q], H);
      if (q < 4) continue;
      const int w = q - 2, p = q - 4;  // right-hand side of the chunk's row p
      const double Hw = 2.0 * hc[w] - hp[w];
      const double hu = hc[w] * hc[w] * hc[w] - hc[w];
      const double mu_l = left1(U[w], hu), mu_r = right1(U[w], hu);
      const double d4x = (left2(B[w], Hw) - 4.0 * BL[w] + 6.0 * B[w] - 4.0 * BR[w] +
                          right2(B[w], Hw)) * K.inv_dx4;
      const double d4y =
          (B[w - 2] - 4.0 * B[w - 1] + 6.0 * B[w] - 4.0 * B[w + 1] + B[w + 2]) * K.inv_dy4;
      const double dyy_w = BL[w + 1] + BL[w - 1] - 2.0 * BL[w];
      const double dyy_c = B[w + 1] + B[w - 1] - 2.0 * B[w];
      const double dyy_e = BR[w + 1] + BR[w - 1] - 2.0 * BR[w];
      const double dxxyy = (dyy_e + dyy_w - 2.0 * dyy_c) * K.inv_dx2dy2;
      const double bih = d4x + 2.0 * dxxyy + d4y;
      const double lap = (mu_r + mu_l - 2.0 * U[w]) * K.inv_dx2 +
                         (U[w + 1] + U[w - 1] - 2.0 * U[w]) * K.inv_dy2;
      const double r = -(2.0 / 3.0) * (xc[w] - xp[w]) - K.a * bih + K.b * lap;
      if (DIAG) {
        const double ww = xc[w] * xc[w] - 1.0;
        const double gx = (right1(xc[w], hc[w]) - xc[w]) * D.inv_dx;
        const double gy = (xc[w + 1] - xc[w]) * D.inv_dy;
        const bool in = !RAG || p < len;
        msum += in ? xc[w] : 0.0;
        const double ee = 0.25 * ww * ww + D.half_gamma * (gx * gx + gy * gy);
        esum += in ? ee : 0.0;
      }
      f[p] = r;
      if constexpr (RAG) {
#pragma unroll
        for (int a = 0; a < P; ++a) {
          fs[a] = p == li + a ? r : fs[a];
          asm volatile("" : "+v"(fs[a]));
        }
      }
    }
  }
  column_solve<P, M, L, RAG>(A, f, fs, part, rho, blk, k, c, me, nxt, prv, active, last, li);
  if (sv) column_store<P, M, RAG>(f, fs, dst + (long)row0 * ldd + i, ldd, li);
  if (DIAG) {
    msum = sv ? msum : 0.0;
    esum = sv ? esum : 0.0;
    group_sum2(msum, esum, dred);
    if (threadIdx.x == 0) {
      dpart[2 * blockIdx.x] = msum;
      dpart[2 * blockIdx.x + 1] = esum;
    }
  }
}

// Mass and energy of a plain field by one workgroup: small grids, where a
// second launch costs more than the sum.
__global__ __launch_bounds__(1024) void diag_small(const double* __restrict__ c, long ld, int nx,
                                                   int ny, const ChCoef K,
                                                   double* __restrict__ out) {
  __shared__ double red[2 * 16];
  double m = 0.0, e = 0.0;
  for (int j = threadIdx.x >> 6; j < ny; j += 16) {
    const double* const row = c + (long)j * ld;
    const double* const up = c + (long)(j + 1 == ny ? 0 : j + 1) * ld;
    for (int i = threadIdx.x & 63; i < nx; i += 64) {
      const double x = row[i];
      const double gx = (row[i + 1 == nx ? 0 : i + 1] - x) * K.inv_dx;
      const double gy = (up[i] - x) * K.inv_dy;
      const double w = x * x - 1.0;
      m += x;
      e += 0.25 * w * w + K.half_gamma * (gx * gx + gy * gy);
    }
  }
  group_sum2(m, e, red);
  if (threadIdx.x == 0) {
    out[0] = m * K.dxdy;
    out[1] = e * K.dxdy;
  }
}

hipError_t launch_diag_small(const double* c, long ld, int nx, int ny, const ChCoef& K,
                             double* out, hipStream_t st) {
  hipLaunchKernelGGL(diag_small, dim3(1), dim3(1024), 0, st, c, ld, nx, ny, K, out);
  return hipGetLastError();
}

// Systems per workgroup (16, 32 or 64: whole lines of every row), or 0 where
// 16 systems need more than 1024 threads.  More systems make longer rows of a
// tile and fewer workgroups: 64 where that leaves two workgroups of 512
// threads per CU (524288 systems of 256: 395 us, 419 with 32, 455 with 16), 32
// up to 1024 threads (131072 systems of 1024: 444 us, 457 with 16; 512 points:
// 395 us, 409 with 64), as long as there are two workgroups for every CU
// (1024 systems of 1024: 9.4 us with 16, 12.3 with 32).
// The 1D schemes' steps wait on each other at barriers and want several small
// workgroups per CU: 32 up to 512 threads, else 16 (four steps of 262144
// systems of 256: 268 us with 32, 298 with 64; 65536 of 1024: 343 us with 16,
// 484 with 32).
int il_fused_systems(int S, int batch, bool steps) {
  if (S * 16 > 1024) return 0;
  if (steps) return S * 32 <= 512 && batch >= 32 * 512 ? 32 : 16;
  if (S * 64 <= 512 && batch >= 64 * 512) return 64;
  return S * 32 <= 1024 && batch >= 32 * 512 ? 32 : 16;
}

template <int P, int L, bool RAG, int KIND>
static hipError_t fused_launch(const FusedArgs& a, hipStream_t st) {
  const dim3 grid((unsigned)((a.batch + L - 1) / L)), block(((L * a.S + 63) / 64) * 64);
  const size_t lds = ((size_t)2 * P * a.S * L + blocks_lds<RAG>(a.dcount)) * sizeof(double);
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
  switch (il_fused_systems(a.S, a.batch, kind >= 0)) {
    case 64: return fused_launch<P, 64, RAG, -1>(a, st);
    case 32: return fused_kind<P, 32, RAG>(kind, a, st);
    case 16: return fused_kind<P, 16, RAG>(kind, a, st);
    default: return hipErrorInvalidValue;
  }
}

static FusedArgs fused_args(const DevRagged& c, double* x, long ld, int batch) {
  FusedArgs a{};
  a.x = x;
  a.ld = ld;
  a.batch = batch;
  a.nsteps = 1;
  a.S = c.S;
  a.m = c.m;
  a.r = c.r;
  a.dlo = c.dlo;
  a.dcount = c.dcount;
  a.rec = c.rec;
  a.recl = c.recl;
  a.blocks = c.blocks;
  for (int i = 0; i < 5; ++i) a.bd.c[i] = c.coef[i];
  return a;
}

hipError_t launch_il_fused(const DevRagged& c, int kind, double* x, long ld, int batch, int nsteps,
                           double s, double al, hipStream_t st) {
  if (c.M != kChunk) return hipErrorInvalidValue;
  FusedArgs a = fused_args(c, x, ld, batch);
  a.nsteps = nsteps;
  a.s = s;
  a.al = al;
  if (c.even) return c.P == 2 ? fused_any<2, false>(kind, a, st) : fused_any<1, false>(kind, a, st);
  return c.P == 2 ? fused_any<2, true>(kind, a, st) : fused_any<1, true>(kind, a, st);
}

bool rows_any_fits(const DevRagged& c) { return c.S >= 1 && c.S <= 256; }

static hipError_t rows_any_launch(const DevRagged& c, const double* src, long lds, double* dst,
                                  long ldd, int rows, const DiagTail* tail, bool stream,
                                  const StateUpdate* update, hipStream_t st) {
  if (!rows_any_fits(c)) return hipErrorInvalidValue;
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
  const size_t lds_bytes =
      ((size_t)2 * c.P * T + (c.even ? 0 : 12 * c.dcount) + nel + nel / c.M + 1) * sizeof(double);
  const unsigned magic = (unsigned)(((1ull << 32) + c.n - 1) / c.n);
  const dim3 grid((unsigned)((rows + R - 1) / R + (tail ? 1 : 0)));
  const FusedArgs a = fused_args(c, nullptr, 0, rows);
  const DiagTail d = tail ? *tail : DiagTail{};
  const StateUpdate up = update ? *update : StateUpdate{};
#define CHX_ROWS(P_, M_, RAG_, U_)                                                               \
  hipLaunchKernelGGL((rows_any<P_, M_, RAG_, U_>), grid, dim3(T), lds_bytes, st, src, lds, dst,  \
                     ldd, rows, c.n, magic, R, a, d, stream, up)
#define CHX_ROWS_M(RAG_, U_)                            \
  do {                                                  \
    if (c.M == 8) CHX_ROWS(2, 8, RAG_, U_);             \
    else if (c.M == 16) CHX_ROWS(2, 16, RAG_, U_);      \
    else CHX_ROWS(2, kChunk, RAG_, U_);                 \
  } while (0)
  if (c.P == 1) {
    if (c.even || c.M != kChunk || update) return hipErrorInvalidValue;
    CHX_ROWS(1, kChunk, true, false);
  } else if (update) {
    if (c.even) CHX_ROWS_M(false, true);
    else CHX_ROWS_M(true, true);
  } else {
    if (c.even) CHX_ROWS_M(false, false);
    else CHX_ROWS_M(true, false);
  }
#undef CHX_ROWS_M
#undef CHX_ROWS
  return hipGetLastError();
}

hipError_t launch_rows_any(const DevRagged& c, const double* src, long lds, double* dst, long ldd,
                           int rows, const DiagTail* tail, bool stream, hipStream_t st) {
  return rows_any_launch(c, src, lds, dst, ldd, rows, tail, stream, nullptr, st);
}

hipError_t launch_rows_update(const DevRagged& c, const double* src, long lds, int rows,
                              const StateUpdate& update, const DiagTail* tail, hipStream_t st) {
  return rows_any_launch(c, src, lds, nullptr, 0, rows, tail, false, &update, st);
}

// Columns per workgroup, or 0 where 4 columns need more than 512 threads.
int column_whole_columns(int nx, int S) {
  if (S * 4 > 512) return 0;
  if (nx >= 16 * 256 && S * 16 <= 512) return 16;
  if (nx >= 8 * 256 && S * 8 <= 512) return 8;
  return nx >= 4 ? 4 : 0;
}

long column_whole_blocks(int nx, int S) {
  const int L = column_whole_columns(nx, S);
  return L > 0 ? (nx + L - 1) / L : 0;
}

hipError_t launch_column_whole(const DevRagged& c, const double* src, long lds, double* dst,
                               long ldd, int nx, int ny, const ChCoef& K, double* dpart,
                               hipStream_t st) {
  const int L = column_whole_columns(nx, c.S);
  if (c.P != 2 || L == 0 || c.n != ny || src == dst) return hipErrorInvalidValue;
  const dim3 grid((unsigned)((nx + L - 1) / L)), block(((L * c.S + 63) / 64) * 64);
  const size_t lds_bytes =
      ((size_t)4 * c.S * L + (c.even ? 0 : 12 * c.dcount) + 16) * sizeof(double);
  const FusedArgs a = fused_args(c, nullptr, 0, nx);
  const bool diag = dpart != nullptr;
#define CHX_COLW(M_, L_, RAG_, D_)                                                               \
  hipLaunchKernelGGL((column_whole<M_, L_, RAG_, D_>), grid, block, lds_bytes, st, src, lds, dst, \
                     ldd, nx, ny, K, dpart, a)
#define CHX_COLW_L(M_, RAG_, D_)             \
  do {                                       \
    if (L == 16) CHX_COLW(M_, 16, RAG_, D_); \
    else if (L == 8) CHX_COLW(M_, 8, RAG_, D_); \
    else CHX_COLW(M_, 4, RAG_, D_);          \
  } while (0)
#define CHX_COLW_M(RAG_, D_)                      \
  do {                                            \
    if (c.M == 8) CHX_COLW_L(8, RAG_, D_);        \
    else if (c.M == 16) CHX_COLW_L(16, RAG_, D_); \
    else CHX_COLW_L(kChunk, RAG_, D_);            \
  } while (0)
  if (c.even && diag) CHX_COLW_M(false, true);
  else if (c.even) CHX_COLW_M(false, false);
  else if (diag) CHX_COLW_M(true, true);
  else CHX_COLW_M(true, false);
#undef CHX_COLW_M
#undef CHX_COLW_L
#undef CHX_COLW
  return hipGetLastError();
}

hipError_t launch_column_whole2(const DevRagged& c, const double* C, long ldc, const double* Cp,
                                long ldp, double* dst, long ldd, int nx, int ny,
                                const Ch2Coef& K, const ChCoef& D, double* dpart,
                                hipStream_t st) {
  if (c.P != 2 || c.M > 16 || c.S * 4 > 512 || nx < 5 || c.n != ny || dst == C || dst == Cp)
    return hipErrorInvalidValue;
  const dim3 grid((unsigned)((nx + 3) / 4)), block(((4 * c.S + 63) / 64) * 64);
  const size_t lds_bytes =
      ((size_t)16 * c.S + (c.even ? 0 : 12 * c.dcount) + 16) * sizeof(double);
  const FusedArgs a = fused_args(c, nullptr, 0, nx);
#define CHX_COL2(M_, RAG_, D_)                                                                    \
  hipLaunchKernelGGL((column_whole2<M_, RAG_, D_>), grid, block, lds_bytes, st, C, ldc, Cp, ldp, \
                     dst, ldd, nx, ny, K, D, dpart, a)
#define CHX_COL2_M(RAG_, D_)             \
  do {                                   \
    if (c.M == 8) CHX_COL2(8, RAG_, D_); \
    else CHX_COL2(16, RAG_, D_);         \
  } while (0)
  if (dpart) {
    if (c.even) CHX_COL2_M(false, true);
    else CHX_COL2_M(true, true);
  } else {
    if (c.even) CHX_COL2_M(false, false);
    else CHX_COL2_M(true, false);
  }
#undef CHX_COL2_M
#undef CHX_COL2
  return hipGetLastError();
}

}  // namespace chx

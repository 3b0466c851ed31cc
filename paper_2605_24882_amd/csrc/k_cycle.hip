// The coarse part of the multigrid V-cycle in one launch (on the smallest spaces all of it).
//
// The columns of a batch are independent systems, so a block that owns 16 columns can run every step
// of the V-cycle on the coarsest levels by itself: smoothing, residual, restriction, the dense solve
// and the way back up need no other block, only barriers within it.  Launched one by one these steps
// are some eight kernels per level of 4 to 20 us each, whatever little they compute: their time is the
// latency of the launch and of a handful of dependent loads.
//
// Mapping: 1024 threads as 64 groups of 16 lanes, lane = column, group = coefficient row.  A group's
// lanes hold its row's stencil (lane l of chunk k: tap 16 k + l of the level's M and S) and each tap
// is broadcast within the 16 lanes by DPP, as in k_stencil.  The current level's iterate, the one
// before it and its right-hand side lie in LDS, 16 columns of every patch coefficient without ghost
// rows: taps that leave the patch have the coefficient zero and read whatever row follows, so no index
// is clamped.  What the way back up needs of a finer level (right-hand side, iterate) waits in the
// level's batch vectors.  The index tables and diagonals of all levels are copied to LDS first, so that
// a step waits for memory once at most (for its first row's stencil, loaded before the barrier ahead
// of it).  Patch-boundary rows take two phases, as in the launches: the patch contributions first, then
// the sum over the copies and the step.
#include "gf_internal.h"
#include "k_solve.h"
#include "k_stencil.h"

namespace gf {

constexpr int kCycThreads = 1024;
constexpr int kCycCols = 16;                        // columns per block
constexpr int kCycGroups = kCycThreads / kCycCols;  // rows in flight per block
constexpr size_t kCycLds = (160 << 10) - 512;       // a compute unit's LDS less the block's own reductions

template <typename T, int P, bool SAME>
struct Cycle {
  static constexpr int S = 2 * P + 1, SS = S * S, NCH = (SS + 15) / 16;
  const CycleArgs<T> &g;
  Global<double> Ainv;  // coarse inverses (their address is loaded first of all)
  char *tab;     // tables (offsets in CycleArg)
  T *cb, *rr;    // patch contributions of the shared rows, right-hand side of the current level
  int j, gid, col;
  T sg;
  T m[NCH], s[NCH];  // stencil of the next row

  template <typename U>
  __device__ __forceinline__ const U *t(int off) const {
    return reinterpret_cast<const U *>(tab + off);
  }
  __device__ __forceinline__ int64_t at(int row) const { return (int64_t)row * g.ldb + col; }
  __device__ __forceinline__ T diag(const CycleArg<T> &L, int i) const { return sg * t<T>(L.o_dM)[i] + t<T>(L.o_dS)[i]; }

  __device__ __forceinline__ void load(const CycleArg<T> &L, int i) {
    const int64_t row = t<int>(L.o_row)[i];
#pragma unroll
    for (int k = 0; k < NCH; ++k) {
      const int tap = min(16 * k + j, SS - 1);
      m[k] = L.stM[row * SS + tap];
      s[k] = L.stS[row * SS + tap];
    }
  }
  // the stencil of this group's first row on level L, ahead of the barrier before rows_apply
  __device__ __forceinline__ void preload(const CycleArg<T> &L) {
    if (gid < L.nrow) load(L, gid);
  }
  // A z of every row this group owns, epi(row, A z); the stencil of the next row is loaded before the
  // arithmetic of the current one
  template <class F>
  __device__ __forceinline__ void rows_apply(const CycleArg<T> &L, const T *z, F epi) {
    for (int i = gid; i < L.nrow; i += kCycGroups) {
      T cm[NCH], cs[NCH];
#pragma unroll
      for (int k = 0; k < NCH; ++k) {
        cm[k] = SAME ? sg * m[k] + s[k] : m[k];
        cs[k] = s[k];
      }
      if (i + kCycGroups < L.nrow) load(L, i + kCycGroups);
      T am = 0, as = 0;
      taps<0>(am, as, cm, cs, z + (i - P * L.n1 - P) * kCycCols + j, L.n1 * kCycCols);
      epi(i, SAME ? am : sg * am + as);
    }
  }
  // row DY of the stencil sum: its values are read first, then one (SAME) or two multiply-adds each
  template <int DY>
  __device__ __forceinline__ void taps(T &am, T &as, const T (&cm)[NCH], const T (&cs)[NCH], const T *z,
                                       int pitch) const {
    if constexpr (DY < S) {
      T x[S];
#pragma unroll
      for (int dx = 0; dx < S; ++dx) x[dx] = z[dx * kCycCols];
      row_taps<DY, 0>(am, as, cm, cs, x);
      taps<DY + 1>(am, as, cm, cs, z + pitch, pitch);
    }
  }
  template <int DY, int DX>
  __device__ __forceinline__ void row_taps(T &am, T &as, const T (&cm)[NCH], const T (&cs)[NCH], const T (&x)[S]) const {
    if constexpr (DX < S) {
      constexpr int tap = DY * S + DX;
      fma_row_bcast<tap % 16, tap % 16 == 0>(am, cm[tap / 16], x[DX]);
      if constexpr (!SAME) fma_row_bcast<tap % 16, tap % 16 == 0>(as, cs[tap / 16], x[DX]);
      row_taps<DY, DX + 1>(am, as, cm, cs, x);
    }
  }
  // every shared unknown this group owns: epi(first, last) over the positions of its copies
  template <class F>
  __device__ __forceinline__ void shared(const CycleArg<T> &L, F epi) const {
    const int *gp = t<int>(L.o_gp);
    for (int q = gid; q < L.ngroups; q += kCycGroups) epi(gp[q], gp[q + 1]);
  }
  __device__ __forceinline__ T contributions(int k0, int k1) const {
    T v = 0;
    for (int k = k0; k < k1; ++k) v += cb[k * kCycCols + j];
    return v;
  }

  // right-hand side: the sum of its patch contributions over the copies
  __device__ __forceinline__ void sum_rhs(const CycleArg<T> &L) const {
    const int *gc = t<int>(L.o_gc);
    shared(L, [&](int k0, int k1) {
      T v = 0;
      for (int k = k0; k < k1; ++k) v += rr[gc[k] * kCycCols + j];
      for (int k = k0; k < k1; ++k) rr[gc[k] * kCycCols + j] = v;
    });
    __syncthreads();
  }
  // z = c2 r / D
  __device__ __forceinline__ void first_step(const CycleArg<T> &L, T *z) const {
    const T c2 = L.cf[(int64_t)L.deg * g.ldb + col];
    for (int i = gid; i < L.nrow; i += kCycGroups) z[i * kCycCols + j] = c2 * rr[i * kCycCols + j] / diag(L, i);
  }
  // step k of the smoothing polynomial: zo holds the iterate before z and takes the new one (prev 0: no
  // previous direction, 1: it is z itself, 2: z - zo); preload and a barrier come first
  __device__ __forceinline__ void smooth(const CycleArg<T> &L, int k, int prev, const T *z, T *zo) {
    const T c1 = prev ? L.cf[(int64_t)k * g.ldb + col] : T(0), c2 = L.cf[(int64_t)(L.deg + k) * g.ldb + col];
    const int *pos = t<int>(L.o_pos), *gc = t<int>(L.o_gc);
    auto step = [&](int i, T Az) {
      const int q = i * kCycCols + j;
      const T zc = z[q], dp = prev == 2 ? zc - zo[q] : (prev == 1 ? zc : T(0));
      zo[q] = zc + (c1 * dp + c2 * ((rr[q] - Az) / diag(L, i)));
    };
    rows_apply(L, z, [&](int i, T Az) {
      const int p = pos[i];
      if (p >= 0) cb[p * kCycCols + j] = Az;
      else step(i, Az);
    });
    __syncthreads();
    shared(L, [&](int k0, int k1) {
      const T v = contributions(k0, k1);
      for (int q = k0; q < k1; ++q) step(gc[q], v);
    });
  }
  // out = r - A z on the owner copies and 0 on the others (one contribution per unknown)
  __device__ __forceinline__ void residual(const CycleArg<T> &L, const T *z, T *out) {
    const int *pos = t<int>(L.o_pos), *gc = t<int>(L.o_gc);
    rows_apply(L, z, [&](int i, T Az) {
      const int p = pos[i];
      if (p >= 0) cb[p * kCycCols + j] = Az;
      else out[i * kCycCols + j] = rr[i * kCycCols + j] - Az;
    });
    __syncthreads();
    shared(L, [&](int k0, int k1) {
      const T v = contributions(k0, k1);
      for (int k = k0; k < k1; ++k) out[gc[k] * kCycCols + j] = k == k0 ? rr[gc[k] * kCycCols + j] - v : T(0);
    });
    __syncthreads();
  }
  // the coarser level's right-hand side P^T a, patch by patch
  __device__ __forceinline__ void restrict_to(const CycleArg<T> &L, const CycleArg<T> &C, const T *a) const {
    const int *rs = t<int>(L.o_rs);
    const T *rc = t<T>(L.o_rc);
    for (int i = gid; i < C.nrow; i += kCycGroups) {
      const int mp = i / (C.n1 * C.n1), iy = (i / C.n1) % C.n1, ix = i % C.n1;
      const T *a0 = a + ((mp * L.n1 + rs[iy]) * L.n1 + rs[ix]) * kCycCols + j;
      T acc = 0;
      for (int l = 0; l < L.rw; ++l) {
        T v = 0;
        for (int k = 0; k < L.rw; ++k) v += rc[iy * L.rw + k] * a0[(k * L.n1 + l) * kCycCols];
        acc += rc[ix * L.rw + l] * v;
      }
      rr[i * kCycCols + j] = acc;
    }
    __syncthreads();
  }
  // z + P zc into z2, and the level's right-hand side back into LDS; z and r from the batch vectors
  __device__ __forceinline__ void prolong_from(const CycleArg<T> &L, const CycleArg<T> &C, const T *zc, T *z2) const {
    const int *ps = t<int>(L.o_ps), *row = t<int>(L.o_row);
    const T *pc = t<T>(L.o_pc);
    for (int i = gid; i < L.nrow; i += kCycGroups) {
      const T zs = L.za[at(row[i])], rs = L.r[at(row[i])];
      const int mp = i / (L.n1 * L.n1), iy = (i / L.n1) % L.n1, ix = i % L.n1;
      const T *c0 = zc + ((mp * C.n1 + ps[iy]) * C.n1 + ps[ix]) * kCycCols + j;
      T acc = 0;
      for (int l = 0; l < L.pw; ++l) {
        T v = 0;
        for (int k = 0; k < L.pw; ++k) v += pc[iy * L.pw + k] * c0[(k * C.n1 + l) * kCycCols];
        acc += pc[ix * L.pw + l] * v;
      }
      z2[i * kCycCols + j] = zs + acc;
      rr[i * kCycCols + j] = rs;
    }
  }
  // z0 = (sigma M0 + S0)^-1 r0 by the rows of the inverse, in FP64
  __device__ __forceinline__ void coarse_solve(const CycleArg<T> &C, double *rhs, double *sol, T *z) const {
    const int *un = t<int>(g.o_gid);
    for (int i = gid; i < C.nrow; i += kCycGroups) rhs[un[i] * kCycCols + j] = (double)rr[i * kCycCols + j];
    __syncthreads();
    // (SAME: the node of the block's first column, for padding columns as well)
    const Global<double> A = Ainv + (size_t)g.node[SAME ? col - j : col] * g.N0 * g.N0;
    for (int i = gid; i < g.N0; i += kCycGroups) {
      const Global<double> Ai = A + (size_t)i * g.N0;
      double acc = 0.0;
      if (SAME) {  // the columns share the node: a chunk of the row per lane, broadcast entry by entry
        for (int c = 0; c < g.N0; c += 16) {
          const double a = Ai[min(c + j, g.N0 - 1)];
          dot16<0>(acc, a, rhs + c * kCycCols + j);
        }
      } else {
#pragma unroll 8
        for (int k = 0; k < g.N0; ++k) acc += Ai[k] * rhs[k * kCycCols + j];
      }
      sol[i * kCycCols + j] = acc;
    }
    __syncthreads();
    for (int i = gid; i < C.nrow; i += kCycGroups) z[i * kCycCols + j] = (T)sol[un[i] * kCycCols + j];
    __syncthreads();
  }
  template <int K>
  __device__ __forceinline__ void dot16(double &acc, double a, const double *x) const {
    if constexpr (K < 16) {
      fma_row_bcast<K, K == 0>(acc, a, x[K * kCycCols]);
      dot16<K + 1>(acc, a, x);
    }
  }
};

template <typename U>
__device__ __forceinline__ void table_copy(char *tab, int off, const U *src, int n) {
  for (int i = threadIdx.x; i < n; i += kCycThreads) reinterpret_cast<U *>(tab + off)[i] = src[i];
}

template <typename T, int P, bool SAME>
__global__ __launch_bounds__(kCycThreads) void k_cycle(CycleArgs<T> g) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  if (g.active && !g.active[blockIdx.x / (CT / kCycCols)]) return;
  const int j = threadIdx.x & 15, gid = threadIdx.x >> 4, col = blockIdx.x * kCycCols + j;
  // columns that have converged (or pad the tile, or never had a load) need no correction; all 16 of
  // them: it is zero, not what an earlier batch left in the buffer (their search direction takes it up,
  // with a step of zero length)
  if (!__syncthreads_or(!g.cs[col].done)) {
    const CycleArg<T> &L = g.lev[g.top];
    T *out = g.top == 0 ? L.za : L.zb;
    for (int i = gid; i < L.nrow; i += kCycGroups) out[(int64_t)L.crow[i] * g.ldb + col] = T(0);
    return;
  }
  const uint64_t inv = (uint64_t)(uintptr_t)*g.Ainv;  // (the same for all threads: in scalar registers)
  const Global<double> Ainv = (Global<double>)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(inv >> 32)) << 32 |
                                               (uint32_t)__builtin_amdgcn_readfirstlane((int)inv));
  double *rhs = reinterpret_cast<double *>(smem), *sol = rhs + g.n0r * kCycCols;
  T *cb = reinterpret_cast<T *>(sol + g.n0r * kCycCols);
  T *z = cb + g.ncb * kCycCols, *z2 = z + g.nrow * kCycCols, *rr = z2 + g.nrow * kCycCols;
  char *tab = reinterpret_cast<char *>(rr + g.nrow * kCycCols);
  // rows before, between and after a level's rows are read with zero coefficients: no stale bits
  for (int i = threadIdx.x; i < (int)((tab - smem) / 4); i += kCycThreads) reinterpret_cast<int *>(smem)[i] = 0;
  for (int l = 0; l <= g.top; ++l) {
    const CycleArg<T> &L = g.lev[l];
    table_copy(tab, L.o_row, L.crow, L.nrow);
    table_copy(tab, L.o_pos, L.cpos, L.nrow);
    table_copy(tab, L.o_gp, L.gp, L.ngroups + 1);
    table_copy(tab, L.o_gc, L.gc, L.ncopies);
    for (int i = threadIdx.x; i < L.nrow; i += kCycThreads) {
      const int row = L.crow[i];
      reinterpret_cast<T *>(tab + L.o_dM)[i] = L.dM[row];
      reinterpret_cast<T *>(tab + L.o_dS)[i] = L.dS[row];
      if (l == 0) reinterpret_cast<int *>(tab + g.o_gid)[i] = g.rgid[row];
    }
    if (l > 0) {
      const int n1c = g.lev[l - 1].n1;
      table_copy(tab, L.o_rs, L.rs, n1c);
      table_copy(tab, L.o_rc, L.rcoef, n1c * L.rw);
      table_copy(tab, L.o_ps, L.ps, L.n1);
      table_copy(tab, L.o_pc, L.pcoef, L.n1 * L.pw);
    }
  }
  __syncthreads();
  Cycle<T, P, SAME> c{g, Ainv, tab, cb, rr, j, gid, col, g.sig[col]};
  auto flip = [&] {
    T *x = z;
    z = z2;
    z2 = x;
  };
  {
    const CycleArg<T> &L = g.lev[g.top];
    const int *row = c.template t<int>(L.o_row);
    for (int i = gid; i < L.nrow; i += kCycGroups) {
      const int64_t q = c.at(row[i]);
      rr[i * kCycCols + j] = g.rfine ? (T)g.rfine[q] : L.r[q];
    }
    __syncthreads();
  }
  for (int l = g.top; l >= 1; --l) {
    const CycleArg<T> &L = g.lev[l];
    const bool fine = g.rfine && l == g.top;
    if (!fine) c.sum_rhs(L);
    // kept for the way back up
    const int *row = c.template t<int>(L.o_row);
    if (!fine || sizeof(T) == 4)
      for (int i = gid; i < L.nrow; i += kCycGroups) L.r[c.at(row[i])] = rr[i * kCycCols + j];
    c.first_step(L, z);
    c.preload(L);
    __syncthreads();
    for (int k = 1; k < L.deg; ++k) {
      c.smooth(L, k, k == 1 ? 1 : 2, z, z2);
      c.preload(L);
      __syncthreads();
      flip();
    }
    for (int i = gid; i < L.nrow; i += kCycGroups) L.za[c.at(row[i])] = z[i * kCycCols + j];
    c.residual(L, z, z2);
    c.restrict_to(L, g.lev[l - 1], z2);
  }
  c.sum_rhs(g.lev[0]);
  c.coarse_solve(g.lev[0], rhs, sol, z);
  for (int l = 1; l <= g.top; ++l) {
    const CycleArg<T> &L = g.lev[l];
    c.prolong_from(L, g.lev[l - 1], z, z2);
    flip();
    for (int k = 0; k < L.deg; ++k) {
      c.preload(L);
      __syncthreads();
      c.smooth(L, k, k == 0 ? 0 : 2, z, z2);
      flip();
    }
    __syncthreads();
  }
  const CycleArg<T> &L = g.lev[g.top];
  const int *row = c.template t<int>(L.o_row);
  T *out = g.top == 0 ? L.za : L.zb;
  for (int i = gid; i < L.nrow; i += kCycGroups) out[c.at(row[i])] = z[i * kCycCols + j];
}

// LDS layout of levels 0 .. top: two FP64 vectors of the coarsest level (rounded up to whole chunks of its
// matrix rows), the shared rows' contributions (at least the rows that taps may read below the
// iterate), two iterates and the right-hand side of the largest level, the tables of every level
template <typename T>
size_t cycle_layout(CycleArgs<T> &g) {
  int off = 0;
  auto take = [&](int n, int bytes) {
    const int o = off;
    off += (n * bytes + 15) / 16 * 16;
    return o;
  };
  g.n0r = (g.N0 + 15) / 16 * 16;
  g.ncb = g.nrow = 0;
  for (int l = 0; l <= g.top; ++l) {
    CycleArg<T> &L = g.lev[l];
    g.ncb = std::max(g.ncb, std::max(L.ncopies, g.p * L.n1 + g.p));
    g.nrow = std::max(g.nrow, std::max(L.nrow, g.p * L.n1 + g.p));
    L.o_row = take(L.nrow, 4);
    L.o_pos = take(L.nrow, 4);
    L.o_dM = take(L.nrow, sizeof(T));
    L.o_dS = take(L.nrow, sizeof(T));
    L.o_gp = take(L.ngroups + 1, 4);
    L.o_gc = take(L.ncopies, 4);
    if (l == 0) {
      g.o_gid = take(L.nrow, 4);
    } else {
      const int n1c = g.lev[l - 1].n1;
      L.o_rs = take(n1c, 4);
      L.o_rc = take(n1c * L.rw, sizeof(T));
      L.o_ps = take(L.n1, 4);
      L.o_pc = take(L.n1 * L.pw, sizeof(T));
    }
  }
  g.lds = (size_t)kCycCols * (2 * g.n0r * sizeof(double) + ((size_t)g.ncb + 3 * (size_t)g.nrow) * sizeof(T)) + off;
  return g.lds;
}
template size_t cycle_layout<double>(CycleArgs<double> &);
template size_t cycle_layout<float>(CycleArgs<float> &);

bool cycle_fits(size_t lds) { return lds <= kCycLds; }

template <typename T, int P, bool SAME>
static void launch_cycle(const CycleArgs<T> &g, int ntiles, hipStream_t s) {
  raise_lds(reinterpret_cast<const void *>(&k_cycle<T, P, SAME>), kCycLds);
  hipLaunchKernelGGL((k_cycle<T, P, SAME>), dim3(ntiles * (CT / kCycCols)), dim3(kCycThreads), (unsigned)g.lds, s, g);
  HIPCHK(hipGetLastError());
}

template <typename T>
void coarse_cycle(const CycleArgs<T> &g, int ntiles, bool same16, hipStream_t s) {
  if (!cycle_fits(g.lds)) fail(GF_EUNSUPPORTED, "coarse levels exceed the block's LDS");
  switch (g.p) {
#define GF_CY(PP)                                                                                \
  case PP:                                                                                       \
    same16 ? launch_cycle<T, PP, true>(g, ntiles, s) : launch_cycle<T, PP, false>(g, ntiles, s); \
    break;
    GF_CY(1) GF_CY(2) GF_CY(3) GF_CY(4) GF_CY(5)
#undef GF_CY
    default: fail(GF_EUNSUPPORTED, "degree out of range");
  }
}
template void coarse_cycle<double>(const CycleArgs<double> &, int, bool, hipStream_t);
template void coarse_cycle<float>(const CycleArgs<float> &, int, bool, hipStream_t);

}  // namespace gf

// Point evaluation of spline fields, its transpose, and the per-sample accumulation of the
// kappa-gradient terms.
//
// A field of S^0_{j,p} restricted to patch m is the tensor spline sum c[m,iy,ix] b_ix(s) b_iy(t)
// (Sec. 2.3, Sec. 3.1); its value at the surface point F_m(s,t) is that sum, so evaluation at a set of
// points is a sparse matrix Phi with (p+1)^2 entries per point.  The basis values come from the
// triangular Cox-de Boor scheme on the open dyadic knot vector (p+1-fold end knots, interior knots
// i 2^-j), evaluated on the device for every point.
#include "gf_internal.h"
#include "k_solve.h"

#include <algorithm>
#include <type_traits>

namespace gf {

// knot i of the open uniform knot vector with nel elements and degree p
__device__ __forceinline__ double knot_at(int i, int p, int nel) {
  const int k = min(max(i - p, 0), nel);
  return (double)k / (double)nel;
}

// The element containing u (the last one for u = 1) and the P+1 B-splines that are nonzero on it: values into
// N[0..P] for the functions e..e+P; returns e.
__device__ __forceinline__ int element_of(double u, int nel) { return min(max((int)floor(u * nel), 0), nel - 1); }
template <int P>
__device__ __forceinline__ int span_basis(double u, int nel, double (&N)[P + 1]) {
  const int e = element_of(u, nel);
  const int span = e + P;  // knot interval [knot(span), knot(span + 1))
  double left[P + 1], right[P + 1];
  N[0] = 1.0;
#pragma unroll
  for (int j = 1; j <= P; ++j) {
    left[j] = u - knot_at(span + 1 - j, P, nel);
    right[j] = knot_at(span + j, P, nel) - u;
    double carry = 0.0;
#pragma unroll
    for (int r = 0; r < j; ++r) {
      const double den = right[r + 1] + left[j - r];
      const double t = den != 0.0 ? N[r] / den : 0.0;
      N[r] = carry + right[r + 1] * t;
      carry = left[j - r] * t;
    }
    N[j] = carry;
  }
  return e;
}

struct EvalGeom {
  int nel, W, n1, N, npts, nvec, ngroups;
};

// flag |= 1 for a patch index, 2 for a parameter out of range
__global__ __launch_bounds__(256) void k_check_points(int npts, int npatch, const int *__restrict__ patch,
                                                      const double *__restrict__ st, int *flag) {
  int bad = 0;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < npts; i += gridDim.x * 256) {
    if (patch[i] < 0 || patch[i] >= npatch) bad |= 1;
    for (int c = 0; c < 2; ++c)
      if (!(st[2 * i + c] >= 0.0 && st[2 * i + c] <= 1.0)) bad |= 2;
  }
  if (bad) atomicOr(flag, bad);
}

// vals[v][i] = sum over the (P+1)^2 basis functions of point i of B(s_i, t_i) u[v][gid], one thread per point and
// vector: the loads of a point's coefficients are its latency, so the vectors run side by side (one thread
// per point, its basis in scratch memory and the vectors one after the other: 72 us for 1000 points of 16
// fields on degree 3, 64 x 64; 4.7 us so)
template <int P>
__global__ __launch_bounds__(256) void k_eval(EvalGeom g, const int *__restrict__ patch, const double *__restrict__ st,
                                              const int *__restrict__ row_gid, const double *__restrict__ u,
                                              double *__restrict__ vals) {
  const int i = blockIdx.x * 64 + (threadIdx.x & 63), v = blockIdx.y * 4 + (threadIdx.x >> 6);
  if (i >= g.npts || v >= g.nvec) return;
  double bs[P + 1], bt[P + 1];
  const int ex = span_basis<P>(st[2 * i], g.nel, bs);
  const int ey = span_basis<P>(st[2 * i + 1], g.nel, bt);
  const int *gid = row_gid + (int64_t)patch[i] * g.W * g.W + (int64_t)(ey + P) * g.W + (ex + P);
  const double *uv = u + (int64_t)v * g.N;
  double acc = 0.0;
#pragma unroll
  for (int a = 0; a <= P; ++a) {
    double ra = 0.0;
#pragma unroll
    for (int b = 0; b <= P; ++b) ra += bs[b] * uv[gid[a * g.W + b]];
    acc += bt[a] * ra;
  }
  vals[(int64_t)v * g.npts + i] = acc;
}

// The transpose Phi^T r without atomics on the values.  The points are sorted by element (counts and an
// exclusive scan; within an element by point number, from each point's rank among the element's points),
// then every coefficient sums over its copies, the elements of its support and their points in that order:
// the result does not depend on the scheduling and is the same bit for bit on every run.  (The lists were
// built on the host before: points copied back, a table of N + 1 entries filled and sent, some 200 us for 1000
// points.)
constexpr int kScan = 1024;  // elements per block of the scan

__global__ __launch_bounds__(256) void k_bin_points(EvalGeom g, const int *__restrict__ patch,
                                                    const double *__restrict__ st, int *__restrict__ cnt,
                                                    int *__restrict__ elem, int *__restrict__ slot) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= g.npts) return;
  const int e = (patch[i] * g.nel + element_of(st[2 * i + 1], g.nel)) * g.nel + element_of(st[2 * i], g.nel);
  elem[i] = e;
  slot[i] = atomicAdd(&cnt[e], 1);
}

// off[i] = exclusive sum within the block of 1024, sums[block] its total (off may be cnt)
__global__ __launch_bounds__(kScan) void k_scan_blocks(const int *cnt, int n, int *off, int *sums) {
  __shared__ int part[kScan / 64];
  const int i = blockIdx.x * kScan + threadIdx.x, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int c = i < n ? cnt[i] : 0;
  int x = c;
  for (int d = 1; d < 64; d *= 2) {
    const int y = __shfl_up(x, d);
    if (lane >= d) x += y;
  }
  if (lane == 63) part[w] = x;
  __syncthreads();
  int base = 0;
  for (int k = 0; k < w; ++k) base += part[k];
  if (i < n) off[i] = base + x - c;
  if (threadIdx.x == kScan - 1) sums[blockIdx.x] = base + x;
}
// exclusive sums of the block totals, one block
__global__ __launch_bounds__(kScan) void k_scan_sums(int *sums, int n) {
  __shared__ int part[kScan / 64];
  __shared__ int carry;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (threadIdx.x == 0) carry = 0;
  for (int i0 = 0; i0 < n; i0 += kScan) {
    __syncthreads();
    const int i = i0 + threadIdx.x, c = i < n ? sums[i] : 0;
    int x = c;
    for (int d = 1; d < 64; d *= 2) {
      const int y = __shfl_up(x, d);
      if (lane >= d) x += y;
    }
    if (lane == 63) part[w] = x;
    __syncthreads();
    int base = carry;
    for (int k = 0; k < w; ++k) base += part[k];
    if (i < n) sums[i] = base + x - c;
    __syncthreads();
    if (threadIdx.x == kScan - 1) carry = base + x;
  }
}
__device__ __forceinline__ int bin_start(const int *off, const int *sums, int e) { return off[e] + sums[e / kScan]; }

__global__ __launch_bounds__(256) void k_fill_bins(int npts, const int *__restrict__ elem, const int *__restrict__ slot,
                                                   const int *__restrict__ off, const int *__restrict__ sums,
                                                   int *__restrict__ list) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < npts) list[bin_start(off, sums, elem[i]) + slot[i]] = i;
}

// every bin in point order, the element columns of the points beside it, and the basis products of every point,
// w[i][a (P+1) + b] = B_a(t_i) B_b(s_i)
template <int P>
__global__ __launch_bounds__(256) void k_rank_points(EvalGeom g, const double *__restrict__ st,
                                                     const int *__restrict__ elem, const int *__restrict__ off,
                                                     const int *__restrict__ sums, const int *__restrict__ list,
                                                     int *__restrict__ sorted, int *__restrict__ column,
                                                     double *__restrict__ w) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= g.npts) return;
  const int e = elem[i], q0 = bin_start(off, sums, e), q1 = bin_start(off, sums, e + 1);
  int rank = 0;
#pragma unroll 8
  for (int q = q0; q < q1; ++q) rank += list[q] < i ? 1 : 0;
  sorted[q0 + rank] = i;
  column[q0 + rank] = e % g.nel;
  double bs[P + 1], bt[P + 1];
  span_basis<P>(st[2 * i], g.nel, bs);
  span_basis<P>(st[2 * i + 1], g.nel, bt);
#pragma unroll
  for (int a = 0; a <= P; ++a)
#pragma unroll
    for (int b = 0; b <= P; ++b) w[(int64_t)i * (P + 1) * (P + 1) + a * (P + 1) + b] = bt[a] * bs[b];
}

// out[v][gid], VC vectors at a time; unknowns off the patch boundary by their number, the others by their group of
// copies (numbers N .. N + ngroups); coefficients no point touches get 0.  WAVE false: a thread per
// coefficient walks its points, unless points are bunched: where the longest list of a wavefront's coefficients
// is longer than twice the steps that all 64 lanes need for its lists one after the other, they do that instead.
// WAVE true: a wavefront per coefficient -- for meshes with many points per element, whose few coefficients leave
// the chip idle otherwise (see launch_eval_adjoint).  Lanes' sums are added in a fixed tree.  The walk waits for
// its loads: all vectors of a point are loaded together (past the last vector: the last one again).
// 20000 points in one element of 64 x 64, degree 3, 16 vectors: a call took 60.5 ms with each thread walking its lists
// element by element and a branch around every vector's load, 1.1 so; 12000 points spread over the mesh 144 -> 87 us.
template <int P, bool WAVE, int VC>
__global__ __launch_bounds__(256) void k_eval_gather(EvalGeom g, const int *__restrict__ off, const int *__restrict__ sums,
                                                     const int *__restrict__ sorted, const int *__restrict__ column,
                                                     const double *__restrict__ w, const double *__restrict__ r,
                                                     double *__restrict__ out,
                                                     const int *__restrict__ orow, const int *__restrict__ rgid,
                                                     const int *__restrict__ gp, const int *__restrict__ gr) {
  constexpr int NB = P + 1;
  const int id = WAVE ? blockIdx.x * 4 + (threadIdx.x >> 6) : blockIdx.x * 256 + threadIdx.x;
  const int lane = threadIdx.x & 63;
  const int v0 = blockIdx.y * VC, last = g.nvec - 1 - v0;
  // row(patch, ly, lx) of every copy of coefficient c
  auto copies = [&](int c, auto row) {
    auto one = [&](int rw) {
      const int m = rw / (g.W * g.W), q = rw - m * g.W * g.W;
      row(m, q / g.W - P, q % g.W - P);
    };
    if (c < g.N) {
      one(orow[c]);
    } else {
      for (int k = gp[c - g.N], k1 = gp[c - g.N + 1]; k < k1; ++k) one(gr[k]);
    }
  };
  // acc[v] += every step-th point of coefficient c from the first on: the elements of a row are neighbours in the
  // list, so that lanes with different elements of the row walk theirs at the same time
  auto walk = [&](int c, int first, int step, double (&acc)[VC]) {
    copies(c, [&](int m, int ly, int lx) {
      const int x0 = max(lx - P, 0), x1 = min(lx, g.nel - 1);
      for (int b = 0; b < NB; ++b) {
        const int ey = ly - b;
        if (ey < 0 || ey >= g.nel) continue;
        const int e = (m * g.nel + ey) * g.nel, q1 = bin_start(off, sums, e + x1 + 1);
        auto take = [&](int k, auto count) {  // that many points, loaded together
          constexpr int K = decltype(count)::value;
          double wi[K], rv[K][VC];
#pragma unroll
          for (int u = 0; u < K; ++u) {
            const int i = sorted[k + u * step], a = lx - column[k + u * step];
            wi[u] = w[(int64_t)i * NB * NB + b * NB + a];
#pragma unroll
            for (int v = 0; v < VC; ++v) rv[u][v] = r[(int64_t)(v0 + min(v, last)) * g.npts + i];
          }
#pragma unroll
          for (int u = 0; u < K; ++u)
#pragma unroll
            for (int v = 0; v < VC; ++v) acc[v] += wi[u] * rv[u][v];
        };
        int k = bin_start(off, sums, e + x0) + first;
        for (; k + 3 * step < q1; k += 4 * step) take(k, std::integral_constant<int, 4>());
        for (; k < q1; k += step) take(k, std::integral_constant<int, 1>());
      }
    });
  };
  auto over_lanes = [&](double (&acc)[VC]) {
#pragma unroll
    for (int v = 0; v < VC; ++v)
      for (int d = 32; d > 0; d /= 2) acc[v] += __shfl_xor(acc[v], d);
  };
  bool on = id < g.N + g.ngroups;  // (the lanes of a wavefront stay together)
  if (on && id < g.N) {
    const int row = orow[id], q = row % (g.W * g.W), ly = q / g.W - P, lx = q % g.W - P;
    on = lx != 0 && lx != g.n1 - 1 && ly != 0 && ly != g.n1 - 1;
  }
  double acc[VC];
#pragma unroll
  for (int v = 0; v < VC; ++v) acc[v] = 0.0;
  if (WAVE) {
    if (!on) return;
    walk(id, lane, 64, acc);
    over_lanes(acc);
    on = lane == 0;
  } else {
    int n = 0;  // points of this lane's coefficient
    if (on)
      copies(id, [&](int m, int ly, int lx) {
        const int x0 = max(lx - P, 0), x1 = min(lx, g.nel - 1);
        for (int ey = max(ly - P, 0); ey <= min(ly, g.nel - 1); ++ey) {
          const int e = (m * g.nel + ey) * g.nel;
          n += bin_start(off, sums, e + x1 + 1) - bin_start(off, sums, e + x0);
        }
      });
    int most = n, steps = n > 0 ? n / 64 + NB : 0;  // (a list per row)
    for (int d = 32; d > 0; d /= 2) {
      most = max(most, __shfl_xor(most, d));
      steps += __shfl_xor(steps, d);
    }
    if (most > steps) {
      for (unsigned long long todo = __ballot(n > 0); todo; todo &= todo - 1) {
        const int l = __builtin_ctzll(todo);
        double t[VC];
#pragma unroll
        for (int v = 0; v < VC; ++v) t[v] = 0.0;
        walk(__shfl(id, l), lane, 64, t);
        over_lanes(t);
        if (lane == l)
#pragma unroll
          for (int v = 0; v < VC; ++v) acc[v] = t[v];
      }
    } else if (n > 0) {
      walk(id, 0, 1, acc);
    }
  }
  if (!on) return;
  const int gid = id < g.N ? id : rgid[gr[gp[id - g.N]]];
#pragma unroll
  for (int v = 0; v < VC; ++v)
    if (v <= last) out[(int64_t)(v0 + v) * g.N + gid] = acc[v];
}

void launch_check_points(const Level &L, int npts, const int *patch, const double *st, int *flag, hipStream_t s) {
  HIPCHK(hipMemsetAsync(flag, 0, sizeof(int), s));
  hipLaunchKernelGGL(k_check_points, dim3(std::min((npts + 255) / 256, 1024)), dim3(256), 0, s, npts, L.npatch, patch, st,
                     flag);
  HIPCHK(hipGetLastError());
}

#define GF_DEGREES(DO)                                                                      \
  switch (L.p) {                                                                            \
    case 1: DO(1); break;                                                                   \
    case 2: DO(2); break;                                                                   \
    case 3: DO(3); break;                                                                   \
    case 4: DO(4); break;                                                                   \
    case 5: DO(5); break;                                                                   \
    default: fail(GF_EUNSUPPORTED, "degree out of range");                                  \
  }

static EvalGeom eval_geom(const Level &L, int npts, int nvec) {
  return EvalGeom{L.nel, L.W, L.n1, L.N, npts, nvec, L.ngroups};
}

void launch_eval(const Level &L, int npts, const int *patch, const double *st, int nvec, const double *u,
                 double *vals, hipStream_t s) {
  if (npts == 0 || nvec == 0) return;
  for (int v0 = 0; v0 < nvec; v0 += 4 * 16384) {  // (the grid's second dimension)
    const int nv = std::min(nvec - v0, 4 * 16384);
    const EvalGeom g = eval_geom(L, npts, nv);
#define GF_EV(P)                                                                                                  \
  hipLaunchKernelGGL(k_eval<P>, dim3((npts + 63) / 64, (nv + 3) / 4), dim3(256), 0, s, g, patch, st, L.row_gid.p, \
                     u + (int64_t)v0 * L.N, vals + (int64_t)v0 * npts)
    GF_DEGREES(GF_EV)
#undef GF_EV
    HIPCHK(hipGetLastError());
  }
}

size_t eval_adjoint_ints(const Level &L, int npts) {
  const size_t ne = (size_t)L.npatch * L.nel * L.nel + 1;
  return ne + (ne + kScan - 1) / kScan + 4 * (size_t)npts;
}

void launch_eval_adjoint(const Level &L, int npts, const int *patch, const double *st, int *iw, double *w, int nvec,
                         const double *r, double *out, hipStream_t s) {
  if (nvec == 0) return;
  const int ne = L.npatch * L.nel * L.nel + 1, nsum = (ne + kScan - 1) / kScan;  // (a last, empty bin)
  int *off = iw, *sums = off + ne, *elem = sums + nsum, *slot = elem + npts, *list = slot + npts, *sorted = list + npts;
  const EvalGeom g0 = eval_geom(L, npts, nvec);
  HIPCHK(hipMemsetAsync(off, 0, ne * sizeof(int), s));
  const dim3 gp((npts + 255) / 256);
  if (npts > 0) hipLaunchKernelGGL(k_bin_points, gp, dim3(256), 0, s, g0, patch, st, off, elem, slot);
  hipLaunchKernelGGL(k_scan_blocks, dim3(nsum), dim3(kScan), 0, s, off, ne, off, sums);
  hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(kScan), 0, s, sums, nsum);
  if (npts > 0) hipLaunchKernelGGL(k_fill_bins, gp, dim3(256), 0, s, npts, elem, slot, off, sums, list);
  for (int v0 = 0; v0 < nvec; v0 += 4 * 16384) {  // (the grid's second dimension)
    const int nv = std::min(nvec - v0, 4 * 16384);
    const EvalGeom g = eval_geom(L, npts, nv);
    // a wavefront per coefficient from one point an element on (16 vectors, a thread / a wavefront per coefficient:
    // 20000 points on degree 3, 32 x 32 elements, 137 / 107 us a call, 12000 on 64 x 64 87 / 171; just above the line
    // 600 on degree 2, 8 x 8, 90 / 65, but 25000 on degree 3, 64 x 64, 105 / 192)
    const bool wave = npts >= ne, one = nv == 1;
    const int vc = one ? 1 : wave ? 4 : 8;
    const dim3 gg(wave ? (L.N + L.ngroups + 3) / 4 : (L.N + L.ngroups + 255) / 256, (nv + vc - 1) / vc);
#define GF_EA(P)                                                                                                       \
  do {                                                                                                                 \
    if (npts > 0 && v0 == 0)                                                                                           \
      hipLaunchKernelGGL(k_rank_points<P>, gp, dim3(256), 0, s, g, st, elem, off, sums, list, sorted, slot, w);        \
    auto gather = wave ? (one ? k_eval_gather<P, true, 1> : k_eval_gather<P, true, 4>)                                 \
                       : (one ? k_eval_gather<P, false, 1> : k_eval_gather<P, false, 8>);                              \
    hipLaunchKernelGGL(gather, gg, dim3(256), 0, s, g, off, sums, sorted, slot, w, r + (int64_t)v0 * npts,             \
                       out + (int64_t)v0 * L.N, L.owner_row.p, L.row_gid.p, L.grp_ptr.p, L.grp_rows.p);                \
  } while (0)
    GF_DEGREES(GF_EA)
#undef GF_EA
    HIPCHK(hipGetLastError());
  }
}
#undef GF_DEGREES

// acc[s] += sum_k w[k] dots[k * nsamp + s], k ascending (one thread per sample)
__global__ void k_grad_accum(const double *__restrict__ dots, const double *__restrict__ w, int K, int nsamp,
                             double *acc) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= nsamp) return;
  double t = 0.0;
  for (int k = 0; k < K; ++k) t += w[k] * dots[(int64_t)k * nsamp + s];
  acc[s] += t;
}

// out[s] = c * acc[s]
__global__ void k_grad_scale(const double *__restrict__ acc, int nsamp, double c, double *out) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s < nsamp) out[s] = c * acc[s];
}

void grad_accum(const double *dots, const double *w, int K, int nsamp, double *acc, hipStream_t s) {
  hipLaunchKernelGGL(k_grad_accum, dim3((nsamp + 255) / 256), dim3(256), 0, s, dots, w, K, nsamp, acc);
  HIPCHK(hipGetLastError());
}

void grad_scale(const double *acc, int nsamp, double c, double *out, hipStream_t s) {
  hipLaunchKernelGGL(k_grad_scale, dim3((nsamp + 255) / 256), dim3(256), 0, s, acc, nsamp, c, out);
  HIPCHK(hipGetLastError());
}

}  // namespace gf

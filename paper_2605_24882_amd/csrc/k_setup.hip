// Setup kernels: metric terms at the Gauss points, the matrix-free sum-factorised
// operator application, stencil extraction by probing, diagonals, the element-wise
// white-noise load and the coarse-level Cholesky factors.
#include "gf_internal.h"
#include "k_solve.h"
#include "k_stencil.h"

namespace gf {

// cube-face frames of the six patches (same table as the host's kPatchFrames)
__constant__ int c_frames[6][4] = {{0, 1, 1, 2}, {0, -1, 2, 1}, {1, 1, 2, 0},
                                   {1, -1, 0, 2}, {2, 1, 0, 1}, {2, -1, 1, 0}};

// Surface point and its parameter derivatives for patch m at (s, t) (Sec. 2.2 maps).
// xh = v/|v| has d xh = (dv - xh (xh . dv))/|v|; the perturbed surface r(xh) xh with
// r = 1 + amp sin(3x) sin(2y) cos(z) has d(r xh) = (grad r . d xh) xh + r d xh.
__device__ void surface_derivs(int m, double s, double t, double amp, double Fs[3], double Ft[3]) {
  const int fa = c_frames[m][0], fs = c_frames[m][1], aa = c_frames[m][2], ba = c_frames[m][3];
  double v[3], vs[3] = {0, 0, 0}, vt[3] = {0, 0, 0};
  v[fa] = (double)fs;
  v[aa] = 2.0 * s - 1.0;
  v[ba] = 2.0 * t - 1.0;
  vs[aa] = 2.0;
  vt[ba] = 2.0;
  const double nv = sqrt(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
  double xh[3], xs[3], xt[3];
  for (int i = 0; i < 3; ++i) xh[i] = v[i] / nv;
  const double ps = xh[0] * vs[0] + xh[1] * vs[1] + xh[2] * vs[2];
  const double pt = xh[0] * vt[0] + xh[1] * vt[1] + xh[2] * vt[2];
  for (int i = 0; i < 3; ++i) {
    xs[i] = (vs[i] - xh[i] * ps) / nv;
    xt[i] = (vt[i] - xh[i] * pt) / nv;
  }
  if (amp == 0.0) {
    for (int i = 0; i < 3; ++i) { Fs[i] = xs[i]; Ft[i] = xt[i]; }
    return;
  }
  const double X = xh[0], Y = xh[1], Z = xh[2];
  const double r = 1.0 + amp * sin(3.0 * X) * sin(2.0 * Y) * cos(Z);
  const double gr[3] = {3.0 * amp * cos(3.0 * X) * sin(2.0 * Y) * cos(Z),
                        2.0 * amp * sin(3.0 * X) * cos(2.0 * Y) * cos(Z), -amp * sin(3.0 * X) * sin(2.0 * Y) * sin(Z)};
  const double rs = gr[0] * xs[0] + gr[1] * xs[1] + gr[2] * xs[2];
  const double rt = gr[0] * xt[0] + gr[1] * xt[1] + gr[2] * xt[2];
  for (int i = 0; i < 3; ++i) {
    Fs[i] = rs * xh[i] + r * xs[i];
    Ft[i] = rt * xh[i] + r * xt[i];
  }
}

// ---- rational tensor-product B-spline patches (Sec. 2.2: the patch maps of a NURBS surface)
constexpr int kMaxGeomDeg = 4;

// knot span i with U[i] <= u < U[i+1] among the n basis functions of degree d (open knot vector
// U[0 .. n+d]); u = U[n] falls into the last non-empty span
__device__ int nurbs_span(const double *U, int n, int d, double u) {
  if (u >= U[n]) {
    int i = n - 1;
    while (i > d && U[i] >= U[i + 1]) --i;
    return i;
  }
  int lo = d, hi = n;  // U[lo] <= u < U[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) / 2;
    if (u < U[mid]) hi = mid;
    else lo = mid;
  }
  return lo;
}

// values N[j] and first derivatives dN[j] of the d+1 basis functions span-d+j (j = 0..d) at u, by
// the Cox-de Boor recursion over the degrees 0..d (terms with a vanishing denominator dropped)
__device__ void nurbs_basis(const double *U, int span, int d, double u, double *N, double *dN) {
  double tri[kMaxGeomDeg + 1][kMaxGeomDeg + 1];
  tri[0][0] = 1.0;
  for (int k = 1; k <= d; ++k)
    for (int j = 0; j <= k; ++j) {
      const int i = span - k + j;
      double v = 0.0;
      if (j > 0) {
        const double den = U[i + k] - U[i];
        if (den > 0.0) v += (u - U[i]) / den * tri[k - 1][j - 1];
      }
      if (j < k) {
        const double den = U[i + k + 1] - U[i + 1];
        if (den > 0.0) v += (U[i + k + 1] - u) / den * tri[k - 1][j];
      }
      tri[k][j] = v;
    }
  for (int j = 0; j <= d; ++j) {
    N[j] = tri[d][j];
    const int i = span - d + j;
    double v = 0.0;
    if (d > 0) {
      if (j > 0) {
        const double den = U[i + d] - U[i];
        if (den > 0.0) v += d * tri[d - 1][j - 1] / den;
      }
      if (j < d) {
        const double den = U[i + d + 1] - U[i + 1];
        if (den > 0.0) v -= d * tri[d - 1][j] / den;
      }
    }
    dN[j] = v;
  }
}

// F = P / w with P = sum N_a(s) N_b(t) w_ab X_ab, w = sum N_a N_b w_ab; dF = (dP - F dw) / w
__device__ void nurbs_derivs(const SurfaceArgs &g, int m, double s, double t, double Fs[3], double Ft[3]) {
  const int *pi = g.pinfo + 5 * m;
  const int ns = pi[0], nt = pi[1];
  const double *U = g.knots + pi[2], *V = g.knots + pi[3], *C = g.ctrl + 4 * (int64_t)pi[4];
  const int su = nurbs_span(U, ns, g.du, s), sv = nurbs_span(V, nt, g.dv, t);
  double Nu[kMaxGeomDeg + 1], dNu[kMaxGeomDeg + 1], Nv[kMaxGeomDeg + 1], dNv[kMaxGeomDeg + 1];
  nurbs_basis(U, su, g.du, s, Nu, dNu);
  nurbs_basis(V, sv, g.dv, t, Nv, dNv);
  double P[4] = {0, 0, 0, 0}, Ps[4] = {0, 0, 0, 0}, Pt[4] = {0, 0, 0, 0};  // homogeneous (x w, y w, z w, w)
  for (int b = 0; b <= g.dv; ++b)
    for (int a = 0; a <= g.du; ++a) {
      const double *c = C + 4 * ((int64_t)(sv - g.dv + b) * ns + (su - g.du + a));
      const double h[4] = {c[0] * c[3], c[1] * c[3], c[2] * c[3], c[3]};
      for (int k = 0; k < 4; ++k) {
        P[k] += Nu[a] * Nv[b] * h[k];
        Ps[k] += dNu[a] * Nv[b] * h[k];
        Pt[k] += Nu[a] * dNv[b] * h[k];
      }
    }
  for (int k = 0; k < 3; ++k) {
    const double F = P[k] / P[3];
    Fs[k] = (Ps[k] - F * Ps[3]) / P[3];
    Ft[k] = (Pt[k] - F * Pt[3]) / P[3];
  }
}

// m = w a, G = w a K^-1 at every Gauss point (Sec. 3.2: K first fundamental form,
// a = sqrt(det K)); w is the tensor Gauss weight of the element (area 1/nel^2).
__global__ void k_metric(double *metric, int nel, int q, SurfaceArgs g, const double *gx, const double *gw) {
  const int64_t total = (int64_t)g.npatch * nel * nel * q * q;
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= total) return;
  int64_t t = id;
  const int qx = t % q; t /= q;
  const int qy = t % q; t /= q;
  const int ex = t % nel; t /= nel;
  const int ey = t % nel; t /= nel;
  const int m = (int)t;
  const double s = (ex + gx[qx]) / nel, tt = (ey + gx[qy]) / nel;
  double Fs[3], Ft[3];
  if (g.kind == SURF_NURBS) nurbs_derivs(g, m, s, tt, Fs, Ft);
  else surface_derivs(m, s, tt, g.amp, Fs, Ft);
  const double k11 = Fs[0] * Fs[0] + Fs[1] * Fs[1] + Fs[2] * Fs[2];
  const double k12 = Fs[0] * Ft[0] + Fs[1] * Ft[1] + Fs[2] * Ft[2];
  const double k22 = Ft[0] * Ft[0] + Ft[1] * Ft[1] + Ft[2] * Ft[2];
  const double det = k11 * k22 - k12 * k12;
  const double a = sqrt(det);
  const double w = gw[qx] * gw[qy] / ((double)nel * nel);
  double *o = metric + id * 4;
  o[0] = w * a;
  o[1] = w * a * k22 / det;
  o[2] = -w * a * k12 / det;
  o[3] = w * a * k11 / det;
}

void launch_metric(const Level &L, const SurfaceArgs &g, const double *gx, const double *gw, hipStream_t s) {
  const int64_t total = (int64_t)g.npatch * L.nel * L.nel * L.q * L.q;
  hipLaunchKernelGGL(k_metric, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, L.metric.p, L.nel, L.q, g,
                     gx, gw);
  HIPCHK(hipGetLastError());
}

// ------------------------------------------------------------------ matrix-free apply
// y = (ca M + cb S) x per column, patch by patch (no interface sum), evaluating the element integrals of
// eq. mass / eq. stiffness at the Q x Q Gauss points on the fly (sum factorisation).  Per element
// (NB = p+1 basis functions per direction, coefficients c[b][a], b along t, a along s):
//   U0[b][qx] = sum_a c[b][a] Bx[qx][a],  U1[b][qx] = sum_a c[b][a] Dx[qx][a]
//   u = sum_b U0 By, us = sum_b U1 By, ut = sum_b U0 Dy                        (at each qy, qx)
//   v = ca m u,  gs = cb (G11 us + G12 ut),  gt = cb (G12 us + G22 ut)
//   V0[b][qx] = sum_qy v By + gt Dy,  V1[b][qx] = sum_qy gs By
//   y_e[b][a] = sum_qx V0 Bx + V1 Dx
// (evaluated one quadrature column qx at a time: only NB-long intermediates are live)
// Every element is evaluated once.  Element rows are coloured by ey mod NB: the rows of one colour
// touch disjoint coefficient rows (ey .. ey+p), so one launch per colour adds them into y (zeroed
// first) without atomics, in a fixed order.  A block runs one element row of one patch for four column
// tiles (one wavefront each, lane = column): the four share each element's metric terms and basis
// tables Bx, Dx, staged in LDS a chunk of elements at a time (the row's By, Dy are uniform loads).  Along the row a wavefront keeps the NB x NB
// coefficients of the current element and an NB-column ring of output sums in registers; column ex
// is complete once element ex is done and is added to y.
constexpr int kSfChunk = 16;  // elements staged per LDS chunk

template <typename T, int P, int Q>
__global__ __launch_bounds__(256) void k_sumfact(const T *__restrict__ metric, const T *__restrict__ basis,
                                                 const T *__restrict__ x, T *__restrict__ y, const T *__restrict__ ca,
                                                 const T *__restrict__ cb, int nel, int n1, int W, int ldb, int ntiles,
                                                 const int *__restrict__ active, int colour, int nrow, int np) {
  constexpr int NB = P + 1, QQ = Q * Q, BT = Q * NB;  // BT: one basis table (Q points x NB functions)
  constexpr int CHUNK = kSfChunk;
  __shared__ T sm[CHUNK][QQ * 4];       // metric terms of the chunk's elements
  __shared__ T sb[CHUNK][2 * BT];       // Bx, Dx of the chunk's elements
  const int ntg = (ntiles + 3) / 4;
  const int tg = blockIdx.x % ntg, rr = (blockIdx.x / ntg) % nrow, m = blockIdx.x / (ntg * nrow);
  if (m >= np) return;
  const int ey = colour + rr * NB;
  if (ey >= nel) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int ct = tg * 4 + wave;
  const bool on = ct < ntiles && (!active || active[ct]);
  const int64_t col = (int64_t)ct * CT + lane;
  // the row's basis tables By, Dy are the same for every element of the row: uniform loads (scalar
  // registers); the metric terms and Bx, Dx change per element and are staged in LDS
  const T *By = basis + (size_t)ey * 2 * BT, *Dy = By + BT;
  const T sig = on ? ca[col] : T(0), ss = on ? cb[col] : T(0);
  const int64_t prow = (int64_t)m * W * W;
  // coefficient rows ey .. ey+p of the patch (padded rows ey+P .. ey+2P, columns shifted by P)
  auto xat = [&](int b, int a) { return x[(prow + (int64_t)(ey + b + P) * W + (a + P)) * ldb + col]; };
  auto yadd = [&](int b, int a, T v) {
    T *py = y + (prow + (int64_t)(ey + b + P) * W + (a + P)) * ldb + col;
    *py += v;
  };
  T c[NB][NB], ring[NB][NB];  // ring[b][k]: output column (ex + k) mod NB of coefficient row ey + b
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int k = 0; k < NB; ++k) ring[b][k] = T(0);
  if (on) {
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int a = 0; a < P; ++a) c[b][a + 1] = xat(b, a);  // columns 0 .. P-1, shifted in below
  }
  for (int e0 = 0; e0 < nel; e0 += CHUNK) {
    const int ne = min(CHUNK, nel - e0);
    __syncthreads();  // the previous chunk's reads are done
    for (int k = threadIdx.x; k < ne * QQ * 4; k += 256)
      sm[k / (QQ * 4)][k % (QQ * 4)] = metric[((((size_t)m * nel + ey) * nel + e0) * QQ) * 4 + k];
    for (int k = threadIdx.x; k < ne * 2 * BT; k += 256)
      sb[k / (2 * BT)][k % (2 * BT)] = basis[(size_t)e0 * 2 * BT + k];
    __syncthreads();
    if (!on) continue;
    for (int el = 0; el < ne; ++el) {
      const int ex = e0 + el;
      // the element's coefficient window: shift by one column, load column ex + P
#pragma unroll
      for (int b = 0; b < NB; ++b) {
#pragma unroll
        for (int a = 0; a < P; ++a) c[b][a] = c[b][a + 1];
        c[b][P] = xat(b, ex + P);
      }
      const T *Bx = sb[el], *Dx = sb[el] + BT, *mt = sm[el];
      // one quadrature column qx at a time (only NB-long intermediates live); local column a of the
      // element is output column ex + a, ring slot a
#pragma unroll 1
      for (int qx = 0; qx < Q; ++qx) {
        T U0[NB], U1[NB], V0[NB], V1[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          T s0 = 0, s1 = 0;
#pragma unroll
          for (int a = 0; a < NB; ++a) {
            s0 = fma(c[b][a], Bx[qx * NB + a], s0);
            s1 = fma(c[b][a], Dx[qx * NB + a], s1);
          }
          U0[b] = s0;
          U1[b] = s1;
          V0[b] = 0;
          V1[b] = 0;
        }
#pragma unroll
        for (int qy = 0; qy < Q; ++qy) {
          T u = 0, us = 0, ut = 0;
#pragma unroll
          for (int b = 0; b < NB; ++b) {
            u = fma(U0[b], By[qy * NB + b], u);
            us = fma(U1[b], By[qy * NB + b], us);
            ut = fma(U0[b], Dy[qy * NB + b], ut);
          }
          const T *gq = mt + (qy * Q + qx) * 4;
          const T v = sig * gq[0] * u;
          const T gs = ss * (gq[1] * us + gq[2] * ut);
          const T gt = ss * (gq[2] * us + gq[3] * ut);
#pragma unroll
          for (int b = 0; b < NB; ++b) {
            V0[b] = fma(v, By[qy * NB + b], fma(gt, Dy[qy * NB + b], V0[b]));
            V1[b] = fma(gs, By[qy * NB + b], V1[b]);
          }
        }
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int a = 0; a < NB; ++a)
            ring[b][a] = fma(V0[b], Bx[qx * NB + a], fma(V1[b], Dx[qx * NB + a], ring[b][a]));
      }
      // output column ex is complete: add it to y and rotate the ring by one column
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        yadd(b, ex, ring[b][0]);
#pragma unroll
        for (int k = 0; k < P; ++k) ring[b][k] = ring[b][k + 1];
        ring[b][P] = T(0);
      }
    }
  }
  if (on) {
    // the row's last P output columns nel .. nel+P-1
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int k = 0; k < P; ++k) yadd(b, nel + k, ring[b][k]);
  }
}

// y = 0 on the rows of the patches, active column tiles
template <typename T>
__global__ void k_zero_rows(T *y, int64_t R, int ldb, int ntiles, const int *active) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= R * ldb) return;
  const int ct = (int)(i % ldb) / CT;
  if (active && !active[ct]) return;
  y[i] = T(0);
}

template <typename T>
static const T *metric_of(const Level &L);
template <>
const double *metric_of<double>(const Level &L) { return L.metric.p; }
template <>
const float *metric_of<float>(const Level &L) { return L.metric32.p; }
template <typename T>
static const T *basis_of(const Level &L);
template <>
const double *basis_of<double>(const Level &L) { return L.basis.p; }
template <>
const float *basis_of<float>(const Level &L) { return L.basis32.p; }

template <typename T>
void launch_sumfact_apply(const Level &L, const T *x, T *y, const T *ca, const T *cb, int ldb, int ntiles,
                          const int *active, hipStream_t s) {
  const T *mt = metric_of<T>(L), *bs = basis_of<T>(L);
  if (L.q != L.p + 1 && L.q != L.p + 2) fail(GF_EUNSUPPORTED, "quadrature order out of range");
  const bool q2 = L.q == L.p + 2;
  const int64_t tot = L.R * ldb;
  hipLaunchKernelGGL(k_zero_rows<T>, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, y, L.R, ldb, ntiles,
                     active);
  const int NB = L.p + 1, ntg = (ntiles + 3) / 4;
  for (int colour = 0; colour < NB && colour < L.nel; ++colour) {
    const int nrow = (L.nel - colour + NB - 1) / NB;
    const dim3 grid((unsigned)(L.npatch * nrow * ntg)), block(256);
    switch (L.p) {
#define GF_SF(PP)                                                                                              \
  case PP:                                                                                                     \
    if (q2)                                                                                                    \
      hipLaunchKernelGGL((k_sumfact<T, PP, PP + 2>), grid, block, 0, s, mt, bs, x, y, ca, cb, L.nel, L.n1, L.W, \
                         ldb, ntiles, active, colour, nrow, L.npatch);                                         \
    else                                                                                                       \
      hipLaunchKernelGGL((k_sumfact<T, PP, PP + 1>), grid, block, 0, s, mt, bs, x, y, ca, cb, L.nel, L.n1, L.W, \
                         ldb, ntiles, active, colour, nrow, L.npatch);                                         \
    break;
      GF_SF(1) GF_SF(2) GF_SF(3) GF_SF(4) GF_SF(5)
#undef GF_SF
      default: fail(GF_EUNSUPPORTED, "degree out of range");
    }
  }
  HIPCHK(hipGetLastError());
}
template void launch_sumfact_apply<double>(const Level &, const double *, double *, const double *, const double *,
                                           int, int, const int *, hipStream_t);
template void launch_sumfact_apply<float>(const Level &, const float *, float *, const float *, const float *, int,
                                          int, const int *, hipStream_t);

// ------------------------------------------------------------------ stencil by probing
// Column c < S*S probes colour c = (iy mod S)*S + (ix mod S) for M, column S*S + c the same
// colour for S.  Within the (2p+1)^2 window of any coefficient each colour occurs exactly
// once, so (A x_c)[row] is the single stencil entry of that colour.
__global__ void k_probe(double *x, int ldb, int n1, int W, int P, int Sw, int64_t R) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.y + threadIdx.y;
  if (r >= R) return;
  const int lx = (int)(r % W) - P, ly = (int)((r / W) % W) - P;
  const bool inside = lx >= 0 && lx < n1 && ly >= 0 && ly < n1;
  const int colour = inside ? (ly % Sw) * Sw + (lx % Sw) : -1;
  for (int c = threadIdx.x; c < ldb; c += blockDim.x) {
    const double v = (inside && c < 2 * Sw * Sw && c % (Sw * Sw) == colour) ? 1.0 : 0.0;
    x[r * ldb + c] = v;
  }
}

void launch_probe_vectors(const Level &L, double *x, int ldb, hipStream_t s) {
  dim3 block(64, 4);
  dim3 grid((unsigned)((L.R + block.y - 1) / block.y));
  hipLaunchKernelGGL(k_probe, grid, block, 0, s, x, ldb, L.n1, L.W, L.p, L.S, L.R);
  HIPCHK(hipGetLastError());
}

__global__ void k_extract(const double *y, int ldb, double *stM, double *stS, int n1, int W, int P, int Sw,
                          int64_t R) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= R) return;
  const int lx = (int)(r % W) - P, ly = (int)((r / W) % W) - P;
  const bool inside = lx >= 0 && lx < n1 && ly >= 0 && ly < n1;
  for (int dy = -P; dy <= P; ++dy)
    for (int dx = -P; dx <= P; ++dx) {
      const int d = (dy + P) * Sw + (dx + P);
      const int nx = lx + dx, ny = ly + dy;
      double vm = 0.0, vs = 0.0;
      if (inside && nx >= 0 && nx < n1 && ny >= 0 && ny < n1) {
        const int colour = (ny % Sw) * Sw + (nx % Sw);
        vm = y[r * ldb + colour];
        vs = y[r * ldb + Sw * Sw + colour];
      }
      stM[r * Sw * Sw + d] = vm;
      stS[r * Sw * Sw + d] = vs;
    }
}

void launch_extract_stencil(const Level &L, const double *y, int ldb, double *stM, double *stS, hipStream_t s) {
  hipLaunchKernelGGL(k_extract, dim3((unsigned)((L.R + 255) / 256)), dim3(256), 0, s, y, ldb, stM, stS, L.n1, L.W,
                     L.p, L.S, L.R);
  HIPCHK(hipGetLastError());
}

// diagonals: the stencil centre of every copy, then summed over the copies of shared unknowns
// Ghost rows (outside every patch grid) get dM = 1, dS = 0: their D = sigma is positive, so the
// streaming kernels may run over ghost rows, whose vector entries stay zero.
__global__ void k_diag_centre(const double *stM, const double *stS, double *dM, double *dS, int64_t R, int c, int W,
                              int n1) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= R) return;
  const int lx = (int)(r % W) - c, ly = (int)((r / W) % W) - c;
  if (lx < 0 || lx >= n1 || ly < 0 || ly >= n1) {
    dM[r] = 1.0;
    dS[r] = 0.0;
    return;
  }
  dM[r] = stM[r * (2 * c + 1) * (2 * c + 1) + c * (2 * c + 1) + c];
  dS[r] = stS[r * (2 * c + 1) * (2 * c + 1) + c * (2 * c + 1) + c];
}
__global__ void k_diag_sum(double *dM, double *dS, const int *gp, const int *gr, int ng) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= ng) return;
  double sm = 0, ss = 0;
  for (int k = gp[g]; k < gp[g + 1]; ++k) { sm += dM[gr[k]]; ss += dS[gr[k]]; }
  for (int k = gp[g]; k < gp[g + 1]; ++k) { dM[gr[k]] = sm; dS[gr[k]] = ss; }
}
__global__ void k_to_f32(const double *a, float *b, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) b[i] = (float)a[i];
}

void launch_stencil_diag(const Level &L, hipStream_t s) {
  hipLaunchKernelGGL(k_diag_centre, dim3((unsigned)((L.R + 255) / 256)), dim3(256), 0, s, L.stM.p, L.stS.p, L.dM.p,
                     L.dS.p, L.R, L.p, L.W, L.n1);
  if (L.ngroups > 0)
    hipLaunchKernelGGL(k_diag_sum, dim3((L.ngroups + 255) / 256), dim3(256), 0, s, L.dM.p, L.dS.p, L.grp_ptr.p,
                       L.grp_rows.p, L.ngroups);
  HIPCHK(hipGetLastError());
}

void launch_to_f32(const double *a, float *b, int64_t n, hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_to_f32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a, b, n);
  HIPCHK(hipGetLastError());
}

// ------------------------------------------------------------------ white noise (Sec. 3.3)
// Pass 1: element mass matrices M_e = sum_q m_q phi_i phi_j, their lower Cholesky factors L_e, and
// y_e = L_e z_e for the samples s0 .. s1.  Pass 2 gathers.  Both stream: z is read once, and the pass
// between them (y) stays small enough for the last-level cache where that leaves enough samples to pay for
// the factorisation.  64 samples on degree 2, 64 x 64 (113 MB of z, 13 MB of loads): 280 us of kernels
// before (one thread per element, its matrix in scratch memory on degree 3; gathered one word per cache line),
// 130 us so; 9 samples on degree 3, 256 x 256: 10.7 -> 1.39 ms a call.
//
// Degrees up to 3 (at most 16 functions an element): 16 lanes per element, lane i = row i of the matrix,
// in registers; columns of the factor and the entries of z are broadcast by DPP.
template <int J, int NL>
__device__ __forceinline__ void noise_mass(double (&A)[NL], double ph, double t) {
  if constexpr (J < NL) {
    fma_row_bcast<J, J == 0>(A[J], ph, t);
    noise_mass<J + 1, NL>(A, ph, t);
  }
}
template <int J, int K, int NL>
__device__ __forceinline__ void noise_update(double (&A)[NL], double nl, double l) {
  if constexpr (K < NL) {
    fma_row_bcast<K, K == J + 1>(A[K], nl, l);
    noise_update<J, K + 1, NL>(A, nl, l);
  }
}
template <int J, int NL>
__device__ __forceinline__ void noise_factor(double (&A)[NL], int i) {
  if constexpr (J < NL) {
    // (a DPP source written by the vector instruction before it needs two cycles; the compiler does not
    // see that the asm above wrote A[J])
    asm volatile("s_nop 1" : "+v"(A[J]));
    const double d = sqrt(row_bcast<J>(A[J]));
    const double l = i == J ? d : (i > J ? A[J] / d : 0.0);
    A[J] = l;
    noise_update<J, J + 1, NL>(A, -l, l);
    noise_factor<J + 1, NL>(A, i);
  }
}
// v = sum_{k <= i} A[k] z_k (row i reads no entry past its own: what is not finite there stays there)
template <int K, int NL>
__device__ __forceinline__ void noise_row(double &v, const double (&A)[NL], double z, int i) {
  if constexpr (K < NL) {
    double t = v;
    fma_row_bcast<K, K == 0>(t, z, A[K]);
    v = K <= i ? t : v;
    noise_row<K + 1, NL>(v, A, z, i);
  }
}
template <int P, int Q>
__global__ __launch_bounds__(256) void k_noise_apply(const double *__restrict__ metric, const double *__restrict__ basis,
                                                     const double *__restrict__ z, double *__restrict__ ye, int nel,
                                                     int s0, int s1, int np) {
  constexpr int NB = P + 1, NL = NB * NB, U = 4;
  const int64_t ne_tot = (int64_t)np * nel * nel;
  const int64_t e0 = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4);
  const int64_t e = e0 < ne_tot ? e0 : ne_tot - 1;  // (whole groups of lanes run, the last ones without a result)
  const int lane = threadIdx.x & 15, i = min(lane, NL - 1);
  const bool on = e0 < ne_tot && lane < NL;
  const int ex = (int)(e % nel), ey = (int)((e / nel) % nel);
  const double *Bx = basis + (size_t)ex * 2 * Q * NB, *By = basis + (size_t)ey * 2 * Q * NB, *mt = metric + e * Q * Q * 4;
  double A[NL];
#pragma unroll
  for (int k = 0; k < NL; ++k) A[k] = 0.0;
#pragma unroll 4
  for (int q = 0; q < Q * Q; ++q) {
    const double ph = By[(q / Q) * NB + i / NB] * Bx[(q % Q) * NB + i % NB];
    noise_mass<0, NL>(A, ph, mt[q * 4] * ph);
  }
  noise_factor<0, NL>(A, i);
  // this block's samples of s0 .. s1
  const int ns = s1 - s0, per = (ns + gridDim.y - 1) / gridDim.y;
  const int sa = s0 + per * blockIdx.y, sb = min(sa + per, s1);
  for (int s = sa; s < sb; s += U) {
    double zv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) zv[u] = z[((size_t)min(s + u, sb - 1) * ne_tot + e) * NL + i];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      double v = 0.0;
      noise_row<0, NL>(v, A, zv[u], i);
      if (on && s + u < sb) ye[((size_t)(s + u - s0) * ne_tot + e) * NL + i] = v;
    }
  }
}

// Degrees 4 and 5: one thread per element.
template <int P, int Q>
__global__ void k_noise_elements(const double *metric, const double *basis, const double *z, double *ye, int nel,
                                 int s0, int s1, int np) {
  constexpr int NB = P + 1, NL = NB * NB;
  const int64_t ne_tot = (int64_t)np * nel * nel;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= ne_tot) return;
  const int ex = (int)(e % nel), ey = (int)((e / nel) % nel);
  const double *Bx = basis + (size_t)ex * 2 * Q * NB;
  const double *By = basis + (size_t)ey * 2 * Q * NB;
  const double *mt = metric + e * Q * Q * 4;
  double A[NL][NL];
  for (int i = 0; i < NL; ++i)
    for (int j = 0; j < NL; ++j) A[i][j] = 0.0;
  for (int qy = 0; qy < Q; ++qy)
    for (int qx = 0; qx < Q; ++qx) {
      const double w = mt[(qy * Q + qx) * 4];
      double phi[NL];
      for (int b = 0; b < NB; ++b)
        for (int a = 0; a < NB; ++a) phi[b * NB + a] = By[qy * NB + b] * Bx[qx * NB + a];
      for (int i = 0; i < NL; ++i)
        for (int j = 0; j < NL; ++j) A[i][j] += w * phi[i] * phi[j];
    }
  // in-place lower Cholesky
  for (int j = 0; j < NL; ++j) {
    double d = A[j][j];
    for (int k = 0; k < j; ++k) d -= A[j][k] * A[j][k];
    d = sqrt(d);
    A[j][j] = d;
    for (int i = j + 1; i < NL; ++i) {
      double v = A[i][j];
      for (int k = 0; k < j; ++k) v -= A[i][k] * A[j][k];
      A[i][j] = v / d;
    }
  }
  for (int s = s0; s < s1; ++s) {
    const double *zs = z + ((size_t)s * ne_tot + e) * NL;
    double *ys = ye + ((size_t)(s - s0) * ne_tot + e) * NL;
    for (int i = 0; i < NL; ++i) {
      double v = 0.0;
      for (int k = 0; k <= i; ++k) v += A[i][k] * zs[k];
      ys[i] = v;
    }
  }
}

// Pass 2: b[s][g] of every unknown g: the contributions of all elements that contain it, summed within each
// patch and then over the copies.  Unknowns off the patch boundary by their number, the others by their
// group of copies (threads N .. N + ngroups).
template <int P>
__global__ __launch_bounds__(256) void k_noise_gather(const double *__restrict__ ye, double *__restrict__ b, int nel,
                                                      int n1, int W, int N, int ngroups, int np,
                                                      const int *__restrict__ orow, const int *__restrict__ rgid,
                                                      const int *__restrict__ gp, const int *__restrict__ gr) {
  constexpr int NB = P + 1, NL = NB * NB;
  const int id = blockIdx.x * 256 + threadIdx.x;
  if (id >= N + ngroups) return;
  const int64_t ne_tot = (int64_t)np * nel * nel;
  const double *ys = ye + (size_t)blockIdx.y * ne_tot * NL;
  auto patch_sum = [&](int row) {
    const int m = row / (W * W), q = row - m * W * W, ly = q / W - P, lx = q % W - P;
    double v = 0.0;
#pragma unroll
    for (int bb = 0; bb < NB; ++bb) {
      const int ey = ly - bb;
      if (ey < 0 || ey >= nel) continue;
#pragma unroll
      for (int a = 0; a < NB; ++a) {
        const int ex = lx - a;
        if (ex < 0 || ex >= nel) continue;
        v += ys[(((int64_t)m * nel + ey) * nel + ex) * NL + bb * NB + a];
      }
    }
    return v;
  };
  double v = 0.0;
  int g = id;
  if (id < N) {
    const int row = orow[id], q = row % (W * W), ly = q / W - P, lx = q % W - P;
    if (lx == 0 || lx == n1 - 1 || ly == 0 || ly == n1 - 1) return;
    v = patch_sum(row);
  } else {
    const int k0 = gp[id - N], k1 = gp[id - N + 1];
    for (int k = k0; k < k1; ++k) v += patch_sum(gr[k]);
    g = rgid[gr[k0]];
  }
  b[(size_t)blockIdx.y * N + g] = v;
}

// samples per pass: y within 96 MB, but at least 16 (a pass factorises every element anew).  Degrees 4 and 5, whose
// factorisation by one thread takes longer than everything else, in one pass: 64 samples on degree 4, 64 x 64,
// 16.3 ms in four passes, 6.9 in one.
int noise_chunk(const Level &L, int nsamp) {
  if (L.p > 3) return nsamp;
  const int64_t per = (int64_t)L.npatch * L.nel * L.nel * (L.p + 1) * (L.p + 1) * 8;
  return (int)std::min<int64_t>(nsamp, std::max<int64_t>(16, ((int64_t)96 << 20) / per));
}
constexpr int kNoiseGrid = 16384;  // samples per launch of the second pass

// ye: work space for `chunk` samples' element contributions; b: [nsamp][N]
void launch_white_noise(const Level &L, const double *z, int nsamp, int chunk, double *ye, double *b, hipStream_t s) {
  const int64_t ne_tot = (int64_t)L.npatch * L.nel * L.nel, nl = ne_tot * (L.p + 1) * (L.p + 1);
  if (L.q != L.p + 1 && L.q != L.p + 2) fail(GF_EUNSUPPORTED, "quadrature order out of range");
  const bool q2 = L.q == L.p + 2;
  const unsigned nb = (unsigned)((ne_tot + 15) / 16);
  for (int s0 = 0; s0 < nsamp; s0 += chunk) {
    const int s1 = std::min(nsamp, s0 + chunk);
    // few elements: the samples are split over blocks as well, down to four a block
    const unsigned ny = std::max(1u, std::min((unsigned)(s1 - s0 + 3) / 4, 1024u / nb));
    const dim3 gn(nb, ny), go((unsigned)((ne_tot + 63) / 64));
    switch (L.p) {
#define GF_NE(PP, KERN, GRID, BLOCK)                                                                               \
  case PP:                                                                                                         \
    if (q2) hipLaunchKernelGGL((KERN<PP, PP + 2>), GRID, BLOCK, 0, s, L.metric.p, L.basis.p, z, ye, L.nel, s0, s1, \
                               L.npatch);                                                                          \
    else hipLaunchKernelGGL((KERN<PP, PP + 1>), GRID, BLOCK, 0, s, L.metric.p, L.basis.p, z, ye, L.nel, s0, s1,    \
                            L.npatch);                                                                             \
    for (int t0 = s0; t0 < s1; t0 += kNoiseGrid) /* (the grid's second dimension) */                               \
      hipLaunchKernelGGL(k_noise_gather<PP>,                                                                       \
                         dim3((L.N + L.ngroups + 255) / 256, std::min(s1 - t0, kNoiseGrid)), dim3(256), 0, s,      \
                         ye + (t0 - s0) * nl, b + (size_t)t0 * L.N, L.nel, L.n1, L.W, L.N, L.ngroups, L.npatch,    \
                         L.owner_row.p, L.row_gid.p, L.grp_ptr.p, L.grp_rows.p);                                   \
    break;
      GF_NE(1, k_noise_apply, gn, dim3(256))
      GF_NE(2, k_noise_apply, gn, dim3(256))
      GF_NE(3, k_noise_apply, gn, dim3(256))
      GF_NE(4, k_noise_elements, go, dim3(64))
      GF_NE(5, k_noise_elements, go, dim3(64))
#undef GF_NE
      default: fail(GF_EUNSUPPORTED, "degree out of range");
    }
    HIPCHK(hipGetLastError());
  }
}

// ------------------------------------------------------------------ coarse Cholesky
// One thread per node: A = sigma M0 + S0 (dense, global numbering of the coarsest level),
// lower Cholesky factor in place.  info = 0 on success, k+1 if pivot k is not positive.
__global__ void k_coarse_factor(const double *M0, const double *S0, int n, const double *sig, int nnode, double *Lf,
                                int *info) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= nnode) return;
  double *A = Lf + (size_t)k * n * n;
  const double sg = sig[k];
  for (int i = 0; i < n * n; ++i) A[i] = sg * M0[i] + S0[i];
  int bad = 0;
  for (int j = 0; j < n && !bad; ++j) {
    double d = A[j * n + j];
    for (int t = 0; t < j; ++t) d -= A[j * n + t] * A[j * n + t];
    if (!(d > 0.0)) { bad = j + 1; break; }
    d = sqrt(d);
    A[j * n + j] = d;
    for (int i = j + 1; i < n; ++i) {
      double v = A[i * n + j];
      for (int t = 0; t < j; ++t) v -= A[i * n + t] * A[j * n + t];
      A[i * n + j] = v / d;
    }
    for (int i = 0; i < j; ++i) A[i * n + j] = 0.0;  // clear the upper triangle
  }
  info[k] = bad;
}

// Factor and inverse in one launch, a block per node, the packed lower triangle in LDS: right-looking, the
// trailing update shared by all threads, then thread j builds column j of the inverse from the factor.  The
// sums run in the order of the two kernels above and below, which serve matrices that do not fit: one thread
// factorises a node there, 3.9 ms for 41 nodes of 56 unknowns and 0.3 ms for the inverses; 0.30 ms for both here.
constexpr size_t kFactorLds = 144 << 10;
__global__ __launch_bounds__(256) void k_coarse_both(const double *__restrict__ M0, const double *__restrict__ S0, int n,
                                                     const double *__restrict__ sig, double *__restrict__ Ainv, int *info) {
  extern __shared__ double A[];  // row i at i (i + 1) / 2
  const int node = blockIdx.x, t = threadIdx.x;
  const double sg = sig[node];
  for (int q = t; q < n * n; q += 256) {
    const int i = q / n, j = q - i * n;
    if (j <= i) A[i * (i + 1) / 2 + j] = sg * M0[q] + S0[q];
  }
  __syncthreads();
  for (int j = 0; j < n; ++j) {
    const double p = A[j * (j + 1) / 2 + j], d = sqrt(p);
    if (!(p > 0.0)) {  // (the same value for every thread)
      if (t == 0) info[node] = j + 1;
      return;
    }
    __syncthreads();  // the pivot is read before it is overwritten
    for (int i = j + t; i < n; i += 256) A[i * (i + 1) / 2 + j] = i == j ? d : A[i * (i + 1) / 2 + j] / d;
    __syncthreads();
    const int r = n - j - 1;  // trailing rows: entry (i, k), k <= i, minus l_ij l_kj
    for (int q = t; q < r * r; q += 256) {
      const int i = j + 1 + q / r, k = j + 1 + q % r;
      if (k <= i) A[i * (i + 1) / 2 + k] -= A[i * (i + 1) / 2 + j] * A[k * (k + 1) / 2 + j];
    }
    __syncthreads();
  }
  double *X = Ainv + (size_t)node * n * n;
  for (int j = t; j < n; j += 256) {
    for (int i = 0; i < n; ++i) {
      double s = (i == j) ? 1.0 : 0.0;
      const double *Li = A + i * (i + 1) / 2;
      for (int k = j; k < i; ++k) s -= Li[k] * X[(size_t)k * n + j];
      X[(size_t)i * n + j] = (i < j) ? 0.0 : s / Li[i];
    }
    for (int i = n - 1; i >= 0; --i) {
      double s = X[(size_t)i * n + j];
      for (int k = i + 1; k < n; ++k) s -= A[k * (k + 1) / 2 + i] * X[(size_t)k * n + j];
      X[(size_t)i * n + j] = s / A[i * (i + 1) / 2 + i];
    }
  }
  if (t == 0) info[node] = 0;
}
bool launch_coarse_both(const double *M0, const double *S0, int N0, const double *sig, int nnode, double *Ainv, int *info,
                        hipStream_t s) {
  const size_t lds = (size_t)N0 * (N0 + 1) / 2 * sizeof(double);
  if (lds > kFactorLds) return false;
  raise_lds(reinterpret_cast<const void *>(&k_coarse_both), kFactorLds);
  hipLaunchKernelGGL(k_coarse_both, dim3(nnode), dim3(256), (unsigned)lds, s, M0, S0, N0, sig, Ainv, info);
  HIPCHK(hipGetLastError());
  return true;
}

void launch_coarse_factor(const double *M0, const double *S0, int N0, const double *sig, int nnode, double *Lf,
                          int *info, hipStream_t s) {
  hipLaunchKernelGGL(k_coarse_factor, dim3((nnode + 63) / 64), dim3(64), 0, s, M0, S0, N0, sig, nnode, Lf, info);
  HIPCHK(hipGetLastError());
}

// A^-1 = L^-T L^-1 from the Cholesky factor, one block per node, thread j builds column j:
// forward substitution L y = e_j, then back substitution L^T x = y, both in place in the column.
__global__ void k_coarse_inverse(const double *Lf, int n, int nnode, double *Ainv) {
  const int k = blockIdx.x;
  if (k >= nnode) return;
  const double *L = Lf + (size_t)k * n * n;
  double *X = Ainv + (size_t)k * n * n;
  for (int j = threadIdx.x; j < n; j += blockDim.x) {
    for (int i = 0; i < n; ++i) {
      double s = (i == j) ? 1.0 : 0.0;
      for (int t = j; t < i; ++t) s -= L[(size_t)i * n + t] * X[(size_t)t * n + j];
      X[(size_t)i * n + j] = (i < j) ? 0.0 : s / L[(size_t)i * n + i];
    }
    for (int i = n - 1; i >= 0; --i) {
      double s = X[(size_t)i * n + j];
      for (int t = i + 1; t < n; ++t) s -= L[(size_t)t * n + i] * X[(size_t)t * n + j];
      X[(size_t)i * n + j] = s / L[(size_t)i * n + i];
    }
  }
}

void launch_coarse_inverse(const double *Lf, int N0, int nnode, double *Ainv, hipStream_t s) {
  hipLaunchKernelGGL(k_coarse_inverse, dim3(nnode), dim3(std::min(1024, (N0 + 63) / 64 * 64)), 0, s, Lf, N0, nnode,
                     Ainv);
  HIPCHK(hipGetLastError());
}

}  // namespace gf

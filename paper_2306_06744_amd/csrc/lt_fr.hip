// lt_fr.hip -- flux reconstruction on the adapted tree: common fluxes with
// mortars at hanging faces (Section 4.3) and the FR residual with the
// three-stage Runge-Kutta step (Section 2.1, eq. rk3), for the Euler
// equations on Gauss-Legendre solution points.
//
// Common fluxes alone (lt_fr_face_flux): a face buffer FB[f][v][q][ld] (face
// f = 2 axis + side, variable v, face point q with the tangential axes in
// increasing order, the lower fastest, element fastest) first holds the
// solution's traces, then -- overwritten in place -- the common normal fluxes:
//   k_fr_trace   one lane per element: u -> traces of every face;
//   k_fr_conf    one lane per element and axis: a conforming face pair is
//                owned by its low-side element, which reads both traces and
//                writes the Rusanov flux into both slots;
//   k_fr_mortar  one wave per hanging-face row, lane = (mortar s, face point):
//                the coarse trace L2-projected onto the mortar (exact for the
//                same degree: the half-interval interpolation factors A_b),
//                the fine trace, the Rusanov flux on the mortar into the fine
//                slot, and the coarse slot's L2 projection of the mortar
//                fluxes (the half-interval projection factors P_b) summed
//                over the mortars through LDS.
// Residual and Runge-Kutta stages: no face buffer; k_fr_stage forms traces and
// fluxes where it uses them, and only the hanging faces' fluxes are stored
// (k_fr_rows, k_fr_hang; see there).
// Every slot is read and written by exactly one owner: no atomics on values,
// and the result is the same on every run (the paper accumulates the coarse
// side with atomic additions).
#include <hip/hip_runtime.h>

#include <cmath>
#include <string>
#include <vector>

#include "tree.hpp"

namespace lt {
namespace {

// shares the error word with the scans' ERR_* bits
enum : unsigned { ERR_FR_ROW = 1u << 13 };

// Per-degree FP64 tables (device, n1 = p + 1):
//   D[n1][n1] (D[i][j] = l_j'(z_i)), lL[n1], lR[n1] (l_j(-1), l_j(1)),
//   dgL[n1], dgR[n1] (Radau correction derivatives at z_i),
//   A0, A1 (half-interval interpolation, A_b[i][k] = l_k((z_i + 2b - 1)/2)),
//   P0, P1 (half-interval L2 projection back onto the whole interval).
struct FrTab {
  static constexpr int kD = 0;
  __host__ __device__ static constexpr int lL(int n) { return n * n; }
  __host__ __device__ static constexpr int lR(int n) { return n * n + n; }
  __host__ __device__ static constexpr int dgL(int n) { return n * n + 2 * n; }
  __host__ __device__ static constexpr int dgR(int n) { return n * n + 3 * n; }
  __host__ __device__ static constexpr int A(int n, int b) { return n * n + 4 * n + b * n * n; }
  __host__ __device__ static constexpr int P(int n, int b) { return 3 * n * n + 4 * n + b * n * n; }
  __host__ __device__ static constexpr int size(int n) { return 5 * n * n + 4 * n; }
};

// The 1D operators are built by constexpr functions, so that the volume
// kernel takes them as literal constants (no loads, no registers held across
// its loop) and the device tables of the other kernels hold the same values.

// cos by its Taylor series (|x| <= pi; a starting guess only).
constexpr double cx_cos(double x) {
  double term = 1.0, sum = 1.0;
  for (int k = 1; k < 30; ++k) {
    term *= -x * x / ((2.0 * k - 1.0) * (2.0 * k));
    sum += term;
  }
  return sum;
}

constexpr double cx_abs(double x) { return x < 0.0 ? -x : x; }

// P_n(x) and P_{n-1}(x) by the three-term (Bonnet) recurrence.
constexpr void legendre_pair(int n, double x, double* pn, double* pm) {
  double p0 = 1.0, p1 = x;
  for (int k = 2; k <= n; ++k) {
    const double p2 = ((2.0 * k - 1.0) * x * p1 - (k - 1.0) * p0) / k;
    p0 = p1;
    p1 = p2;
  }
  *pn = n == 0 ? 1.0 : p1;
  *pm = n == 0 ? 0.0 : p0;
}

template <int Q>
struct GaussLegendre {
  double z[Q] = {};
  double w[Q] = {};
};

// Gauss-Legendre nodes (ascending) and weights: Newton on P_Q from the usual
// cosine guess, w = 2 / ((1 - z^2) P_Q'(z)^2).
template <int Q>
constexpr GaussLegendre<Q> gauss_legendre() {
  GaussLegendre<Q> r;
  for (int i = 0; i < Q; ++i) {
    double x = -cx_cos(M_PI * (i + 0.75) / (Q + 0.5));
    for (int it = 0; it < 100; ++it) {
      double pn = 0.0, pm = 0.0;
      legendre_pair(Q, x, &pn, &pm);
      const double dp = Q * (x * pn - pm) / (x * x - 1.0);
      const double dx = pn / dp;
      x -= dx;
      if (cx_abs(dx) < 1e-16) break;
    }
    double pn = 0.0, pm = 0.0;
    legendre_pair(Q, x, &pn, &pm);
    const double dp = Q * (x * pn - pm) / (x * x - 1.0);
    r.z[i] = x;
    r.w[i] = 2.0 / ((1.0 - x * x) * dp * dp);
  }
  return r;
}

// Lagrange basis l_k on the nodes z (n of them) and its derivative.
constexpr double lag(const double* z, int n, int k, double x) {
  double v = 1.0;
  for (int m = 0; m < n; ++m)
    if (m != k) v *= (x - z[m]) / (z[k] - z[m]);
  return v;
}

constexpr double lag_d(const double* z, int n, int k, double x) {
  double s = 0.0;
  for (int r = 0; r < n; ++r) {
    if (r == k) continue;
    double t = 1.0 / (z[k] - z[r]);
    for (int m = 0; m < n; ++m)
      if (m != k && m != r) t *= (x - z[m]) / (z[k] - z[m]);
    s += t;
  }
  return s;
}

// P_n'(x) from P_{k+1}' = P_{k-1}' + (2k+1) P_k.
constexpr double leg_d(int n, double x) {
  if (n == 0) return 0.0;
  double pm = 1.0, pc = x, dm = 0.0, dc = 1.0;
  for (int k = 1; k < n; ++k) {
    const double pn = ((2.0 * k + 1.0) * x * pc - k * pm) / (k + 1.0);
    const double dn = dm + (2.0 * k + 1.0) * pc;
    pm = pc;
    pc = pn;
    dm = dc;
    dc = dn;
  }
  return dc;
}

// The operators of degree N - 1 on N Gauss-Legendre points, laid out as the
// device table (FrTab).
template <int N>
struct Ops1D {
  double t[5 * N * N + 4 * N] = {};
};

template <int N>
constexpr Ops1D<N> ops_1d() {
  constexpr int p = N - 1;
  const GaussLegendre<N> gl = gauss_legendre<N>();
  const GaussLegendre<N + 1> gq = gauss_legendre<N + 1>();
  Ops1D<N> o;
  double* T = o.t;
  for (int i = 0; i < N; ++i)
    for (int j = 0; j < N; ++j) T[FrTab::kD + i * N + j] = lag_d(gl.z, N, j, gl.z[i]);
  for (int j = 0; j < N; ++j) {
    T[FrTab::lL(N) + j] = lag(gl.z, N, j, -1.0);
    T[FrTab::lR(N) + j] = lag(gl.z, N, j, 1.0);
  }
  // g_L = (-1)^(p+1)/2 (P_{p+1} - P_p), g_R = (P_{p+1} + P_p)/2
  const double sL = (p + 1) % 2 ? -0.5 : 0.5;
  for (int i = 0; i < N; ++i) {
    T[FrTab::dgL(N) + i] = sL * (leg_d(p + 1, gl.z[i]) - leg_d(p, gl.z[i]));
    T[FrTab::dgR(N) + i] = 0.5 * (leg_d(p + 1, gl.z[i]) + leg_d(p, gl.z[i]));
  }
  for (int b = 0; b < 2; ++b) {
    for (int i = 0; i < N; ++i)
      for (int k = 0; k < N; ++k) T[FrTab::A(N, b) + i * N + k] = lag(gl.z, N, k, (gl.z[i] + 2.0 * b - 1.0) / 2.0);
    // P_b = M^-1 S_b, M = diag(w) (exact for GL), S_b[j][i] = int_{half b} l_j l^_i
    for (int j = 0; j < N; ++j)
      for (int i = 0; i < N; ++i) {
        double s = 0.0;
        for (int q = 0; q < N + 1; ++q)
          s += gq.w[q] / 2.0 * lag(gl.z, N, j, (gq.z[q] + 2.0 * b - 1.0) / 2.0) * lag(gl.z, N, i, gq.z[q]);
        T[FrTab::P(N, b) + j * N + i] = s / gl.w[j];
      }
  }
  return o;
}

template <int N>
std::vector<double> tables_of() {
  constexpr Ops1D<N> o = ops_1d<N>();
  return std::vector<double>(o.t, o.t + FrTab::size(N));
}

std::vector<double> fr_tables(int p) {
  switch (p + 1) {
    case 2: return tables_of<2>();
    case 3: return tables_of<3>();
    case 4: return tables_of<4>();
    case 5: return tables_of<5>();
    case 6: return tables_of<6>();
    case 7: return tables_of<7>();
    default: return tables_of<8>();
  }
}

// ------------------------------------------------------------------ physics
template <int DIM>
__device__ inline double pressure(const double* U, double gm1) {
  double kin = 0.0;
#pragma unroll
  for (int a = 0; a < DIM; ++a) kin += U[1 + a] * U[1 + a];
  return gm1 * (U[DIM + 1] - 0.5 * kin / U[0]);
}

// Euler flux along axis a of the state U (nvar = DIM + 2 values).
template <int DIM>
__device__ inline void euler_flux(const double* U, int a, double gm1, double* F) {
  const double p = pressure<DIM>(U, gm1);
  const double ua = U[1 + a] / U[0];
  F[0] = U[1 + a];
#pragma unroll
  for (int b = 0; b < DIM; ++b) F[1 + b] = U[1 + b] * ua + (b == a ? p : 0.0);
  F[DIM + 1] = (U[DIM + 1] + p) * ua;
}

// Rusanov flux across a face normal to axis a, UL on the low side.
template <int DIM>
__device__ inline void rusanov(const double* UL, const double* UR, int a, double gamma, double* F) {
  constexpr int NV = DIM + 2;
  const double gm1 = gamma - 1.0;
  double FL[NV], FR[NV];
  euler_flux<DIM>(UL, a, gm1, FL);
  euler_flux<DIM>(UR, a, gm1, FR);
  const double sL = fabs(UL[1 + a] / UL[0]) + sqrt(gamma * pressure<DIM>(UL, gm1) / UL[0]);
  const double sR = fabs(UR[1 + a] / UR[0]) + sqrt(gamma * pressure<DIM>(UR, gm1) / UR[0]);
  const double lam = fmax(sL, sR);
#pragma unroll
  for (int v = 0; v < NV; ++v) F[v] = 0.5 * (FL[v] + FR[v]) - 0.5 * lam * (UR[v] - UL[v]);
}

// ------------------------------------------------------------------ indexing
// Point index i = sum_b idx_b N^b; face point q of a face normal to axis a:
// the other axes in increasing order, the lower fastest.
template <int DIM, int N>
__device__ inline int face_point(const int* idx, int a) {
  int q = 0, m = 1;
#pragma unroll
  for (int b = 0; b < DIM; ++b)
    if (b != a) {
      q += idx[b] * m;
      m *= N;
    }
  return q;
}

template <int DIM>
__device__ inline int64_t fb_index(int f, int v, int q, int nfp, int64_t ldf, int64_t e) {
  return (int64_t(f * (DIM + 2) + v) * nfp + q) * ldf + e;
}

// ------------------------------------------------------------------ kernels
template <int DIM, int N>
__global__ __launch_bounds__(256) void k_fr_trace(const double* __restrict__ u, int64_t ld, int64_t n,
                                                  const double* __restrict__ tab,
                                                  double* __restrict__ fb, int64_t ldf) {
  constexpr int NP = DIM == 3 ? N * N * N : N * N;
  constexpr int NFP = NP / N;
  const int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e >= n) return;
  double lL[N], lR[N];
#pragma unroll
  for (int j = 0; j < N; ++j) {
    lL[j] = tab[FrTab::lL(N) + j];
    lR[j] = tab[FrTab::lR(N) + j];
  }
  for (int v = 0; v < DIM + 2; ++v) {
    double x[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) x[i] = u[(int64_t(v) * NP + i) * ld + e];
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
      int stride = 1;
      for (int b = 0; b < a; ++b) stride *= N;
#pragma unroll
      for (int q = 0; q < NFP; ++q) {
        // first point of the line through face point q
        int idx[3] = {0, 0, 0}, r = q;
#pragma unroll
        for (int b = 0; b < DIM; ++b)
          if (b != a) {
            idx[b] = r % N;
            r /= N;
          }
        int i0 = 0, m = 1;
#pragma unroll
        for (int b = 0; b < DIM; ++b) {
          i0 += idx[b] * m;
          m *= N;
        }
        double sl = 0.0, sr = 0.0;
#pragma unroll
        for (int j = 0; j < N; ++j) {
          sl += lL[j] * x[i0 + j * stride];
          sr += lR[j] * x[i0 + j * stride];
        }
        fb[fb_index<DIM>(2 * a, v, q, NFP, ldf, e)] = sl;
        fb[fb_index<DIM>(2 * a + 1, v, q, NFP, ldf, e)] = sr;
      }
    }
  }
}

template <int DIM, int N>
__global__ __launch_bounds__(256) void k_fr_conf(KeyGeom g, const uint64_t* __restrict__ keys,
                                                 const int32_t* __restrict__ nbr, int64_t n,
                                                 double gamma, double* __restrict__ fb, int64_t ldf,
                                                 unsigned* err) {
  constexpr int NFP = DIM == 3 ? N * N : N;
  constexpr int NV = DIM + 2;
  const int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e >= n) return;
  const int de = key_depth(g, keys[e]);
#pragma unroll 1
  for (int a = 0; a < DIM; ++a) {
    const int f = 2 * a + 1;
    const int64_t j = nbr[e * 2 * DIM + f];
    if (j == -2 || nbr[e * 2 * DIM + f - 1] == -2) {
      atomicOr(err, ERR_INVALID_TREE);  // a non-periodic face: not supported
      continue;
    }
    if (j < 0 || j >= n || key_depth(g, keys[j]) != de) continue;  // hanging: the mortar kernel
#pragma unroll 1
    for (int q = 0; q < NFP; ++q) {
      double UL[NV], UR[NV], F[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        UL[v] = fb[fb_index<DIM>(f, v, q, NFP, ldf, e)];
        UR[v] = fb[fb_index<DIM>(f - 1, v, q, NFP, ldf, j)];
      }
      rusanov<DIM>(UL, UR, a, gamma, F);
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        fb[fb_index<DIM>(f, v, q, NFP, ldf, e)] = F[v];
        fb[fb_index<DIM>(f - 1, v, q, NFP, ldf, j)] = F[v];
      }
    }
  }
}

// One wave per hanging-face row [c, f, k_0 .. k_{S-1}], lane = s * NFP + q.
template <int DIM, int N>
__global__ __launch_bounds__(256) void k_fr_mortar(const int32_t* __restrict__ hang, int64_t nrows,
                                                   int64_t n, const double* __restrict__ tab,
                                                   double gamma, double* __restrict__ fb, int64_t ldf,
                                                   unsigned* err) {
  constexpr int NFP = DIM == 3 ? N * N : N;
  constexpr int S = 1 << (DIM - 1);
  constexpr int NV = DIM + 2;
  constexpr int W = 2 + S;
  static_assert(S * NFP <= 64, "one wave per row");
  __shared__ double Fm[4][S * NFP][NV];  // mortar fluxes of the wave's row
  __shared__ double Uc[4][NFP][NV];      // coarse trace
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t r = int64_t(blockIdx.x) * (blockDim.x >> 6) + wv;
  const bool row_ok = r < nrows;
  const int s = lane / NFP, q = lane % NFP;
  const bool act = row_ok && lane < S * NFP;
  int64_t c = 0, k = 0;
  int f = 0;
  if (row_ok) {
    c = hang[r * W];
    f = hang[r * W + 1];
  }
  if (act) k = hang[r * W + 2 + s];
  const bool ok = !row_ok || (c >= 0 && c < n && f >= 0 && f < 2 * DIM && k >= 0 && k < n);
  if (!ok) atomicOr(err, ERR_FR_ROW);
  const bool go = act && ok;
  if (go && s == 0)
    for (int v = 0; v < NV; ++v) Uc[wv][q][v] = fb[fb_index<DIM>(f, v, q, NFP, ldf, c)];
  __syncthreads();
  const int a = f >> 1, side = f & 1;
  // tangential child bits of mortar s and the face point's tangential indices
  const int b0 = s & 1, b1 = (s >> 1) & 1;
  const int q0 = q % N, q1 = q / N;
  double Um[NV], Uk[NV], F[NV];
  if (go) {
    const double* A0 = tab + FrTab::A(N, b0);
    const double* A1 = tab + FrTab::A(N, b1);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      double acc = 0.0;
      if (DIM == 2) {
#pragma unroll
        for (int i = 0; i < N; ++i) acc += A0[q0 * N + i] * Uc[wv][i][v];
      } else {
#pragma unroll
        for (int i1 = 0; i1 < N; ++i1) {
          double t = 0.0;
#pragma unroll
          for (int i0 = 0; i0 < N; ++i0) t += A0[q0 * N + i0] * Uc[wv][i1 * N + i0][v];
          acc += A1[q1 * N + i1] * t;
        }
      }
      Um[v] = acc;
      Uk[v] = fb[fb_index<DIM>(f ^ 1, v, q, NFP, ldf, k)];
    }
    if (side == 1)
      rusanov<DIM>(Um, Uk, a, gamma, F);
    else
      rusanov<DIM>(Uk, Um, a, gamma, F);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      fb[fb_index<DIM>(f ^ 1, v, q, NFP, ldf, k)] = F[v];
      Fm[wv][lane][v] = F[v];
    }
  }
  __syncthreads();
  // coarse face: sum over the mortars of (P_b1 x P_b0) applied to their fluxes
  if (go && s == 0) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      double acc = 0.0;
#pragma unroll
      for (int m = 0; m < S; ++m) {
        const double* P0 = tab + FrTab::P(N, m & 1);
        const double* P1 = tab + FrTab::P(N, (m >> 1) & 1);
        if (DIM == 2) {
#pragma unroll
          for (int i = 0; i < N; ++i) acc += P0[q0 * N + i] * Fm[wv][m * NFP + i][v];
        } else {
#pragma unroll
          for (int i1 = 0; i1 < N; ++i1) {
            double t = 0.0;
#pragma unroll
            for (int i0 = 0; i0 < N; ++i0) t += P0[q0 * N + i0] * Fm[wv][m * NFP + i1 * N + i0][v];
            acc += P1[q1 * N + i1] * t;
          }
        }
      }
      fb[fb_index<DIM>(f, v, q, NFP, ldf, c)] = acc;
    }
  }
}

// ------------------------------------------------- residual and RK3 stages
// A stage reads the state and writes the next one in a single kernel,
// k_fr_stage: a lane takes one line of points of one element along one axis
// after the other, and at both ends of its line forms the neighbour's trace
// from the neighbour's own line.  Nothing is stored per face, except for the
// few hanging faces (k_fr_rows once per call, k_fr_hang before each stage).
//
// Per p = 3 element in 3D a stage moves 2560 B of state in and out (2560 more
// where the step's first state enters) and reads the neighbours' lines, six
// elements' worth, through the caches: in Morton order nearly all of them are
// being worked on nearby.  The form with a face buffer (traces written, both
// traces read and the fluxes written by face, the fluxes read by element)
// moved 23 to 25.6 KB per element and stage.
//
// Hanging faces: HB[row][S + 1][nvar][nfp] holds a row's S fine fluxes and
// its coarse one; code[e * 2 dim + f] = row * (S + 1) + slot where bit f of
// hm[e] is set.

// Pointwise quantities of a state along axis a.
template <int DIM>
struct Point {
  double ua, p, c;
};

template <int DIM>
__device__ inline Point<DIM> point_of(const double* U, int a, double gamma) {
  const double ir = 1.0 / U[0];
  double kin = 0.0;
#pragma unroll
  for (int b = 0; b < DIM; ++b) kin += U[1 + b] * U[1 + b];
  Point<DIM> r;
  r.p = (gamma - 1.0) * (U[DIM + 1] - 0.5 * kin * ir);
  r.ua = U[1 + a] * ir;
  r.c = sqrt(gamma * r.p * ir);
  return r;
}

// Rusanov flux, UL on the low side (one reciprocal and one root per side).
template <int DIM>
__device__ inline void rusanov1(const double* UL, const double* UR, int a, double gamma, double* F) {
  const Point<DIM> L = point_of<DIM>(UL, a, gamma), R = point_of<DIM>(UR, a, gamma);
  const double lam = fmax(fabs(L.ua) + L.c, fabs(R.ua) + R.c);
#pragma unroll
  for (int v = 0; v < DIM + 2; ++v) {
    double fl = v == DIM + 1 ? (UL[v] + L.p) * L.ua : UL[v] * L.ua;
    double fr = v == DIM + 1 ? (UR[v] + R.p) * R.ua : UR[v] * R.ua;
    if (v == 1 + a) {
      fl += L.p;
      fr += R.p;
    }
    F[v] = 0.5 * (fl + fr) - 0.5 * lam * (UR[v] - UL[v]);
  }
}

// First point of line q along axis a, and the distance between its points:
// q counts the points of a face normal to a (face_point's order).
template <int DIM, int N>
__device__ inline int line_base(int a, int q) {
  if (a == 0) return q * N;
  if (DIM == 2) return q;
  return a == 1 ? q % N + (q / N) * (N * N) : q;
}
constexpr int line_stride(int n, int a) { return a == 0 ? 1 : (a == 1 ? n : n * n); }

// The hanging faces' codes and mask bits (hm zeroed before), once per call.
__global__ __launch_bounds__(256) void k_fr_rows(const int32_t* __restrict__ hang, int64_t nrows, int dim,
                                                 int64_t n, int32_t* __restrict__ code,
                                                 uint32_t* __restrict__ hm, unsigned* err) {
  const int S = 1 << (dim - 1), nf = 2 * dim, W = 2 + S;
  const int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  const int64_t r = t / (S + 1);
  const int slot = int(t % (S + 1));
  if (r >= nrows) return;
  const int64_t e = slot == S ? hang[r * W] : hang[r * W + 2 + slot];
  const int fc = hang[r * W + 1];
  if (e < 0 || e >= n || fc < 0 || fc >= nf) {
    atomicOr(err, ERR_FR_ROW);
    return;
  }
  const int f = slot == S ? fc : fc ^ 1;
  code[e * nf + f] = int32_t(t);
  atomicOr(&hm[e >> 2], 1u << (8 * int(e & 3) + f));  // one byte per leaf
}

// Fluxes of the hanging faces from the state: one wave per row, lane = (slot
// s, face point q), with the traces formed from the elements' lines.
template <int DIM, int N>
__global__ __launch_bounds__(256) void k_fr_hang(const int32_t* __restrict__ hang, int64_t nrows,
                                                 int64_t n, const double* __restrict__ tab, double gamma,
                                                 const double* __restrict__ u, int64_t ld,
                                                 double* __restrict__ HB) {
  constexpr int NFP = DIM == 3 ? N * N : N;
  constexpr int NP = NFP * N;
  constexpr int S = 1 << (DIM - 1);
  constexpr int NV = DIM + 2;
  constexpr int W = 2 + S;
  static_assert(S * NFP <= 64, "one wave per row");
  __shared__ double Fm[4][S * NFP][NV];  // mortar fluxes of the wave's row
  __shared__ double Uc[4][NFP][NV];      // coarse trace
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t r = int64_t(blockIdx.x) * (blockDim.x >> 6) + wv;
  const int s = lane / NFP, q = lane % NFP;
  int64_t c = 0, k = 0;
  int f = 0;
  if (r < nrows) {
    c = hang[r * W];
    f = hang[r * W + 1];
    if (s < S) k = hang[r * W + 2 + s];
  }
  // rows with a bad entry were reported when their codes were written
  const bool go = r < nrows && s < S && c >= 0 && c < n && f >= 0 && f < 2 * DIM && k >= 0 && k < n;
  const int a = f >> 1, side = f & 1;
  // end values of element e's line through face point q, at its side `hi`
  auto trace = [&](int64_t e, bool hi, double* T) {
    const double* l = tab + (hi ? FrTab::lR(N) : FrTab::lL(N));
    const int b0 = a == 0 ? line_base<DIM, N>(0, q) : (a == 1 ? line_base<DIM, N>(1, q) : line_base<DIM, N>(2, q));
    const int st = line_stride(N, a);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      double x[N];
#pragma unroll
      for (int i = 0; i < N; ++i) x[i] = u[(int64_t(v) * NP + b0 + i * st) * ld + e];
      double t = 0.0;
#pragma unroll
      for (int i = 0; i < N; ++i) t += l[i] * x[i];
      T[v] = t;
    }
  };
  double Uk[NV];
  if (go) {
    trace(k, side == 0, Uk);
    if (s == 0) {
      double T[NV];
      trace(c, side == 1, T);
#pragma unroll
      for (int v = 0; v < NV; ++v) Uc[wv][q][v] = T[v];
    }
  }
  __syncthreads();
  // tangential child bits of mortar s and the face point's tangential indices
  const int b0 = s & 1, b1 = (s >> 1) & 1;
  const int q0 = q % N, q1 = q / N;
  double* out = HB + r * (S + 1) * NV * NFP;
  if (go) {
    const double* A0 = tab + FrTab::A(N, b0);
    const double* A1 = tab + FrTab::A(N, b1);
    double Um[NV], F[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      double acc = 0.0;
      if (DIM == 2) {
#pragma unroll
        for (int i = 0; i < N; ++i) acc += A0[q0 * N + i] * Uc[wv][i][v];
      } else {
#pragma unroll
        for (int i1 = 0; i1 < N; ++i1) {
          double t = 0.0;
#pragma unroll
          for (int i0 = 0; i0 < N; ++i0) t += A0[q0 * N + i0] * Uc[wv][i1 * N + i0][v];
          acc += A1[q1 * N + i1] * t;
        }
      }
      Um[v] = acc;
    }
    double L[NV], H[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      L[v] = side ? Um[v] : Uk[v];
      H[v] = side ? Uk[v] : Um[v];
    }
    if (a == 0)
      rusanov1<DIM>(L, H, 0, gamma, F);
    else if (DIM == 2 || a == 1)
      rusanov1<DIM>(L, H, 1, gamma, F);
    else
      rusanov1<DIM>(L, H, DIM - 1, gamma, F);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      out[(s * NV + v) * NFP + q] = F[v];
      Fm[wv][lane][v] = F[v];
    }
  }
  __syncthreads();
  // coarse face: sum over the mortars of (P_b1 x P_b0) applied to their fluxes
  if (go && s == 0) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      double acc = 0.0;
#pragma unroll
      for (int m = 0; m < S; ++m) {
        const double* P0 = tab + FrTab::P(N, m & 1);
        const double* P1 = tab + FrTab::P(N, (m >> 1) & 1);
        if (DIM == 2) {
#pragma unroll
          for (int i = 0; i < N; ++i) acc += P0[q0 * N + i] * Fm[wv][m * NFP + i][v];
        } else {
#pragma unroll
          for (int i1 = 0; i1 < N; ++i1) {
            double t = 0.0;
#pragma unroll
            for (int i0 = 0; i0 < N; ++i0) t += P0[q0 * N + i0] * Fm[wv][m * NFP + i1 * N + i0][v];
            acc += P1[q1 * N + i1] * t;
          }
        }
      }
      out[(S * NV + v) * NFP + q] = acc;
    }
  }
}

// Elements of a workgroup.  3D keeps the state and the residual sums of its
// elements in LDS (80 KB at p = 3 with 16 elements, so that two workgroups
// share a compute unit), 2D the sums alone.  Few elements in flight also keep
// a neighbour's lines in the L2 (4 MB per XCD) until they are wanted.
constexpr bool stage_lds(int dim) { return dim == 3; }
constexpr int stage_elems(int dim, int n) {
  return dim == 3 ? (n >= 3 ? 16 : 64) : (n >= 7 ? 32 : 64);
}

// Rows of one variable: base address and length in bytes.  A lane that wants
// nothing from a row passes kNoLoad, which lies past any length: the load
// returns zero and reaches no memory, without a branch around it.
constexpr uint32_t kNoLoad = 0xFFFFFFF0u;
__device__ inline __amdgpu_buffer_rsrc_t var_rsrc(const double* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(base), 0, int(bytes), 0x00020000);
}
typedef unsigned int u32x2 __attribute__((__vector_size__(2 * sizeof(unsigned int))));
constexpr int kStream = 2;  // cache-policy bit of the buffer access: streaming

// One stage out = c0 u0 + c1 u + c2 R(u) for EB elements per workgroup: lane =
// element, wave (or wave part) = line.  Axis by axis (z, y, x) the lane takes
// its line, forms the line's end values, the common fluxes and the corrected
// flux derivative along it, and the axes' sums pass from one axis' lines to
// the next through LDS; in 3D the state does too, so that it is read once.  A
// neighbour's end value comes from its lane of the same wave where the
// neighbour is one of the wave's elements (consecutive elements are a block in
// space), else the lane sums the neighbour's own line; those lines are asked
// for at the start, for every axis.  Every lane holds a whole line, so the 1D
// operators are literal constants.
//
// Bound: the reads from beyond the L2, with two waves per SIMD (80 KB of LDS a
// workgroup) waiting for them.  At 1.90M p = 3 elements in 3D a stage reads 17.9 GB
// and writes 5.1 (3.7 and 1.05 times the state, of 1.67 and 1 that three stages
// need on average) at 4.2 TB/s, vector units 38% and LDS 11% busy; a step of three
// stages takes 16.6 ms (35.2 ms with the face buffer, 22.2 with every
// neighbour's line loaded and the state read again for each axis; without the
// lines outside the wave it would take 10.0, of which 3.4 is the issue of their
// loads).  p = 2: 17.2 -> 8.9 ms, p = 1: 6.2 -> 2.0 ms; 2D p = 4, 40 006 leaves, one
// residual: 73 -> 41 us.
// WIDE: 64-bit addresses, for arrays whose rows of one variable pass 2^32
// bytes.
template <int DIM, int N, bool WIDE>
__global__ __launch_bounds__(stage_elems(DIM, N) * (DIM == 3 ? N * N : N), 2) void k_fr_stage(
    KeyGeom g, const uint64_t* __restrict__ keys, const int32_t* __restrict__ nbr,
    const uint8_t* __restrict__ hm, const int32_t* __restrict__ code, const double* __restrict__ HB,
    int64_t n, double length, double gamma, const double* __restrict__ u, int64_t ld,
    const double* u0, int64_t ld0, double c0, double c1, double c2, double* out, int64_t ldo,
    unsigned* err) {
  constexpr int NL = DIM == 3 ? N * N : N;  // lines along each axis, points of a face
  constexpr int NP = NL * N;
  constexpr int NV = DIM + 2;
  constexpr int EB = stage_elems(DIM, N);
  constexpr Ops1D<N> O = ops_1d<N>();
  const double* D = O.t + FrTab::kD;
  const double* lL = O.t + FrTab::lL(N);
  const double* lR = O.t + FrTab::lR(N);
  const double* dgL = O.t + FrTab::dgL(N);
  const double* dgR = O.t + FrTab::dgR(N);
  constexpr bool kLds = stage_lds(DIM);
  __shared__ double Rs[NV * NP * EB];
  __shared__ double Us[kLds ? NV * NP * EB : 1];
  const int lane = threadIdx.x & 63;
  const int el = threadIdx.x % EB;
  // the lane's line
  const int q = EB == 64 ? __builtin_amdgcn_readfirstlane(threadIdx.x / EB) : int(threadIdx.x / EB);
  // contiguous runs of elements per XCD (workgroups are dealt round-robin), so
  // that neighbouring lines are read into one L2
  const int64_t nb = gridDim.x, bq = nb >> 3, br = nb & 7;
  const int64_t bx = blockIdx.x & 7, bk = blockIdx.x >> 3;
  const int64_t e0 = (bx * bq + (bx < br ? bx : br) + bk) * EB;
  const bool live = e0 + el < n;
  const int64_t e = live ? e0 + el : n - 1;  // lanes past the end repeat the last element
  int32_t nbe[2 * DIM];
#pragma unroll
  for (int f = 0; f < 2 * DIM; ++f) nbe[f] = nbr[e * (2 * DIM) + f];
  const unsigned hmask = hm[e];
  const double gm1 = gamma - 1.0;
  const double scale = -2.0 / ldexp(length, -key_depth(g, keys[e]));
  const uint32_t bytes = uint32_t(NP * ld * 8);
  // value of variable v at point row `row` (uniform) + lane's part: element j
  // at point `base` of the lane's line
  auto load = [&](int v, int row, int base, int64_t j, bool want) -> double {
    if constexpr (WIDE) {
      const double x = u[int64_t(v * NP + row + base) * ld + (want ? j : e)];
      return want ? x : 0.0;
    } else {
      const uint32_t o = want ? uint32_t((uint32_t(base) * uint64_t(ld) + j) * 8) : kNoLoad;
      return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(
                                            var_rsrc(u + int64_t(v) * NP * ld, bytes), o,
                                            uint32_t(row * ld * 8), 0));
    }
  };
  // 16-element rows start on alternate halves of the banks; swapping point
  // pairs by bit 2 spreads the lines of every axis over both halves
  auto at = [&](int v, int pt) {
    if (EB == 16) pt ^= (pt >> 2) & 1;
    return (v * NP + pt) * EB + el;
  };
  // Hanging faces take their flux from HB; neighbours in the wave are
  // exchanged, the others' lines are read: their end values, per axis.
  bool xl[DIM], xr[DIM];
  int sl[DIM], sr[DIM];
  double zl[DIM][NV], zr[DIM][NV];
  auto outside = [&](int a) {
    const int base = line_base<DIM, N>(a, q);
    const int st = line_stride(N, a);
    const bool hl = (hmask >> (2 * a)) & 1u, hr = (hmask >> (2 * a + 1)) & 1u;
    const int64_t nl = nbe[2 * a], nr = nbe[2 * a + 1];
    const bool okl = nl >= 0 && nl < n, okr = nr >= 0 && nr < n;
    if ((!hl && !okl) || (!hr && !okr)) atomicOr(err, ERR_INVALID_TREE);
    const bool inl = nl >= e0 && nl < e0 + EB, inr = nr >= e0 && nr < e0 + EB;
    xl[a] = !hl && okl && !inl;
    xr[a] = !hr && okr && !inr;
    sl[a] = (lane & ~(EB - 1)) + (inl ? int(nl - e0) : el);
    sr[a] = (lane & ~(EB - 1)) + (inr ? int(nr - e0) : el);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      zl[a][v] = zr[a][v] = 0.0;
#pragma unroll
      for (int k = 0; k < N; ++k) {
        zl[a][v] += lR[k] * load(v, k * st, base, nl, xl[a]);
        zr[a][v] += lL[k] * load(v, k * st, base, nr, xr[a]);
      }
    }
  };
  // asked for an axis ahead where the registers hold it
  constexpr bool kAhead = DIM == 3 || N <= 4;
  double U[NV][N], U0[kAhead ? NV : 1][N];
  constexpr int kFirst = DIM - 1;
#pragma unroll
  for (int v = 0; v < (kAhead ? NV : 1); ++v)
#pragma unroll
    for (int k = 0; k < N; ++k) U0[v][k] = 0.0;
  auto load_u0 = [&](int v, double* x) {
#pragma unroll
    for (int k = 0; k < N; ++k)
      x[k] = __builtin_nontemporal_load(u0 + int64_t(v * NP + line_base<DIM, N>(0, q) + k) * ld0 + e);
  };
#pragma unroll
  for (int v = 0; v < NV; ++v)
#pragma unroll
    for (int k = 0; k < N; ++k) U[v][k] = load(v, k * line_stride(N, kFirst), line_base<DIM, N>(kFirst, q), e, true);
  outside(kFirst);
  if constexpr (kLds)
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
      for (int k = 0; k < N; ++k)
        Us[at(v, line_base<DIM, N>(kFirst, q) + k * line_stride(N, kFirst))] = U[v][k];
#pragma unroll
  for (int a = DIM - 1; a >= 0; --a) {
    const int base = line_base<DIM, N>(a, q);
    const int st = line_stride(N, a);
    const bool hl = (hmask >> (2 * a)) & 1u, hr = (hmask >> (2 * a + 1)) & 1u;
    if (a != kFirst) {
      if constexpr (!kLds)
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
          for (int k = 0; k < N; ++k) U[v][k] = load(v, k * st, base, e, true);
      __syncthreads();  // the sums (and the state) of the axis before
      if constexpr (kLds)
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
          for (int k = 0; k < N; ++k) U[v][k] = Us[at(v, base + k * st)];
    }
    if (!kAhead) {
      if (a != kFirst) outside(a);
    } else if (a > 0) {
      outside(a - 1);
    } else if (c0 != 0.0) {
      // u0's line at once: point by point each load would wait for the
      // stores before it
#pragma unroll
      for (int v = 0; v < NV; ++v) load_u0(v, U0[kAhead ? v : 0]);
    }
    double FL[NV], FR[NV];
    {
      double tl[NV], tr[NV], yl[NV], yr[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        tl[v] = tr[v] = 0.0;
#pragma unroll
        for (int k = 0; k < N; ++k) {
          tl[v] += lL[k] * U[v][k];
          tr[v] += lR[k] * U[v][k];
        }
        const double wl = __shfl(tr[v], sl[a]), wr = __shfl(tl[v], sr[a]);
        yl[v] = xl[a] ? zl[a][v] : wl;
        yr[v] = xr[a] ? zr[a][v] : wr;
      }
      rusanov1<DIM>(yl, tl, a, gamma, FL);
      rusanov1<DIM>(tr, yr, a, gamma, FR);
    }
    if (hl) {
      const double* F = HB + int64_t(code[e * (2 * DIM) + 2 * a]) * (NV * NL) + q;
#pragma unroll
      for (int v = 0; v < NV; ++v) FL[v] = F[v * NL];
    }
    if (hr) {
      const double* F = HB + int64_t(code[e * (2 * DIM) + 2 * a + 1]) * (NV * NL) + q;
#pragma unroll
      for (int v = 0; v < NV; ++v) FR[v] = F[v * NL];
    }
    double ua[N], pr[N];
#pragma unroll
    for (int k = 0; k < N; ++k) {
      const double ir = 1.0 / U[0][k];
      double kin = 0.0;
#pragma unroll
      for (int b = 0; b < DIM; ++b) kin += U[1 + b][k] * U[1 + b][k];
      pr[k] = gm1 * (U[NV - 1][k] - 0.5 * kin * ir);
      ua[k] = U[1 + a][k] * ir;
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      double F[N], fl = 0.0, fr = 0.0;
#pragma unroll
      for (int k = 0; k < N; ++k) {
        F[k] = (U[v][k] + (v == NV - 1 ? pr[k] : 0.0)) * ua[k] + (v == 1 + a ? pr[k] : 0.0);
        fl += lL[k] * F[k];
        fr += lR[k] * F[k];
      }
      const double jl = FL[v] - fl, jr = FR[v] - fr;
      double R[N];
#pragma unroll
      for (int i = 0; i < N; ++i) {
        double d = dgL[i] * jl + dgR[i] * jr;
#pragma unroll
        for (int k = 0; k < N; ++k) d += D[i * N + k] * F[k];
        R[i] = a == kFirst ? d : d + Rs[at(v, base + i * st)];
      }
      if (a > 0) {
#pragma unroll
        for (int i = 0; i < N; ++i) Rs[at(v, base + i * st)] = R[i];
      } else if (live) {
        double* w = U0[kAhead ? v : 0];
        if (!kAhead && c0 != 0.0) load_u0(v, w);
#pragma unroll
        for (int i = 0; i < N; ++i) {
          const int64_t row = int64_t(v * NP + base + i);
          const double r = c1 * U[v][i] + c2 * (scale * R[i]);
          __builtin_nontemporal_store(c0 != 0.0 ? r + c0 * w[i] : r, out + row * ldo + e);
        }
      }
    }
  }
}

template <int DIM, int N>
lt_status fr_faces(lt_tree_s* t, const double* u, int64_t ld, const double* tab, double gamma,
                   double* fb, int64_t ldf, hipStream_t s) {
  const int64_t n = t->n_cur;
  k_fr_trace<DIM, N><<<unsigned((n + 255) / 256), 256, 0, s>>>(u, ld, n, tab, fb, ldf);
  k_fr_conf<DIM, N><<<unsigned((n + 255) / 256), 256, 0, s>>>(t->g, t->kbuf[t->cur], t->nbr, n, gamma,
                                                              fb, ldf, &t->dctr->err);
  if (t->n_hang > 0)
    k_fr_mortar<DIM, N><<<unsigned((t->n_hang + 3) / 4), 256, 0, s>>>(t->hang, t->n_hang, n, tab, gamma,
                                                                       fb, ldf, &t->dctr->err);
  if (hipGetLastError() != hipSuccess) return fail(LT_ERR_HIP, "FR face kernels launch");
  return LT_OK;
}

// Hanging-face tables of the current connectivity, for the stages of one call.
lt_status fr_rows(lt_tree_s* t, int p, hipStream_t s) {
  const int64_t n = t->n_cur, rows = t->n_hang;
  const int dim = t->g.dim, S = 1 << (dim - 1);
  int64_t nfp = 1;
  for (int a = 0; a < dim - 1; ++a) nfp *= p + 1;
  LT_TRY_STATUS(grow(t->A, &t->fr_hm, &t->fr_hm_cap, (n + 3) / 4));
  LT_TRY_STATUS(grow(t->A, &t->fr_code, &t->fr_code_cap, n * 2 * dim));
  LT_TRY_STATUS(grow(t->A, &t->fr_hb, &t->fr_hb_cap, std::max<int64_t>(rows, 1) * (S + 1) * (dim + 2) * nfp));
  launch_fill_u32(t->fr_hm, (n + 3) / 4, 0u, s);
  if (rows > 0)
    k_fr_rows<<<unsigned((rows * (S + 1) + 255) / 256), 256, 0, s>>>(t->hang, rows, dim, n, t->fr_code,
                                                                    t->fr_hm, &t->dctr->err);
  if (hipGetLastError() != hipSuccess) return fail(LT_ERR_HIP, "FR row kernels launch");
  return LT_OK;
}

template <int DIM, int N>
lt_status fr_stage(lt_tree_s* t, const double* tab, double length, double gamma, const double* uin,
                   int64_t ld, const double* u0, int64_t ld0, double c0, double c1, double c2, double* out,
                   int64_t ldo, hipStream_t s) {
  const int64_t n = t->n_cur;
  constexpr int NL = DIM == 3 ? N * N : N;
  constexpr int EB = stage_elems(DIM, N);
  if (t->n_hang > 0)
    k_fr_hang<DIM, N><<<unsigned((t->n_hang + 3) / 4), 256, 0, s>>>(t->hang, t->n_hang, n, tab, gamma, uin,
                                                                    ld, t->fr_hb);
  const unsigned blocks = unsigned((n + EB - 1) / EB);
  const uint8_t* hm = reinterpret_cast<const uint8_t*>(t->fr_hm);
  // one variable's rows within 32-bit byte offsets (8.3M leaves at p = 3 in
  // 3D), and short of the offset that stands for no load
  if (int64_t(NL) * N * ld * 8 <= int64_t(kNoLoad))
    k_fr_stage<DIM, N, false><<<blocks, EB * NL, 0, s>>>(t->g, t->kbuf[t->cur], t->nbr, hm, t->fr_code,
                                                         t->fr_hb, n, length, gamma, uin, ld, u0, ld0, c0, c1,
                                                         c2, out, ldo, &t->dctr->err);
  else
    k_fr_stage<DIM, N, true><<<blocks, EB * NL, 0, s>>>(t->g, t->kbuf[t->cur], t->nbr, hm, t->fr_code,
                                                        t->fr_hb, n, length, gamma, uin, ld, u0, ld0, c0, c1,
                                                        c2, out, ldo, &t->dctr->err);
  if (hipGetLastError() != hipSuccess) return fail(LT_ERR_HIP, "FR stage kernel launch");
  return LT_OK;
}

}  // namespace
}  // namespace lt

// ------------------------------------------------------------------ entry points
namespace lt {
namespace {

lt_status fr_check(lt_tree_s* t, int p, const char* who) {
  if (!t) return fail(LT_ERR_ARG, std::string(who) + ": NULL tree");
  const int dim = t->g.dim;
  if ((dim == 3 && (p < 1 || p > 3)) || (dim == 2 && (p < 1 || p > LT_MAX_DEGREE)))
    return fail(LT_ERR_ARG, std::string(who) + ": p must be 1..3 in 3D, 1..7 in 2D");
  if (t->g.nmesh != 1) return fail(LT_ERR_ARG, std::string(who) + ": one tree, not an ensemble");
  if (t->g.periodic != (1u << dim) - 1u)
    return fail(LT_ERR_ARG, std::string(who) + ": the domain must be periodic on every axis");
  if (!t->conn_valid) return fail(LT_ERR_STATE, std::string(who) + ": needs lt_connect on the current leaves");
  if (t->n_cur < 1) return fail(LT_ERR_ARG, std::string(who) + ": empty tree");
  return LT_OK;
}

lt_status fr_tab(lt_tree_s* t, int p, hipStream_t s, const double** out) {
  if (!t->fr_tab[p]) {
    const std::vector<double> T = fr_tables(p);
    void* q = nullptr;
    if (dev_malloc(t->A, &q, T.size() * sizeof(double)) != hipSuccess) return fail(LT_ERR_OOM, "FR tables");
    if (hipMemcpyAsync(q, T.data(), T.size() * sizeof(double), hipMemcpyHostToDevice, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess) {
      (void)dev_free(t->A, q);
      return fail(LT_ERR_HIP, "FR table upload");
    }
    t->fr_tab[p] = static_cast<double*>(q);
  }
  *out = t->fr_tab[p];
  return LT_OK;
}

lt_status faces(lt_tree_s* t, int p, const double* u, int64_t ld, const double* tab, double gamma,
                double* fb, int64_t ldf, hipStream_t s) {
#define LT_F(D, NN) return fr_faces<D, NN>(t, u, ld, tab, gamma, fb, ldf, s)
  if (t->g.dim == 3) {
    switch (p) {
      case 1: LT_F(3, 2);
      case 2: LT_F(3, 3);
      default: LT_F(3, 4);
    }
  }
  switch (p) {
    case 1: LT_F(2, 2);
    case 2: LT_F(2, 3);
    case 3: LT_F(2, 4);
    case 4: LT_F(2, 5);
    case 5: LT_F(2, 6);
    case 6: LT_F(2, 7);
    default: LT_F(2, 8);
  }
#undef LT_F
}

lt_status stage(lt_tree_s* t, int p, const double* tab, double length, double gamma, const double* uin,
                int64_t ld, const double* u0, int64_t ld0, double c0, double c1, double c2, double* out,
                int64_t ldo, hipStream_t s) {
#define LT_V(D, NN) return fr_stage<D, NN>(t, tab, length, gamma, uin, ld, u0, ld0, c0, c1, c2, out, ldo, s)
  if (t->g.dim == 3) {
    switch (p) {
      case 1: LT_V(3, 2);
      case 2: LT_V(3, 3);
      default: LT_V(3, 4);
    }
  }
  switch (p) {
    case 1: LT_V(2, 2);
    case 2: LT_V(2, 3);
    case 3: LT_V(2, 4);
    case 4: LT_V(2, 5);
    case 5: LT_V(2, 6);
    case 6: LT_V(2, 7);
    default: LT_V(2, 8);
  }
#undef LT_V
}

}  // namespace
}  // namespace lt

using namespace lt;

extern "C" {

lt_status lt_fr_face_flux(lt_tree t, int p, const double* u, int64_t ld, double gamma, double* fhat,
                          int64_t ld_f, void* stream) {
  LT_TRY_STATUS(fr_check(t, p, "lt_fr_face_flux"));
  if (!u || !fhat) return fail(LT_ERR_ARG, "NULL argument");
  if (ld < t->n_cur || ld_f < t->n_cur) return fail(LT_ERR_ARG, "leading dimension too small");
  if (!(gamma > 1.0)) return fail(LT_ERR_ARG, "gamma must exceed 1");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const double* tab = nullptr;
  LT_TRY_STATUS(fr_tab(t, p, s, &tab));
  return faces(t, p, u, ld, tab, gamma, fhat, ld_f, s);
}

lt_status lt_fr_residual(lt_tree t, int p, const double* u, int64_t ld, double gamma, double length,
                         double* R, int64_t ld_r, void* stream) {
  LT_TRY_STATUS(fr_check(t, p, "lt_fr_residual"));
  if (!u || !R || u == R) return fail(LT_ERR_ARG, "NULL argument or R aliasing u");
  if (ld < t->n_cur || ld_r < t->n_cur) return fail(LT_ERR_ARG, "leading dimension too small");
  if (!(gamma > 1.0) || !(length > 0.0)) return fail(LT_ERR_ARG, "gamma must exceed 1, length be positive");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const double* tab = nullptr;
  LT_TRY_STATUS(fr_tab(t, p, s, &tab));
  LT_TRY_STATUS(fr_rows(t, p, s));
  return stage(t, p, tab, length, gamma, u, ld, u, ld, 0.0, 0.0, 1.0, R, ld_r, s);
}

lt_status lt_fr_rk3(lt_tree t, int p, double* u, int64_t ld, double* work, double dt, double gamma,
                    double length, int steps, void* stream) {
  LT_TRY_STATUS(fr_check(t, p, "lt_fr_rk3"));
  if (!u || !work || u == work) return fail(LT_ERR_ARG, "NULL argument or work aliasing u");
  if (ld < t->n_cur) return fail(LT_ERR_ARG, "leading dimension too small");
  if (!(gamma > 1.0) || !(length > 0.0) || !(dt > 0.0) || steps < 0)
    return fail(LT_ERR_ARG, "gamma must exceed 1, length and dt be positive, steps >= 0");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const double* tab = nullptr;
  LT_TRY_STATUS(fr_tab(t, p, s, &tab));
  if (steps == 0) return LT_OK;
  LT_TRY_STATUS(fr_rows(t, p, s));
  // the first stage's result: a stage reads its neighbours' state, so it
  // cannot write where it reads
  int64_t np = 1;
  for (int a = 0; a < t->g.dim; ++a) np *= p + 1;
  const int64_t n = t->n_cur;
  LT_TRY_STATUS(grow(t->A, &t->fr_u1, &t->fr_u1_cap, (t->g.dim + 2) * np * n));
  double* u1 = t->fr_u1;
  for (int k = 0; k < steps; ++k) {
    // u1 = u + dt R(u)
    LT_TRY_STATUS(stage(t, p, tab, length, gamma, u, ld, u, ld, 0.0, 1.0, dt, u1, n, s));
    // u2 = 3/4 u + 1/4 u1 + 1/4 dt R(u1)
    LT_TRY_STATUS(stage(t, p, tab, length, gamma, u1, n, u, ld, 0.75, 0.25, 0.25 * dt, work, ld, s));
    // u_next = 1/3 u + 2/3 u2 + 2/3 dt R(u2)   (written over u)
    LT_TRY_STATUS(stage(t, p, tab, length, gamma, work, ld, u, ld, 1.0 / 3.0, 2.0 / 3.0, 2.0 / 3.0 * dt, u,
                        ld, s));
  }
  return LT_OK;
}

}  // extern "C"

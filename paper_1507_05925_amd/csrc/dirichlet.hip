// Capacitance and resistance problems: the inverse problems that the paper's numerical section
// solves to test the elastance and mobility solvers (prescribed potentials -> charges; prescribed
// rigid motions -> forces and torques). The paper leaves their equations to the literature; these
// are the classical completed double layers.
//
// Laplace: u = D[mu] + sum_j G_R(x, z_j) int_{Gamma_j} mu, with D[mu](x) = int dG/dn_y mu ds_y,
//   G = -(1/2pi) log|x - y|, G_R(x, z) = -(1/2pi) log(|x - z| / R); exterior boundary values give
//   (1/2 I + D + C) mu = f.
// Stokes: u = Dcal[mu] + sum_j [Gcal_R(x, z_j) a_j + t_j (x - z_j)^perp / (4 pi |x - z_j|^2)],
//   Dcal[mu](x) = (1/pi) int (r.n_y)(r.mu) r / |r|^4 ds_y (r = x - y), the Stokeslet
//   Gcal_R = (1/4pi)(-log(|d|/R) I + d d^T / |d|^2), a_j = int_{Gamma_j} mu,
//   t_j = int_{Gamma_j} ((y - z_j)^perp, mu).
// z_j are the geometry's interior points and R twice the diagonal of the nodes' bounding box.
// The equations hold any boundary data; the bounded solution of the physical problem (u tends to
// a constant, net charge / force zero) is a combination of the data solve with the solves for
// f = 1 (Laplace), resp. f = e_x and e_y (Stokes).
//
// The double-layer sweep is the float64 pair sweep of the direct apply with the sources' normals
// (pairs.h), over all pairs; the smooth diagonal limit is added in the epilogue.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>

#include "internal.h"
#include "pairs.h"

namespace bie {

namespace {

__device__ inline double wg_sum(double v, double *sh) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) sh[wid] = v;
  __syncthreads();
  const double t = (sh[0] + sh[1]) + (sh[2] + sh[3]);
  __syncthreads();
  return t;
}

// Moments of density r over body b: Laplace int mu (one value); Stokes a = int mu (two) and
// t = int ((y - z)^perp, mu) about the body's interior point z. One workgroup; sh: 4 doubles of LDS.
struct MomentArgs {
  const int *body_ptr;
  const double *x, *y, *w, *pint, *mu;
  long long len;
  double *mom;
  int N;
};

template <bool STOKES>
__device__ void moments(const MomentArgs &a, int b, int r, double *sh) {
  const int k0 = a.body_ptr[b], k1 = a.body_ptr[b + 1];
  const double *m = a.mu + (size_t)r * a.len;
  const double zx = a.pint[2 * b], zy = a.pint[2 * b + 1];
  double a1 = 0.0, a2 = 0.0, t = 0.0;
  for (int k = k0 + threadIdx.x; k < k1; k += kBlock) {
    if (!STOKES) {
      a1 += a.w[k] * m[k];
    } else {
      const double m1 = a.w[k] * m[2 * k], m2 = a.w[k] * m[2 * k + 1];
      a1 += m1;
      a2 += m2;
      t += (a.x[k] - zx) * m2 - (a.y[k] - zy) * m1;
    }
  }
  a1 = wg_sum(a1, sh);
  if (STOKES) {
    a2 = wg_sum(a2, sh);
    t = wg_sum(t, sh);
  }
  if (threadIdx.x == 0) {
    if (!STOKES) {
      a.mom[(size_t)r * a.N + b] = a1;
    } else {
      double *o = a.mom + ((size_t)r * a.N + b) * 3;
      o[0] = a1;
      o[1] = a2;
      o[2] = t;
    }
  }
}

// Grid (bodies, densities).
template <bool STOKES>
__global__ __launch_bounds__(kBlock) void k_dl_moments(MomentArgs a) {
  __shared__ double sh[4];
  moments<STOKES>(a, blockIdx.x, blockIdx.y, sh);
}

// Double-layer pair sums of R densities (pairs.h), Laplace (1/2pi) sum_k w_k mu_k (r.n_k) / |r|^2,
// Stokes (1/pi) sum_k (r.n_k)(r.w_k mu_k) r / |r|^4, and in the same launch the densities'
// moments: workgroups [0, N R) form those (few and short; they start first), the others take
// (tile, split) of the sweep.
template <int KIND, int R>
__global__ __launch_bounds__(kBlock, sweep_occupancy(PairShape<KIND, R>::V)) void k_dl_sweep(
    int M, int per, int tiles, int nmom, MomentArgs ma, PairSources src, double factor,
    double *__restrict__ partial) {
  __shared__ double buf[kSweepLds<KIND, R>];
  const int w = blockIdx.x - nmom;
  if (w < 0) {
    moments<KIND == kPairStkDl>(ma, blockIdx.x % ma.N, blockIdx.x / ma.N, buf);
    return;
  }
  const int sp = w / tiles, k0 = sp * per;
  pair_sweep_tile<KIND, R>((w % tiles) * kSweepTile, M, k0, min(k0 + per, M), src, factor,
                           partial + (size_t)sp * R * src.len, buf);
}

// out = alpha (1/2 mu + diagonal limit + sum of the split partials + completion), grid.y = density.
// What bounds it is latency: geometries of this path have few nodes, and a node's splits and bodies
// (a logarithm, for Stokes also a division, each) are two serial chains. So kEpiLanes lanes share a
// node: lane g takes the splits and the bodies g, g + kEpiLanes, ... and three shuffle steps add
// the lanes in a fixed order (splash geometry, 3 Stokes densities: one lane per node 7.3 us,
// eight 4.2 us).
constexpr int kEpi = 64;  // one wave per workgroup
constexpr int kEpiLanes = 8;

__device__ __forceinline__ double epi_sum(double v) {
#pragma unroll
  for (int off = 1; off < kEpiLanes; off <<= 1) v += __shfl_xor(v, off, 64);
  return v;
}

template <bool STOKES>
__global__ __launch_bounds__(kEpi) void k_dl_epilogue(
    int M, int N, int S, int R, const double2 *__restrict__ xy, const double *__restrict__ nx,
    const double *__restrict__ ny, const double *__restrict__ w, const double *__restrict__ kappa,
    const double *__restrict__ pint, const double *__restrict__ scale, const double *__restrict__ mu,
    long long len, const double *__restrict__ partial, const double *__restrict__ mom,
    int with_C, double alpha, double *__restrict__ out) {
  const int t = blockIdx.x * (kEpi / kEpiLanes) + threadIdx.x / kEpiLanes;
  const int g = threadIdx.x % kEpiLanes;
  const int i = min(t, M - 1);  // lanes past the end take part in the shuffles
  const int r = blockIdx.y;
  const double2 p = xy[i];
  const double *m = mu + (size_t)r * len;
  if (!STOKES) {
    const double mi = m[i], kw = kappa[i] * w[i];
    double far = 0.0, c = 0.0, tot = 0.0;
    for (int sp = g; sp < S; sp += kEpiLanes) far += partial[((size_t)sp * R + r) * len + i];
    if (with_C) {
      const double *A = mom + (size_t)r * N;
      for (int b = g; b < N; b += kEpiLanes) {
        const double dx = p.x - pint[2 * b], dy = p.y - pint[2 * b + 1];
        c = fma(A[b], log(fma(dx, dx, dy * dy)), c);
        tot += A[b];
      }
      c = -(0.5 * c - log(scale[0]) * tot) / (2.0 * kPi);
    }
    far = epi_sum(far + c);
    if (g == 0 && t < M)
      out[(size_t)r * len + i] = alpha * (0.5 * mi - kw / (4.0 * kPi) * mi + far);
  } else {
    const double m1 = m[2 * i], m2 = m[2 * i + 1], kw = kappa[i] * w[i];
    const double tx = -ny[i], ty = nx[i];  // unit tangent (n = (tau_2, -tau_1))
    double f1 = 0.0, f2 = 0.0, u1 = 0.0, u2 = 0.0;
    for (int sp = g; sp < S; sp += kEpiLanes) {
      const double *o = partial + ((size_t)sp * R + r) * len;
      f1 += o[2 * i];
      f2 += o[2 * i + 1];
    }
    if (with_C) {
      const double logR = log(scale[0]);
      const double *A = mom + (size_t)r * N * 3;
      for (int b = g; b < N; b += kEpiLanes) {
        const double dx = p.x - pint[2 * b], dy = p.y - pint[2 * b + 1];
        const double dd = fma(dx, dx, dy * dy);
        const double inv = 1.0 / dd;
        const double lg = 0.5 * log(dd) - logR;
        const double a1 = A[3 * b], a2 = A[3 * b + 1], q = A[3 * b + 2];
        const double da = fma(dx, a1, dy * a2) * inv;
        u1 += -lg * a1 + dx * da - q * dy * inv;
        u2 += -lg * a2 + dy * da + q * dx * inv;
      }
    }
    f1 = epi_sum(f1 + u1 / (4.0 * kPi));
    f2 = epi_sum(f2 + u2 / (4.0 * kPi));
    const double d = -kw / (2.0 * kPi) * fma(tx, m1, ty * m2);
    if (g == 0 && t < M) {
      double *o = out + (size_t)r * len;
      o[2 * i] = alpha * (0.5 * m1 + d * tx + f1);
      o[2 * i + 1] = alpha * (0.5 * m2 + d * ty + f2);
    }
  }
}

// Boundary data of the capacitance systems: rows r < nrhs hold phi_{body(i)}, the last row 1.
__global__ void k_cap_rhs(int M, int N, int nrhs, const int *__restrict__ body_of,
                          const double *__restrict__ phi, double *__restrict__ f) {
  const long long t = (long long)blockIdx.x * kBlock + threadIdx.x;
  if (t >= (long long)(nrhs + 1) * M) return;
  const int r = (int)(t / M), i = (int)(t % M);
  f[t] = r < nrhs ? phi[(size_t)r * N + body_of[i]] : 1.0;
}

// Resistance systems: rows r < nrhs hold v_j + omega_j (x - x^c_j)^perp, then e_x and e_y.
__global__ void k_res_rhs(int M, int N, int nrhs, const int *__restrict__ body_of,
                          const double *__restrict__ px, const double *__restrict__ py,
                          const double *__restrict__ VW, double *__restrict__ f) {
  const long long t = (long long)blockIdx.x * kBlock + threadIdx.x;
  if (t >= (long long)(nrhs + 2) * M) return;
  const int r = (int)(t / M), i = (int)(t % M);
  double u1, u2;
  if (r < nrhs) {
    const double *v = VW + ((size_t)r * N + body_of[i]) * 3;
    u1 = v[0] + v[2] * px[i];
    u2 = v[1] + v[2] * py[i];
  } else {
    u1 = r == nrhs ? 1.0 : 0.0;
    u2 = r == nrhs ? 0.0 : 1.0;
  }
  f[(size_t)r * 2 * M + 2 * i] = u1;
  f[(size_t)r * 2 * M + 2 * i + 1] = u2;
}

// Bounded capacitance solution of density r (one workgroup each): beta = sum q~[r] / sum q~[1],
// q = q~[r] - beta q~[1], u_inf = beta.
__global__ __launch_bounds__(kBlock) void k_cap_combine(int N, int nrhs,
                                                        const double *__restrict__ mom,
                                                        double *__restrict__ q,
                                                        double *__restrict__ u_inf,
                                                        double *__restrict__ beta) {
  __shared__ double sh[4];
  const int r = blockIdx.x;
  const double *A = mom + (size_t)r * N, *A1 = mom + (size_t)nrhs * N;
  double s = 0.0, s1 = 0.0;
  for (int b = threadIdx.x; b < N; b += kBlock) {
    s += A[b];
    s1 += A1[b];
  }
  s = wg_sum(s, sh);
  s1 = wg_sum(s1, sh);
  const double be = s / s1;
  for (int b = threadIdx.x; b < N; b += kBlock) q[(size_t)r * N + b] = A[b] - be * A1[b];
  if (threadIdx.x == 0) {
    u_inf[r] = be;
    beta[2 * r] = be;
    beta[2 * r + 1] = 0.0;
  }
}

// Bounded resistance solution of density r: beta solves [sum a[e_x], sum a[e_y]] beta = sum a[r];
// F = a[r] - beta_1 a[e_x] - beta_2 a[e_y] (likewise t); torque about the centroid
// T = t + (z - x^c) x F; u_inf = beta.
__global__ __launch_bounds__(kBlock) void k_res_combine(int N, int nrhs,
                                                        const double *__restrict__ mom,
                                                        const double *__restrict__ pint,
                                                        const double *__restrict__ xc,
                                                        const double *__restrict__ yc,
                                                        double *__restrict__ FT,
                                                        double *__restrict__ u_inf,
                                                        double *__restrict__ beta) {
  __shared__ double sh[4];
  const int r = blockIdx.x;
  const double *A = mom + (size_t)r * N * 3, *X = mom + (size_t)nrhs * N * 3,
               *Y = mom + (size_t)(nrhs + 1) * N * 3;
  double s1 = 0.0, s2 = 0.0, x1 = 0.0, x2 = 0.0, y1 = 0.0, y2 = 0.0;
  for (int b = threadIdx.x; b < N; b += kBlock) {
    s1 += A[3 * b];
    s2 += A[3 * b + 1];
    x1 += X[3 * b];
    x2 += X[3 * b + 1];
    y1 += Y[3 * b];
    y2 += Y[3 * b + 1];
  }
  s1 = wg_sum(s1, sh);
  s2 = wg_sum(s2, sh);
  x1 = wg_sum(x1, sh);
  x2 = wg_sum(x2, sh);
  y1 = wg_sum(y1, sh);
  y2 = wg_sum(y2, sh);
  const double det = x1 * y2 - y1 * x2;
  const double b1 = (s1 * y2 - y1 * s2) / det, b2 = (x1 * s2 - s1 * x2) / det;
  for (int b = threadIdx.x; b < N; b += kBlock) {
    const double F1 = A[3 * b] - b1 * X[3 * b] - b2 * Y[3 * b];
    const double F2 = A[3 * b + 1] - b1 * X[3 * b + 1] - b2 * Y[3 * b + 1];
    const double t = A[3 * b + 2] - b1 * X[3 * b + 2] - b2 * Y[3 * b + 2];
    const double e1 = pint[2 * b] - xc[b], e2 = pint[2 * b + 1] - yc[b];
    double *o = FT + ((size_t)r * N + b) * 3;
    o[0] = F1;
    o[1] = F2;
    o[2] = t + e1 * F2 - e2 * F1;
  }
  if (threadIdx.x == 0) {
    u_inf[2 * r] = b1;
    u_inf[2 * r + 1] = b2;
    beta[2 * r] = b1;
    beta[2 * r + 1] = b2;
  }
}

// Density of the bounded solution: mu[r] - beta_1 mu[nrhs] (- beta_2 mu[nrhs + 1] for Stokes).
__global__ void k_dl_density(long long len, int nrhs, int extra, const double *__restrict__ beta,
                             const double *__restrict__ mu, double *__restrict__ out) {
  const long long t = (long long)blockIdx.x * kBlock + threadIdx.x;
  if (t >= (long long)nrhs * len) return;
  const int r = (int)(t / len);
  const long long j = t % len;
  double v = mu[t] - beta[2 * r] * mu[(size_t)nrhs * len + j];
  if (extra == 2) v -= beta[2 * r + 1] * mu[(size_t)(nrhs + 1) * len + j];
  out[t] = v;
}

inline unsigned nb(long long n) { return (unsigned)((n + kBlock - 1) / kBlock); }

MomentArgs moment_args(const bie_geom *g, long long len, const double *mu, double *mom) {
  return MomentArgs{g->body_ptr, g->x, g->y, g->w, g->pint, mu, len, mom, g->N};
}

template <int KIND, int R>
void launch_sweep(bie_geom *g, int S, bool with_C, const double *mu, long long len, double *mom,
                  double *partial, hipStream_t st) {
  const int tiles = (g->M + kSweepTile - 1) / kSweepTile, nmom = with_C ? g->N * R : 0;
  hipLaunchKernelGGL((k_dl_sweep<KIND, R>), dim3(nmom + tiles * S), dim3(kBlock), 0, st, g->M,
                     (g->M + S - 1) / S, tiles, nmom, moment_args(g, len, mu, mom),
                     PairSources{g->xy, g->nx, g->ny, g->w, mu, len, g->pair_scale, g->pair_away},
                     (KIND == kPairStkDl ? 1.0 : 0.5) / kPi, partial);
}

template <int KIND>
void sweep_chunk(bie_geom *g, int S, int R, bool with_C, const double *mu, long long len,
                 double *mom, double *partial, hipStream_t st) {
  switch (R) {
    case 4: launch_sweep<KIND, 4>(g, S, with_C, mu, len, mom, partial, st); break;
    case 3: launch_sweep<KIND, 3>(g, S, with_C, mu, len, mom, partial, st); break;
    case 2: launch_sweep<KIND, 2>(g, S, with_C, mu, len, mom, partial, st); break;
    case 1: launch_sweep<KIND, 1>(g, S, with_C, mu, len, mom, partial, st); break;
    default:
      if constexpr (KIND == kPairLapDl) launch_sweep<KIND, 8>(g, S, with_C, mu, len, mom, partial, st);
  }
}

int dl_moments(bie_geom *g, int stokes, int nrhs, const double *mu, double *mom, hipStream_t st) {
  const long long len = stokes ? 2LL * g->M : g->M;
  const MomentArgs a = moment_args(g, len, mu, mom);
  if (stokes) hipLaunchKernelGGL(k_dl_moments<true>, dim3(g->N, nrhs), dim3(kBlock), 0, st, a);
  else hipLaunchKernelGGL(k_dl_moments<false>, dim3(g->N, nrhs), dim3(kBlock), 0, st, a);
  BIE_HIP_CHECK(hipGetLastError());
  return BIE_OK;
}

}  // namespace

int dl_apply(bie_geom *g, int stokes, int with_C, double alpha, int nrhs, const double *mu,
             double *out, hipStream_t st) {
  if (nrhs < 1 || !mu || !out) {
    set_error("double-layer apply: nrhs >= 1 and non-NULL mu, out required");
    return BIE_EINVAL;
  }
  const int comps = stokes ? 2 : 1, C = stokes ? 3 : 1;
  const long long len = (long long)g->M * comps;
  const int maxR = stokes ? 4 : 8;
  // chunks of up to maxR densities; workspace: partial [S][R][len] (the largest chunk's), moments
  // [nrhs][N][C]
  const int kind = stokes ? kPairStkDl : kPairLapDl;
  auto chunk = [&](int left) { return left >= maxR ? maxR : std::min(left, 4); };
  size_t part = 0;
  for (int r0 = 0; r0 < nrhs; r0 += chunk(nrhs - r0)) {
    const int R = chunk(nrhs - r0);
    part = std::max(part, (size_t)pair_splits(g->M, pair_values(kind, R)) * R * (size_t)len);
  }
  BIE_TRY(g->ws_apply.reserve((part + (size_t)nrhs * g->N * C) * sizeof(double)));
  double *partial = g->ws_apply.as<double>();
  double *mom = partial + part;
  ProfScope prof(BIE_K_DOUBLE_LAYER, st, (long long)nrhs * g->M * (long long)g->M);
  for (int r0 = 0; r0 < nrhs;) {
    const int R = chunk(nrhs - r0), S = pair_splits(g->M, pair_values(kind, R));
    const size_t off = (size_t)r0 * len;
    double *mo = mom + (size_t)r0 * g->N * C;
    const unsigned nt = (unsigned)((g->M + kEpi / kEpiLanes - 1) / (kEpi / kEpiLanes));
    if (stokes) {
      sweep_chunk<kPairStkDl>(g, S, R, with_C != 0, mu + off, len, mo, partial, st);
      hipLaunchKernelGGL(k_dl_epilogue<true>, dim3(nt, R), dim3(kEpi), 0, st, g->M, g->N,
                         S, R, g->xy, g->nx, g->ny, g->w, g->kappa, g->pint, g->dl_scale,
                         mu + off, len, partial, mo, with_C, alpha, out + off);
    } else {
      sweep_chunk<kPairLapDl>(g, S, R, with_C != 0, mu + off, len, mo, partial, st);
      hipLaunchKernelGGL(k_dl_epilogue<false>, dim3(nt, R), dim3(kEpi), 0, st, g->M,
                         g->N, S, R, g->xy, g->nx, g->ny, g->w, g->kappa, g->pint, g->dl_scale,
                         mu + off, len, partial, mo, with_C, alpha, out + off);
    }
    BIE_HIP_CHECK(hipGetLastError());
    r0 += R;
  }
  return BIE_OK;
}

int dl_solve(bie_geom *g, int stokes, int nrhs, const double *data, double *res, double *u_inf,
             double *mu_out, const bie_opts &opts, bie_info *info, hipStream_t s) {
  const int extra = stokes ? 2 : 1, C = stokes ? 3 : 1;
  const int nsys = nrhs + extra;
  const long long len = stokes ? 2LL * g->M : g->M;
  bie_opts o = opts;
  o.precision = BIE_FP64;  // the double-layer apply is float64 only
  o.method = BIE_DIRECT;
  // ws_out: f [nsys][len], mu [nsys][len]; ws_read: moments [nsys][N][C], beta [nrhs][2]
  BIE_TRY(g->ws_out.reserve(2 * (size_t)nsys * len * 8));
  double *f = g->ws_out.as<double>();
  double *mu = f + (size_t)nsys * len;
  BIE_TRY(g->ws_read.reserve(((size_t)nsys * g->N * C + 2 * (size_t)nrhs) * 8));
  double *mom = g->ws_read.as<double>();
  double *beta = mom + (size_t)nsys * g->N * C;
  if (stokes)
    hipLaunchKernelGGL(k_res_rhs, dim3(nb((long long)nsys * g->M)), dim3(kBlock), 0, s, g->M,
                       g->N, nrhs, g->body_of, g->px, g->py, data, f);
  else
    hipLaunchKernelGGL(k_cap_rhs, dim3(nb((long long)nsys * g->M)), dim3(kBlock), 0, s, g->M,
                       g->N, nrhs, g->body_of, data, f);
  BIE_HIP_CHECK(hipGetLastError());
  int rc = solve_system(g, stokes ? 3 : 2, o, nsys, f, mu, info, s);
  if (rc != BIE_OK && rc != BIE_ENOCONV) return rc;
  BIE_TRY(dl_moments(g, stokes, nsys, mu, mom, s));
  if (stokes)
    hipLaunchKernelGGL(k_res_combine, dim3(nrhs), dim3(kBlock), 0, s, g->N, nrhs, mom, g->pint,
                       g->xc, g->yc, res, u_inf, beta);
  else
    hipLaunchKernelGGL(k_cap_combine, dim3(nrhs), dim3(kBlock), 0, s, g->N, nrhs, mom, res, u_inf,
                       beta);
  BIE_HIP_CHECK(hipGetLastError());
  if (mu_out) {
    hipLaunchKernelGGL(k_dl_density, dim3(nb((long long)nrhs * len)), dim3(kBlock), 0, s, len,
                       nrhs, extra, beta, mu, mu_out);
    BIE_HIP_CHECK(hipGetLastError());
  }
  return rc;
}

}  // namespace bie

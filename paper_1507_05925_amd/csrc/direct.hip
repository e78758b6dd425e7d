// The direct float64 apply: pair sums over all nodes, the diagonal limits, the identity and the
// completion. Every pair of distinct nodes goes through one sweep (pairs on the same body have
// the same float64 kernel as the others), so nothing is left for a per-body pass but the sums
// over the bodies' densities.
//
// What bounds it: small geometries by latency and launches, large ones by the float64 vector rate
// (10 multiply-add slots and a quarter of a reciprocal per Laplace pair). Sources are staged in
// LDS, where scalar loads of the earlier per-body sweep left each wave waiting for its own
// source records (8 workgroups of 128-source chains took 15 us for 512 nodes); the sources of a
// workgroup are split over its four waves, and a lane takes two targets (large) so that a staged
// value serves two pairs: at one target per lane the LDS return path (128 B per clock and
// compute unit, 24 B per pair and lane) would be the limit.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "internal.h"
#include "pairs.h"

namespace bie {
namespace {

// Split sweep: grid (target tiles, source splits of `per` sources), raw sums of split sp to
// partial[sp][r][target comp].
template <int KIND, int R>
__global__ __launch_bounds__(kBlock, sweep_occupancy(PairShape<KIND, R>::V)) void k_pair_sweep(
    int M, int per, PairSources src, double factor, double *__restrict__ partial) {
  __shared__ double buf[kSweepLds<KIND, R>];
  const int k0 = blockIdx.y * per;
  pair_sweep_tile<KIND, R>(blockIdx.x * kSweepTile, M, k0, min(k0 + per, M), src, factor,
                           partial + (size_t)blockIdx.y * R * src.len, buf);
}

// The rest of a split apply: grid (N bodies x target tiles of kBlock, R). A workgroup forms its
// body's completion sums and adds identity, diagonal limit and the splits (in order).
struct FinishArgs {
  const int *body_ptr;
  const double *nx, *ny, *w, *kappa, *px, *py;
  const double *mu;
  double *out;
  double alpha;
  int M, with_L;
};

// identity, diagonal limit and completion of node i: Laplace c[0] = charge; Stokes c = force, torque
__device__ __forceinline__ double lap_terms(const FinishArgs &a, int i, const double *m, double charge) {
  const double mi = m[i];
  double v = 0.5 * mi - a.w[i] * mi * a.kappa[i] / (4.0 * kPi);
  if (a.with_L) v += charge;
  return v;
}
__device__ __forceinline__ double2 stk_terms(const FinishArgs &a, int i, const double *m, double F1,
                                             double F2, double TQ) {
  const double m1 = m[2 * i], m2 = m[2 * i + 1], wi = a.w[i];
  const double t1 = -a.ny[i], t2 = a.nx[i];  // unit tangent; diagonal -(kappa/2pi) w tau (tau . mu)
  const double d = -a.kappa[i] / (2.0 * kPi) * (t1 * (wi * m1) + t2 * (wi * m2));
  double v1 = 0.5 * m1 + d * t1, v2 = 0.5 * m2 + d * t2;
  if (a.with_L) {
    v1 += F1 + a.px[i] * TQ;
    v2 += F2 + a.py[i] * TQ;
  }
  return make_double2(v1, v2);
}

__device__ __forceinline__ double wave_total(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  return v;
}

template <bool STK>
__global__ __launch_bounds__(kBlock) void k_pair_finish(FinishArgs a, int S, int R, int ntile,
                                                        const double *__restrict__ partial) {
  __shared__ double sh[3][4];
  constexpr int C = STK ? 2 : 1;
  const int b = blockIdx.x / ntile, tile = blockIdx.x % ntile, r = blockIdx.y;
  const int k0 = a.body_ptr[b], k1 = a.body_ptr[b + 1];
  if (k0 + tile * kBlock >= k1) return;  // whole workgroup
  const double *m = a.mu + (size_t)r * C * a.M;
  const int i = k0 + tile * kBlock + threadIdx.x;
  const bool valid = i < k1;
  // the splits' sums are read while the completion is reduced
  double far[2] = {0.0, 0.0};
  if (valid)
    for (int sp = 0; sp < S; ++sp)
#pragma unroll
      for (int c = 0; c < C; ++c) far[c] += partial[((size_t)sp * R + r) * C * a.M + (size_t)C * i + c];
  double s[3] = {0.0, 0.0, 0.0};
  if (a.with_L) {
    for (int k = k0 + threadIdx.x; k < k1; k += kBlock) {
      if (STK) {
        const double s1 = a.w[k] * m[2 * k], s2 = a.w[k] * m[2 * k + 1];
        s[0] += s1;
        s[1] += s2;
        s[2] += a.px[k] * s1 + a.py[k] * s2;
      } else {
        s[0] += a.w[k] * m[k];
      }
    }
#pragma unroll
    for (int c = 0; c < (STK ? 3 : 1); ++c) {
      const double v = wave_total(s[c]);
      if ((threadIdx.x & 63) == 0) sh[c][threadIdx.x >> 6] = v;
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < (STK ? 3 : 1); ++c) s[c] = (sh[c][0] + sh[c][1]) + (sh[c][2] + sh[c][3]);
  }
  if (!valid) return;
  if (STK) {
    const double2 v = stk_terms(a, i, m, s[0], s[1], s[2]);
    double *o = a.out + (size_t)r * 2 * a.M + 2 * i;
    o[0] = a.alpha * (v.x + far[0]);
    o[1] = a.alpha * (v.y + far[1]);
  } else {
    a.out[(size_t)r * a.M + i] = a.alpha * (lap_terms(a, i, m, s[0]) + far[0]);
  }
}

// Small geometries: the whole apply in one launch. A workgroup takes 16 targets of one body
// (tile: the body and its first target) against every source: lane % 16 is the target, and the 32
// lane groups of the workgroup take the quads of a staged block (a source per thread) in turn. The
// body's completion sums ride along with the reduction. Latency-bound: 512 nodes take 4.2 us per
// Laplace apply (three launches of 28 us in all before), 2,304 nodes 8.9 us (28 before) and
// 11.9 us per Stokes apply (36 before); 256 threads per workgroup take 10.0 and 13.0 us, 1,024
// threads 9.7 and 13.5.
constexpr int kSmallThreads = 512;
constexpr int kSmallWaves = kSmallThreads / 64;
constexpr int kSmallGroups = kSmallThreads / kSmallTile;

template <int KIND, int R>
__global__ __launch_bounds__(kSmallThreads) void k_pair_small(const int2 *__restrict__ tiles,
                                                       PairSources src, FinishArgs a, double factor) {
  using P = PairShape<KIND, R>;
  constexpr bool STK = P::STK;
  constexpr int NC = STK ? 3 : 1;  // completion sums per right-hand side
  __shared__ double buf[P::ARR * kSmallThreads];
  __shared__ double red[kSmallWaves][P::V][kSmallTile], redc[kSmallWaves][NC * R];
  const int2 tile = tiles[blockIdx.x];
  const int M = a.M, b0 = a.body_ptr[tile.x], b1 = a.body_ptr[tile.x + 1], i0 = tile.y;
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int i = min(i0 + (lane & 15), b1 - 1);
  const int g = t >> 4;
  const double2 z = src.xy[i];
  const double tx = z.x * src.scale, ty = z.y * src.scale, nx = src.nx[i], ny = src.ny[i];
  double acc[P::V];
#pragma unroll
  for (int v = 0; v < P::V; ++v) acc[v] = 0.0;
  PairRaw<KIND, R> rec;
  rec.load(src, min(t, M - 1));
  double comp[NC * R];
#pragma unroll
  for (int c = 0; c < NC * R; ++c) comp[c] = 0.0;
  if (a.with_L)
    for (int k = b0 + t; k < b1; k += kSmallThreads) {
      const double w = a.w[k];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (STK) {
          const double *m = a.mu + (size_t)r * 2 * M;
          const double s1 = w * m[2 * k], s2 = w * m[2 * k + 1];
          comp[3 * r] += s1;
          comp[3 * r + 1] += s2;
          comp[3 * r + 2] += a.px[k] * s1 + a.py[k] * s2;
        } else {
          comp[r] += w * a.mu[(size_t)r * M + k];
        }
      }
    }
  for (int base = 0; base < M; base += kSmallThreads) {
    rec.store(src, base + t < M, buf, kSmallThreads, t);
    __syncthreads();
    rec.load(src, min(base + kSmallThreads + t, M - 1));
    const int nq = (min(M - base, kSmallThreads) + 3) >> 2;
    if (base < i0 + kSmallTile && base + kSmallThreads > i0) {
      for (int q = g; q < nq; q += kSmallGroups)
        pair_quad<KIND, R, true>(buf, kSmallThreads, 4 * q, i - base, tx, ty, nx, ny, acc);
    } else {
      for (int q = g; q < nq; q += kSmallGroups)
        pair_quad<KIND, R, false>(buf, kSmallThreads, 4 * q, -1, tx, ty, nx, ny, acc);
    }
    __syncthreads();
  }
#pragma unroll
  for (int v = 0; v < P::V; ++v) {
    double x = acc[v];
    x += __shfl_xor(x, 16, 64);
    x += __shfl_xor(x, 32, 64);
    if (lane < 16) red[wv][v][lane] = x;
  }
  if (a.with_L) {
#pragma unroll
    for (int c = 0; c < NC * R; ++c) {
      const double x = wave_total(comp[c]);
      if (lane == 0) redc[wv][c] = x;
    }
  }
  __syncthreads();
  const int r = t >> 4, j = t & 15, io = i0 + j;  // 16 threads per right-hand side
  if (r >= R || io >= b1) return;
  auto sum = [&](int v) {
    double x = 0.0;
#pragma unroll
    for (int w = 0; w < kSmallWaves; ++w) x += red[w][v][j];
    return x;
  };
  auto tot = [&](int c) {
    double x = 0.0;
    if (a.with_L)
#pragma unroll
      for (int w = 0; w < kSmallWaves; ++w) x += redc[w][c];
    return x;
  };
  const double f = factor * src.scale;
  if (STK) {
    const double *m = a.mu + (size_t)r * 2 * M;
    const double2 v = stk_terms(a, io, m, tot(3 * r), tot(3 * r + 1), tot(3 * r + 2));
    double *o = a.out + (size_t)r * 2 * M + 2 * io;
    o[0] = a.alpha * (v.x + f * sum(2 * r));
    o[1] = a.alpha * (v.y + f * sum(2 * r + 1));
  } else {
    double far;
    if constexpr (KIND == kPairLap && R == 1) far = f * (a.nx[io] * sum(0) + a.ny[io] * sum(1));
    else far = f * sum(r);
    a.out[(size_t)r * M + io] =
        a.alpha * (lap_terms(a, io, a.mu + (size_t)r * M, tot(r)) + far);
  }
}

PairSources sources_of(const bie_geom *g, const double *mu, long long len) {
  return PairSources{g->xy, g->nx, g->ny, g->w, mu, len, g->pair_scale, g->pair_away};
}

// The traction kernels' constants, -1/(2 pi) and -1/pi.
constexpr double pair_factor(int kind) { return (kind == kPairStk ? -1.0 : -0.5) / kPi; }

template <int KIND, int R>
void sweep(bie_geom *g, int S, const double *mu, long long len, double *partial, hipStream_t st) {
  const unsigned tiles = (unsigned)((g->M + kSweepTile - 1) / kSweepTile);
  hipLaunchKernelGGL((k_pair_sweep<KIND, R>), dim3(tiles, S), dim3(kBlock), 0, st, g->M,
                     (g->M + S - 1) / S,
                     sources_of(g, mu, len), pair_factor(KIND), partial);
}

template <int KIND, int R>
void small(bie_geom *g, const FinishArgs &a, long long len, hipStream_t st) {
  hipLaunchKernelGGL((k_pair_small<KIND, R>), dim3(g->nsmall), dim3(kSmallThreads), 0, st, g->small_tile,
                     sources_of(g, a.mu, len), a, pair_factor(KIND));
}

}  // namespace

// Source splits of the sweep: workgroups all take about the same time and `resident` of them run
// at once, so the count that fills whole rounds best is taken, the smallest within 3 % (more splits
// cost more partial sums), with at least kBlock sources per split (64 up to 12 splits) and at
// most four rounds on small geometries: a Laplace apply on 25,600 nodes takes 240 us with 10 splits (2,000 workgroups in
// two rounds of 1,024) and 244 with 11 (three rounds); on 12,139 nodes (61 bodies) 63 us with 21, 69
// with 11 and 67 with 43. Below one round more splits shorten the sweep but lengthen the sum over
// them: a Stokes double layer of three densities on 1,000 nodes takes 18 us with 3 splits and 15
// with 7, on 2,560 nodes 16 us with 10 and 19 with 43.
// On large ones four rounds leave the last one up to a quarter empty, and the sums over more splits
// are small beside the sweep. With more than two values per node (Stokes of two columns and up): from
// 28,672 nodes up to 12 rounds, Stokes of four columns on 100,096 nodes 11.2 ms with 5 splits and 14.5
// without, on 60,000 3.83 with 12 and 4.32 without. With one or two: from 49,152 nodes up to 8 rounds, one
// Laplace column on 60,000 nodes 1.29 ms against 1.43 within four; below that they gain nothing (45,056
// nodes 0.77 ms with 14 splits, 0.73 with 8).
int pair_splits(int M, int V) {
  const int tiles = (M + kSweepTile - 1) / kSweepTile, resident = 256 * sweep_occupancy(V);
  const int most = std::max({1, M / kBlock, std::min(12, M / 64)});
  const int rounds_most = M < (V > 2 ? 28672 : 49152) ? 4 : V > 2 ? 12 : 8;
  int best = 1;
  double fill = 0.0;
  for (int S = 1; S <= most && S * tiles <= std::max(rounds_most * resident, tiles); ++S) {
    const int W = S * tiles, rounds = (W + resident - 1) / resident;
    const double f = (double)W / ((double)rounds * resident);
    if (f > fill + 0.03) {
      fill = f;
      best = S;
    }
  }
  const int per = (M + best - 1) / best;  // no split is empty
  return (M + per - 1) / per;
}

int pair_sweep(bie_geom *g, int kind, int R, const double *mu, double *partial, hipStream_t st) {
  const long long len = (long long)g->M * ((kind & 1) ? 2 : 1);
  const int S = pair_splits(g->M, pair_values(kind, R));
#define BIE_SWEEP(K, r) case 16 * K + r: sweep<K, r>(g, S, mu, len, partial, st); break
  switch (16 * kind + R) {
    BIE_SWEEP(kPairLap, 1); BIE_SWEEP(kPairLap, 2); BIE_SWEEP(kPairLap, 3); BIE_SWEEP(kPairLap, 4);
    BIE_SWEEP(kPairLap, 8);
    BIE_SWEEP(kPairStk, 1); BIE_SWEEP(kPairStk, 2); BIE_SWEEP(kPairStk, 3); BIE_SWEEP(kPairStk, 4);
    default:
      set_error("pair sweep: unsupported kind or right-hand side count");
      return BIE_EINVAL;
  }
#undef BIE_SWEEP
  BIE_HIP_CHECK(hipGetLastError());
  return BIE_OK;
}

int direct_apply(bie_geom *g, int kind, int with_L, double alpha, int R, const double *mu,
                 double *out, double *partial, hipStream_t st) {
  const long long len = (long long)g->M * (kind == 0 ? 1 : 2);
  const FinishArgs a{g->body_ptr, g->nx, g->ny, g->w, g->kappa, g->px, g->py, mu, out, alpha,
                     g->M, with_L};
  const int kc = kind == 0 ? BIE_K_FAR_LAPLACE_F64 : BIE_K_FAR_STOKES_F64;
  if (g->nsmall > 0) {
    ProfScope prof(kc, st, (long long)g->M * g->M * R);
#define BIE_SMALL(K, r) case 16 * K + r: small<K, r>(g, a, len, st); break
    switch (16 * kind + R) {
      BIE_SMALL(kPairLap, 1); BIE_SMALL(kPairLap, 2); BIE_SMALL(kPairLap, 3); BIE_SMALL(kPairLap, 4);
      BIE_SMALL(kPairLap, 8);
      BIE_SMALL(kPairStk, 1); BIE_SMALL(kPairStk, 2); BIE_SMALL(kPairStk, 3); BIE_SMALL(kPairStk, 4);
      default:
        set_error("direct apply: unsupported right-hand side count");
        return BIE_EINVAL;
    }
#undef BIE_SMALL
    BIE_HIP_CHECK(hipGetLastError());
    return BIE_OK;
  }
  {
    ProfScope prof(kc, st, (long long)g->M * g->M * R);
    BIE_TRY(pair_sweep(g, kind, R, mu, partial, st));
  }
  ProfScope prof(BIE_K_EPILOGUE, st, 0);
  const int S = pair_splits(g->M, pair_values(kind, R));
  const int ntile = std::max(1, (g->max_nb + kBlock - 1) / kBlock);
  if (kind == 0)
    hipLaunchKernelGGL(k_pair_finish<false>, dim3(g->N * ntile, R), dim3(kBlock), 0, st, a,
                       S, R, ntile, partial);
  else
    hipLaunchKernelGGL(k_pair_finish<true>, dim3(g->N * ntile, R), dim3(kBlock), 0, st, a,
                       S, R, ntile, partial);
  BIE_HIP_CHECK(hipGetLastError());
  return BIE_OK;
}

}  // namespace bie

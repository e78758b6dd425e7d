// Device pieces of the direct pair sums in float64, shared by the operator's direct apply
// (direct.hip) and the double layers of the capacitance and resistance problems (dirichlet.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "internal.h"

namespace bie {

// The pair kernels, r = target - source, s the source's strength (w times the density):
//   kPairLap    (r . n_target) s / |r|^2                      kPairLapDl  (r . n_source) s / |r|^2
//   kPairStk    (r . n_target)(r . s) r / |r|^4               kPairStkDl  (r . n_source)(r . s) r / |r|^4
// kPairLap with one right-hand side accumulates s r / |r|^2 (two values) and takes the normal
// component at the end, one multiply-add less per pair; kPairLapN is kPairLap without that
// exception, for callers whose sums must not depend on how many right-hand sides go together.
enum PairKind { kPairLap = 0, kPairStk = 1, kPairLapDl = 2, kPairStkDl = 3, kPairLapN = 4 };

// Loads through the global address space: a pointer that was itself loaded from memory (an item
// descriptor's) is generic to the compiler, and generic loads also wait for LDS.
template <class T>
__device__ __forceinline__ T gload(const T *p, long long i) {
  return ((const T __attribute__((address_space(1))) *)p)[i];
}
typedef double pair_d2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ double2 gload2(const double2 *p, long long i) {
  const pair_d2 v = ((const pair_d2 __attribute__((address_space(1))) *)p)[i];
  return make_double2(v.x, v.y);
}

template <int KIND, int R>
struct PairShape {
  static constexpr bool STK = KIND == kPairStk || KIND == kPairStkDl;
  static constexpr bool DL = KIND == kPairLapDl || KIND == kPairStkDl;
  static constexpr int COMPS = STK ? 2 : 1;                      // components of a density
  static constexpr int V = STK ? 2 * R : (KIND == kPairLap && R == 1 ? 2 : R);  // sums per target
  static constexpr int ARR = 2 + (DL ? 2 : 0) + COMPS * R;       // staged values per source
};

// The reciprocals of four positive numbers from one reciprocal of their product: v_rcp_f64 issues
// at a quarter of the rate of a multiply-add (17.6 against 5.2 cycles per wave), so four of them
// and their refinements cost more than the nine multiplies that share one. The hardware
// estimate (relative error below 5e-8) takes one third-order step, which leaves rounding errors
// only. The callers scale lengths by the geometry's diameter (bie_geom::pair_scale), so that the
// product stays far inside the range of a float64.
__device__ __forceinline__ void rcp4(const double (&a)[4], double (&o)[4]) {
  const double p = a[0] * a[1], q = a[2] * a[3], d = p * q;
  double y = __builtin_amdgcn_rcp(d);
  const double e = fma(-d, y, 1.0);
  y = fma(y, fma(e, e, e), y);
  const double yp = y * q, yq = y * p;
  o[0] = yp * a[1];
  o[1] = yp * a[0];
  o[2] = yq * a[3];
  o[3] = yq * a[2];
}

// Adds the four staged sources at position k of `buf` (arrays of `stride` doubles: x, y, [n_x w,
// n_y w,] then the strengths) to one target's sums. With MASK, source `self` (its index relative
// to the staged block) is the target itself and adds nothing: |r|^2 = 0 is replaced by 1, and
// r = 0 makes every term zero.
template <int KIND, int R, bool MASK>
__device__ __forceinline__ void pair_quad(const double *buf, int stride, int k, int self, double tx,
                                          double ty, double tnx, double tny,
                                          double (&acc)[PairShape<KIND, R>::V]) {
  using S = PairShape<KIND, R>;
  double dx[4], dy[4], rr[4], inv[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    dx[u] = tx - buf[k + u];
    dy[u] = ty - buf[stride + k + u];
    rr[u] = fma(dx[u], dx[u], dy[u] * dy[u]);
    if (MASK) rr[u] = k + u == self ? 1.0 : rr[u];
  }
  rcp4(rr, inv);
  const double *st = buf + (S::DL ? 4 : 2) * stride + k;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    if constexpr (KIND == kPairLap && R == 1) {
      const double t = st[u] * inv[u];
      acc[0] = fma(dx[u], t, acc[0]);
      acc[1] = fma(dy[u], t, acc[1]);
    } else {
      const double nx = S::DL ? buf[2 * stride + k + u] : tnx;
      const double ny = S::DL ? buf[3 * stride + k + u] : tny;
      const double a = fma(dx[u], nx, dy[u] * ny) * inv[u];
      if constexpr (S::STK) {
        const double b = a * inv[u];
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const double c = fma(dx[u], st[2 * r * stride + u], dy[u] * st[(2 * r + 1) * stride + u]) * b;
          acc[2 * r] = fma(c, dx[u], acc[2 * r]);
          acc[2 * r + 1] = fma(c, dy[u], acc[2 * r + 1]);
        }
      } else {
#pragma unroll
        for (int r = 0; r < R; ++r) acc[r] = fma(a, st[r * stride + u], acc[r]);
      }
    }
  }
}

// The sources a pair sweep stages: coordinates and strengths are scaled as they are read.
struct PairSources {
  const double2 *xy;
  const double *nx, *ny, *w;
  const double *mu;  // [R][len], node-major
  long long len;
  double scale, away;  // bie_geom::pair_scale, pair_away
};

// Source k as it lies in memory (kk: any source of the geometry where k is past the end), and its
// staged values at position t of the block: a source past the end (valid false) gets no strength
// and a place away from source kk. The loads are issued a block ahead and used only here, so that
// a block's loads overlap the previous block's pairs.
template <int KIND, int R>
struct PairRaw {
  using S = PairShape<KIND, R>;
  double2 z;
  double w, nx, ny, mu[S::COMPS * R];
  __device__ __forceinline__ void load(const PairSources &a, int kk) {
    z = gload2(a.xy, kk);
    w = gload(a.w, kk);
    if (S::DL) {
      nx = gload(a.nx, kk);
      ny = gload(a.ny, kk);
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int c = 0; c < S::COMPS; ++c)
        mu[r * S::COMPS + c] = gload(a.mu, (long long)r * a.len + (long long)S::COMPS * kk + c);
  }
  __device__ __forceinline__ void store(const PairSources &a, bool valid, double *buf, int stride,
                                        int t) const {
    const double away = valid ? 0.0 : a.away;
    buf[t] = fma(z.x, a.scale, away);
    buf[stride + t] = fma(z.y, a.scale, away);
    if (S::DL) {
      buf[2 * stride + t] = nx;
      buf[3 * stride + t] = ny;
    }
    constexpr int st = S::DL ? 4 : 2;
#pragma unroll
    for (int v = 0; v < S::COMPS * R; ++v) buf[(st + v) * stride + t] = valid ? w * mu[v] : 0.0;
  }
};

// Pair sweep of one tile of targets over a range of sources.
constexpr int kSweepT = 2;                // targets per lane
constexpr int kSweepTile = 64 * kSweepT;  // targets per workgroup
constexpr int kStage = kBlock;            // sources staged at a time: one per thread

// Waves per SIMD that the sweep's registers leave room for (its launch bound), by the number of
// sums per target.
constexpr int sweep_occupancy(int V) { return V <= 2 ? 4 : V <= 4 ? 3 : 2; }

template <int KIND, int R>
constexpr int kSweepLds = PairShape<KIND, R>::ARR * kStage > 4 * kSweepTile * PairShape<KIND, R>::V
                              ? PairShape<KIND, R>::ARR * kStage
                              : 4 * kSweepTile * PairShape<KIND, R>::V;

// Targets i0 .. min(i0 + kSweepTile, i1) - 1, sources k0 .. k1 - 1 (k1 > k0); raw sums to
// out[r][target comp] (of len entries each). A workgroup of kBlock threads; buf: kSweepLds doubles
// of LDS. Wave w takes the quads w, w + 4, ...
// of each staged block; the four waves' sums are added in wave order through LDS. Blocks that
// hold one of the tile's own nodes (a uniform test) mask the pair of a node with itself.
template <int KIND, int R>
__device__ __forceinline__ void pair_sweep_tile(int i0, int i1, int k0, int k1,
                                                const PairSources &src, double factor,
                                                double *__restrict__ out, double *buf) {
  using P = PairShape<KIND, R>;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double tx[kSweepT], ty[kSweepT], nx[kSweepT], ny[kSweepT], acc[kSweepT][P::V];
#pragma unroll
  for (int u = 0; u < kSweepT; ++u) {
    const int i = min(i0 + lane + 64 * u, i1 - 1);
    const double2 z = gload2(src.xy, i);
    tx[u] = z.x * src.scale;
    ty[u] = z.y * src.scale;
    nx[u] = P::DL ? 0.0 : gload(src.nx, i);
    ny[u] = P::DL ? 0.0 : gload(src.ny, i);
#pragma unroll
    for (int v = 0; v < P::V; ++v) acc[u][v] = 0.0;
  }
  PairRaw<KIND, R> rec;
  const int t = threadIdx.x;
  rec.load(src, min(k0 + t, k1 - 1));
  for (int base = k0; base < k1; base += kStage) {
    rec.store(src, base + t < k1, buf, kStage, t);
    __syncthreads();
    rec.load(src, min(base + kStage + t, k1 - 1));  // the next block, during this block's pairs
    const int nq = (min(k1 - base, kStage) + 3) >> 2;  // quads (the last one padded)
    if (base < i0 + kSweepTile && base + kStage > i0) {
      for (int q = wv; q < nq; q += 4)
#pragma unroll
        for (int u = 0; u < kSweepT; ++u)
          pair_quad<KIND, R, true>(buf, kStage, 4 * q, i0 + lane + 64 * u - base, tx[u], ty[u],
                                   nx[u], ny[u], acc[u]);
    } else {
      for (int q = wv; q < nq; q += 4)
#pragma unroll
        for (int u = 0; u < kSweepT; ++u)
          pair_quad<KIND, R, false>(buf, kStage, 4 * q, -1, tx[u], ty[u], nx[u], ny[u], acc[u]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int u = 0; u < kSweepT; ++u)
#pragma unroll
    for (int v = 0; v < P::V; ++v) buf[(wv * P::V + v) * kSweepTile + lane + 64 * u] = acc[u][v];
  __syncthreads();
  const double f = factor * src.scale;
  constexpr int kOut = KIND == kPairLap ? R : P::V;  // values per target after the normal component
  for (int e = t; e < kSweepTile * kOut; e += kBlock) {
    const int j = e % kSweepTile, v = e / kSweepTile, i = i0 + j;
    if (i >= i1) continue;
    auto sum = [&](int c) {
      const double *b = buf + c * kSweepTile + j;
      constexpr int w = P::V * kSweepTile;
      return (b[0] + b[w]) + (b[2 * w] + b[3 * w]);
    };
    if constexpr (KIND == kPairLap && R == 1) {
      out[i] = f * (src.nx[i] * sum(0) + src.ny[i] * sum(1));
    } else if constexpr (P::STK) {
      out[(v / 2) * src.len + 2 * i + (v & 1)] = f * sum(v);
    } else {
      out[v * src.len + i] = f * sum(v);
    }
  }
}

}  // namespace bie

// One operator apply for many geometries at once (batched solves and the server): the pair sweeps
// and the finishing terms of every item run as one launch per kernel class instead of a few per
// geometry. Work is described by task lists built on the host whenever the set of active items
// changes:
//   sweep task  = (item, first rhs of a group of R, tile of kSweepTile targets, source split)
//   finish task = (item, body, rhs, group)
// The sweep is the single-geometry float64 sweep (pairs.h) over all pairs. With BIE_MIXED some items
// take their pairs of different bodies in float32 instead, and the bodies' own blocks in float64:
// items of a batch with many right-hand sides on the matrix cores (k_multi_mm, 16 right-hand sides at
// a time, from kMmRhs on), and large Stokes items otherwise on the vector units (k_multi_far,
// kFarNodes). The rest stay in float64, where float32 takes no less time. Merged items (the server's:
// how many right-hand sides they have depends on the other requests in flight) never choose by that
// number. Float64 right-hand sides go in groups of up to eight (Laplace) or four (Stokes). Splits and
// summation order of the float64 sweep and of k_multi_far depend on the geometry alone, and every group
// size forms a column's sums in the same order: a system's applies depend neither on the rest of the
// batch nor, in float64 and in merged items, on the other right-hand sides of its item. (With
// BIE_MIXED the number of those chooses an unmerged item's sweep; and the single-geometry kernels that
// form an item's right-hand side and read its answer off round by that number.) Items above the
// FMM threshold are applied by the single-geometry path.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "internal.h"
#include "pairs.h"

namespace bie {

struct ItemDesc {
  int M, N, nrhs, S, per;  // S source splits of per nodes
  long long io;       // offset of the item's rhs block in the flat in/out vectors (doubles)
  long long part;     // offset of its partial sums: rhs group r0 at part + r0 S len, [S][R][len]
  const int *body_ptr;
  const double *nx, *ny, *w, *kappa, *px, *py;
  const double2 *xy;
  double scale, away;  // bie_geom::pair_scale, pair_away
  // float32 sweep (mm: the item has it): lists of 16-target tiles (body, first node) and of source
  // chunks (body, first node, nodes); Smm splits of cper chunks, and one more slot of partial sums
  // for the bodies' own blocks: group r0 at part + r0 (Smm + 1) len
  // (k_multi_far: splits of bodies, and the item's float32 strengths from s32 on)
  int mm, ntile, nchunk, cper, Smm;
  long long s32;
  const int *body_of, *split_body;
  const int2 *tile;
  const int4 *chunk;
  const float2 *xr;
  const double *xc, *yc;
};

// Right-hand sides per group of the float32 matrix-core sweep, and the fewest an item of each kind has
// for it: a half-empty group costs as much as a full one. Laplace 8 / 16 / 24 / 32 / 48 on six
// geometries of 4,400 nodes without preconditioner: float64 5.4 / 9.6 / 13.4 / 17.6 / 25.8 ms, matrix
// cores 8.0 / 9.5 / 13.8 / 15.8 / 23.9; Stokes 8 / 16 / 48: 35 / 67 / 202 and 34 / 46 / 131.
// Laplace items of fewer than kMmNodes nodes per body on average stay in float64: their error would
// be above that of the single-geometry float32 sweep (1.02 times at 16 nodes per body, 1.04 at 8,
// 0.78 at 32).
constexpr int kMmGroup = 16;
constexpr int kMmRhs[2] = {25, 8};
constexpr int kMmNodes = 32;
constexpr int kMmChunk = 64;                       // sources staged at a time (one body's)
constexpr int kMmTiles = 2;                        // 16-target tiles per wave
constexpr int kMmTile = 16 * kMmTiles * 4;         // targets per workgroup, at most

// Stokes items of at least kFarNodes nodes take the float32 vector sweep instead of the float64 one
// where they do not take the matrix cores', whatever their right-hand sides (merged items may not
// choose by their number). Served mobility requests, 1 / 4 / 15 at a time, float64 against float32:
// 9,536 nodes 3.1 / 6.4 / 16.1 ms against 3.5 / 7.0 / 13.6; 12,896 nodes 4.1 / 9.0 / 25.9 against
// 4.8 / 9.7 / 21.1; 30,688 nodes 17.5 / 41.9 / 137 against 14.0 / 30.8 / 90.7.
constexpr int kFarNodes = 12288;
constexpr int kFarGroup = 4;
// They take the matrix cores' sweep from kMmRhsLarge right-hand sides on (8 / 10 / 12 / 16 on 19,872
// nodes without preconditioner: vector 79 / 103 / 115 / 151 ms, matrix cores 102 / 111 / 116 / 131;
// on 30,688 174 / 231 / 259 / 341 and 234 / 257 / 267 / 305).
constexpr int kMmRhsLarge = 12;

// Right-hand side group sizes of each kind.
constexpr int kGroups[2][5] = {{8, 4, 3, 2, 1}, {4, 3, 2, 1, 0}};

constexpr int kFmmStreams = 4;

struct MultiPlan {
  DevBuf desc_buf, task_buf, ws;
  // items applied by the FMM run on a small pool of streams (one per geometry, by first
  // appearance), forked from and joined back to the caller's stream
  hipStream_t pool[kFmmStreams] = {};
  hipEvent_t fork = nullptr, join[kFmmStreams] = {};
  int nsweep = 0, nfin = 0, nlap = 0;  // tasks; finish tasks of Laplace items (they come first)
  int nmm[2] = {0, 0};                 // float32 matrix-core sweep tasks per kind
  int nfar = 0, npack = 0;             // float32 vector sweep tasks, and those of its strengths
  int4 *sweep_task = nullptr, *fin_task = nullptr, *mm_task[2] = {nullptr, nullptr};
  int4 *far_task = nullptr, *pack_task = nullptr;
  DevBuf list_buf;  // the items' tile and chunk lists
  ItemDesc *desc = nullptr;
  long long npart = 0, nfloat = 0;  // doubles of partial sums, floats of strengths
  // the plan is reused while every item matches: geometry id, kind, rhs count, method and
  // offset of its block, and the active flags
  std::vector<unsigned long long> key_gen;
  std::vector<int> key_kind, key_nrhs;
  std::vector<char> key_fmm;
  std::vector<long long> key_io;
  std::vector<char> key_active;
  bool valid = false;
};

void multi_destroy(MultiPlan *p) {
  if (!p) return;
  for (int i = 0; i < kFmmStreams; ++i) {
    if (p->pool[i]) {
      (void)hipStreamSynchronize(p->pool[i]);
      (void)hipStreamDestroy(p->pool[i]);
    }
    if (p->join[i]) (void)hipEventDestroy(p->join[i]);
  }
  if (p->fork) (void)hipEventDestroy(p->fork);
  p->desc_buf.release();
  p->list_buf.release();
  p->task_buf.release();
  p->ws.release();
  delete p;
}

namespace {

// The items that take the float32 sweep in an apply, where they have it: none, all, or (sets of at
// most kMaxPrecGroups items only) those whose bit is set.
enum MaskMode { kNone = 0, kAll = 1, kBits = 2 };
struct ItemMask {
  int mode;
  unsigned long long w[kMaxPrecGroups / 64];
};
__device__ __forceinline__ bool in_mask(const ItemMask &m, int it) {
  return m.mode == kBits ? (m.w[it >> 6] >> (it & 63)) & 1ull : m.mode == kAll;
}

// Float64 sweep task: all sources of split sp, or (own) body sp's block of its own targets, which
// goes with the float32 sweep of the others. z: first target.
template <int KIND, int R>
__device__ __forceinline__ void sweep_task(const int4 &t, const ItemDesc &d, bool own,
                                           const double *__restrict__ mu,
                                           double *__restrict__ partial, double *buf) {
  const long long len = (long long)d.M * PairShape<KIND, R>::COMPS;
  const PairSources src{d.xy, d.nx, d.ny, d.w, mu + d.io + t.y * len, len, d.scale, d.away};
  const int sp = t.w & 0xfffff;
  int i1, k0, k1;
  long long at;
  if (own) {  // slot Smm of the rhs group of 16 that t.y lies in
    const int r0 = t.y / kMmGroup * kMmGroup, G = min(kMmGroup, d.nrhs - r0);
    k0 = gload(d.body_ptr, sp);
    i1 = k1 = gload(d.body_ptr, sp + 1);
    at = (long long)r0 * (d.Smm + 1) * len + ((long long)d.Smm * G + (t.y - r0)) * len;
  } else {
    k0 = sp * d.per;
    k1 = min(k0 + d.per, d.M);
    i1 = d.M;
    at = ((long long)t.y * d.S + (long long)sp * R) * len;
  }
  pair_sweep_tile<KIND, R>(t.z, i1, k0, k1, src, (KIND == kPairStk ? -1.0 : -0.5) / kPi,
                           partial + d.part + at, buf);
}

// One launch for every kind and group size: task (item, first rhs, first target, split or body |
// (16 kind + R) << 20 | own << 26).
// Separate launches let the smaller groups keep more waves in flight but ran one after another:
// the remainders of six geometries' P and M took seven launches of about 8 us beside 100 us of
// full groups.
__global__ __launch_bounds__(kBlock, 2) void k_multi_sweep(const int4 *__restrict__ tasks,
                                                           const ItemDesc *__restrict__ D,
                                                           const double *__restrict__ mu,
                                                           const ItemMask mm,
                                                           double *__restrict__ partial) {
  __shared__ double buf[kSweepLds<kPairStk, 4> > kSweepLds<kPairLapN, 8> ? kSweepLds<kPairStk, 4>
                                                                         : kSweepLds<kPairLapN, 8>];
  const int4 t = tasks[blockIdx.x];
  const ItemDesc &d = D[t.x];
  const bool own = t.w >> 26;
  if (own != (d.mm && in_mask(mm, t.x))) return;  // (whole workgroup)
  switch ((t.w >> 20) & 0x3f) {
    case 8: sweep_task<kPairLapN, 8>(t, d, own, mu, partial, buf); break;
    case 4: sweep_task<kPairLapN, 4>(t, d, own, mu, partial, buf); break;
    case 3: sweep_task<kPairLapN, 3>(t, d, own, mu, partial, buf); break;
    case 2: sweep_task<kPairLapN, 2>(t, d, own, mu, partial, buf); break;
    case 1: sweep_task<kPairLapN, 1>(t, d, own, mu, partial, buf); break;
    case 16 + 4: sweep_task<kPairStk, 4>(t, d, own, mu, partial, buf); break;
    case 16 + 3: sweep_task<kPairStk, 3>(t, d, own, mu, partial, buf); break;
    case 16 + 2: sweep_task<kPairStk, 2>(t, d, own, mu, partial, buf); break;
    default: sweep_task<kPairStk, 1>(t, d, own, mu, partial, buf); break;
  }
}

// Float32 pairs of different bodies on the matrix cores: for 16 targets and four sources a lane forms
// one kernel value (target lane % 16, source lane / 16), the A operand of a 16 x 16 x 4 product
// whose B operand holds the sources' strengths of 16 right-hand sides. A Laplace value is one
// operand, a Stokes pair's symmetric 2 x 2 block three, used in four products. A workgroup takes up
// to eight 16-target tiles (two per wave, each of one body) against one split's source chunks
// (at most 64 nodes of one body): coordinates relative to the source body's centroid in float32.
// Laplace normals are pairs of floats, the Stokes block's reciprocal takes a Newton step, and two
// products (eight sources) are summed at a time, those sums over a chunk, the chunks in float64. So the
// error is at most that of the single-geometry float32 sweep, whose sums run over a body (one sum
// per chunk and rounded normals: up to 1.36 times it at 32 nodes per body; now 0.78 Laplace and
// 0.93 Stokes at 32, 0.5 at 96). Bound by the vector work per value and the products, which do not
// overlap: per 64 pairs and 16 right-hand sides about 100 (Laplace) and 230 (Stokes) cycles, where the
// vector sweep took 34 (Stokes) cycles per right-hand side. P and M of 32 geometries of 8 to 128
// bodies with the block preconditioner: 4.0 s, by the vector sweep 5.4 (in float64 throughout: 5.6).
typedef float mm_f4 __attribute__((ext_vector_type(4)));

template <bool STK>
__global__ __launch_bounds__(kBlock) void k_multi_mm(const int4 *__restrict__ tasks,
                                                     const ItemDesc *__restrict__ D,
                                                     const double *__restrict__ mu,
                                                     const ItemMask mm,
                                                     double *__restrict__ partial) {
  constexpr int C = STK ? 2 : 1;
  constexpr int STEPS = 2;               // products per accumulator before they join the chunk's sum
  constexpr int ROW = kMmGroup * C + 2;  // floats per staged source (padded: writes spread over banks)
  __shared__ float2 xs[kMmChunk];
  __shared__ float ss[kMmChunk * ROW];
  const int4 t = tasks[blockIdx.x];  // item, first rhs, first tile, split
  if (!in_mask(mm, t.x)) return;     // (whole workgroup)
  const ItemDesc &d = D[t.x];
  const int r0 = t.y, G = min(kMmGroup, d.nrhs - r0);
  const long long len = (long long)d.M * C;
  const int lane = threadIdx.x & 63, j = lane & 15, q = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // this wave's tiles: body (wave-uniform; -1: none) and this lane's target
  int body[kMmTiles], first[kMmTiles];
  double cx[kMmTiles], cy[kMmTiles];
  float2 pr[kMmTiles];
  float nx[kMmTiles], ny[kMmTiles], tx[kMmTiles], ty[kMmTiles];
  float nxl[kMmTiles], nyl[kMmTiles];  // Laplace: the normals' low parts
  double acc[kMmTiles][C][4];
#pragma unroll
  for (int u = 0; u < kMmTiles; ++u) {
    const int ti = t.z + wv * kMmTiles + u;
    body[u] = -1;
    first[u] = 0;
    if (ti < d.ntile) {
      body[u] = __builtin_amdgcn_readfirstlane(gload(reinterpret_cast<const int *>(d.tile), 2 * ti));
      first[u] = __builtin_amdgcn_readfirstlane(gload(reinterpret_cast<const int *>(d.tile), 2 * ti + 1));
      const int i = min(first[u] + j, gload(d.body_ptr, body[u] + 1) - 1);
      cx[u] = gload(d.xc, body[u]);
      cy[u] = gload(d.yc, body[u]);
      const float *p = reinterpret_cast<const float *>(d.xr);
      pr[u] = make_float2(gload(p, 2LL * i), gload(p, 2LL * i + 1));
      const double n1 = gload(d.nx, i), n2 = gload(d.ny, i);
      nx[u] = (float)n1;
      ny[u] = (float)n2;
      nxl[u] = (float)(n1 - (double)nx[u]);
      nyl[u] = (float)(n2 - (double)ny[u]);
    }
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[u][c][e] = 0.0;
  }
  const int c0 = t.w * d.cper, c1 = min(c0 + d.cper, d.nchunk);
  // staging: thread (row r, kk) takes nodes kk, kk + 16, ... of the chunk for right-hand side r
  const int sr = threadIdx.x >> 4, kk = threadIdx.x & 15;
  const double *m = mu + d.io + (long long)(r0 + min(sr, G - 1)) * len;
  double mv[4][C], wt[4];
  float2 xv;
  int4 ch = d.chunk[c0];
  auto fetch = [&](const int4 &h) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int k = h.y + min(kk + 16 * e, h.z - 1);
      wt[e] = gload(d.w, k);
#pragma unroll
      for (int c = 0; c < C; ++c) mv[e][c] = m[(long long)C * k + c];
    }
    if (threadIdx.x < kMmChunk) {
      const float *p = reinterpret_cast<const float *>(d.xr);
      const long long k = h.y + min((int)threadIdx.x, h.z - 1);
      xv = make_float2(gload(p, 2 * k), gload(p, 2 * k + 1));
    }
  };
  fetch(ch);
  int frame = -1;  // the body whose centroid tx, ty are relative to
  for (int c = c0; c < c1; ++c) {
    const int cb = __builtin_amdgcn_readfirstlane(ch.x), n = __builtin_amdgcn_readfirstlane(ch.z);
    // nodes past the chunk's end: no strength, far away
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int a = 0; a < C; ++a)
        ss[(kk + 16 * e) * ROW + C * sr + a] = kk + 16 * e < n && sr < G ? (float)(wt[e] * mv[e][a]) : 0.0f;
    if (threadIdx.x < kMmChunk)
      xs[threadIdx.x] = (int)threadIdx.x < n ? xv : make_float2(1.0e18f, 1.0e18f);
    __syncthreads();
    if (c + 1 < c1) {
      ch = d.chunk[c + 1];
      fetch(ch);
    }
    if (frame != cb) {
      frame = cb;
      const double sx = gload(d.xc, cb), sy = gload(d.yc, cb);
#pragma unroll
      for (int u = 0; u < kMmTiles; ++u) {
        tx[u] = (float)((cx[u] - sx) + (double)pr[u].x);
        ty[u] = (float)((cy[u] - sy) + (double)pr[u].y);
      }
    }
    mm_f4 y[kMmTiles][C];
#pragma unroll
    for (int u = 0; u < kMmTiles; ++u)
#pragma unroll
      for (int a = 0; a < C; ++a) y[u][a] = mm_f4{0.0f, 0.0f, 0.0f, 0.0f};
    for (int kb = 0; kb < n; kb += 4 * STEPS) {
      mm_f4 z[kMmTiles][C];
#pragma unroll
      for (int u = 0; u < kMmTiles; ++u)
#pragma unroll
        for (int a = 0; a < C; ++a) z[u][a] = mm_f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int w = 0; w < STEPS; ++w) {
        if (kb + 4 * w >= n) break;
        const int k = kb + 4 * w + q;
        const float2 p = xs[k];
        float b[C];
#pragma unroll
        for (int a = 0; a < C; ++a) b[a] = ss[k * ROW + C * j + a];
#pragma unroll
        for (int u = 0; u < kMmTiles; ++u) {
          if (body[u] == cb || body[u] < 0) continue;  // (wave-uniform)
          const float dx = tx[u] - p.x, dy = ty[u] - p.y;
          const float rr = fmaf(dx, dx, dy * dy);
          float inv = __builtin_amdgcn_rcpf(rr);
          if constexpr (STK) {
            inv = fmaf(inv, fmaf(-rr, inv, 1.0f), inv);
            const float a = fmaf(dx, nx[u], dy * ny[u]) * inv;
            const float g = a * inv, gx = g * dx, gy = g * dy;
            const float xx = gx * dx, xy = gx * dy, yy = gy * dy;
            z[u][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(xx, b[0], z[u][0], 0, 0, 0);
            z[u][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(xy, b[0], z[u][1], 0, 0, 0);
            z[u][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(xy, b[C - 1], z[u][0], 0, 0, 0);
            z[u][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(yy, b[C - 1], z[u][1], 0, 0, 0);
          } else {
            const float low = fmaf(dx, nxl[u], dy * nyl[u]);
            const float a = fmaf(dx, nx[u], fmaf(dy, ny[u], low)) * inv;
            z[u][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b[0], z[u][0], 0, 0, 0);
          }
        }
      }
#pragma unroll
      for (int u = 0; u < kMmTiles; ++u)
#pragma unroll
        for (int a = 0; a < C; ++a) y[u][a] += z[u][a];
    }
#pragma unroll
    for (int u = 0; u < kMmTiles; ++u)
#pragma unroll
      for (int a = 0; a < C; ++a)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[u][a][e] += (double)y[u][a][e];
    __syncthreads();  // the chunk is no longer read
  }
  // accumulator layout: lane (j, q) holds targets 4 q + e of right-hand side j
  if (j >= G) return;
  double *o = partial + d.part + (long long)r0 * (d.Smm + 1) * len + ((long long)t.w * G + j) * len;
  const double f = (STK ? -1.0 : -0.5) / kPi;
#pragma unroll
  for (int u = 0; u < kMmTiles; ++u) {
    if (body[u] < 0) continue;
    const int b1 = gload(d.body_ptr, body[u] + 1);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int i = first[u] + 4 * q + e;
      if (i >= b1) continue;
#pragma unroll
      for (int a = 0; a < C; ++a) o[(long long)C * i + a] = f * acc[u][a][e];
    }
  }
}

// Float32 Stokes pairs of different bodies on the vector units, for large items (kFarNodes). Lane =
// target; sources and strengths are wave-uniform and come through scalar registers, coordinates
// relative to the source body's centroid, a body's float32 sums added into float64. The operations
// of a right-hand side do not depend on R, so a request has the same bits whichever others it is
// merged with. Bound by the vector rate: a pair takes about 45 cycles per 64 and 22 more per
// right-hand side, where the float64 sweep takes 70 and 24 and waits for LDS. Sources staged in LDS
// (16 targets and four source lanes per tile, as in k_multi_mm) took 39 and 123 ms for the 1 and 15
// requests on 30,000 nodes that take 14 and 94 here.
constexpr float kFar32 = 1.0e18f;

template <int R>
__device__ __forceinline__ void far_task(const int4 &t, const ItemDesc &d,
                                         const float *__restrict__ s32,
                                         double *__restrict__ partial) {
  const int M = d.M, i = t.z + (int)threadIdx.x, ii = min(i, M - 1);
  const long long len = 2LL * M;
  const int bi = gload(d.body_of, ii);
  const float *sv = s32 + d.s32 + (long long)t.y * len;
  double Gx[R], Gy[R];
#pragma unroll
  for (int r = 0; r < R; ++r) Gx[r] = Gy[r] = 0.0;
  const int c0 = gload(d.split_body, t.w), c1 = gload(d.split_body, t.w + 1);
  const double cxi = gload(d.xc, bi), cyi = gload(d.yc, bi);
  const float *xr = reinterpret_cast<const float *>(d.xr);
  const float px = gload(xr, 2LL * ii), py = gload(xr, 2LL * ii + 1);
  const float nx = (float)gload(d.nx, ii), ny = (float)gload(d.ny, ii);
  for (int c = c0; c < c1; ++c) {
    const bool self = c == bi;
    if (__all(self)) continue;
    const int k0 = gload(d.body_ptr, c), k1 = gload(d.body_ptr, c + 1);
    float tx = (float)((cxi - gload(d.xc, c)) + (double)px);
    float ty = (float)((cyi - gload(d.yc, c)) + (double)py);
    tx = self ? kFar32 : tx;  // no pair of these lanes is near; their sums are dropped
    ty = self ? kFar32 : ty;
    float gx[R], gy[R];
#pragma unroll
    for (int r = 0; r < R; ++r) gx[r] = gy[r] = 0.0f;
#pragma unroll 2
    for (int k = k0; k < k1; ++k) {
      const float dx = tx - gload(xr, 2LL * k), dy = ty - gload(xr, 2LL * k + 1);
      const float inv = __builtin_amdgcn_rcpf(fmaf(dx, dx, dy * dy));
      const float a = fmaf(dx, nx, dy * ny) * (inv * inv);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const float e = fmaf(dx, gload(sv, r * len + 2LL * k), dy * gload(sv, r * len + 2LL * k + 1)) * a;
        gx[r] = fmaf(e, dx, gx[r]);
        gy[r] = fmaf(e, dy, gy[r]);
      }
    }
    if (!self) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        Gx[r] += (double)gx[r];
        Gy[r] += (double)gy[r];
      }
    }
  }
  if (i >= M) return;
  // partial sums lie in the groups of 16 that the finishing launch reads
  const int r0 = t.y / kMmGroup * kMmGroup, G = min(kMmGroup, d.nrhs - r0);
  double *o = partial + d.part + (long long)r0 * (d.Smm + 1) * len +
              ((long long)t.w * G + (t.y - r0)) * len + 2LL * i;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    o[r * len] = -Gx[r] / kPi;
    o[r * len + 1] = -Gy[r] / kPi;
  }
}

// Tasks (item, first rhs | R << 24, first target, split of bodies).
__global__ __launch_bounds__(kBlock) void k_multi_far(const int4 *__restrict__ tasks,
                                                      const ItemDesc *__restrict__ D,
                                                      const float *__restrict__ s32,
                                                      const ItemMask mm,
                                                      double *__restrict__ partial) {
  int4 t = tasks[blockIdx.x];
  if (!in_mask(mm, t.x)) return;  // (whole workgroup)
  const ItemDesc &d = D[t.x];
  const int R = t.y >> 24;
  t.y &= 0xffffff;
  switch (R) {
    case 4: far_task<4>(t, d, s32, partial); break;
    case 3: far_task<3>(t, d, s32, partial); break;
    case 2: far_task<2>(t, d, s32, partial); break;
    default: far_task<1>(t, d, s32, partial); break;
  }
}

// The float32 strengths w mu that k_multi_far reads: tasks (item, rhs, first node).
constexpr int kPackNodes = 2048;
__global__ __launch_bounds__(kBlock) void k_multi_pack(const int4 *__restrict__ tasks,
                                                       const ItemDesc *__restrict__ D,
                                                       const double *__restrict__ mu,
                                                       const ItemMask mm, float *__restrict__ s32) {
  const int4 t = tasks[blockIdx.x];
  if (!in_mask(mm, t.x)) return;
  const ItemDesc &d = D[t.x];
  const long long at = (long long)t.y * 2 * d.M;
  const double *m = mu + d.io + at;
  float *o = s32 + d.s32 + at;
  const int k1 = min(t.z + kPackNodes, d.M);
  for (int k = t.z + threadIdx.x; k < k1; k += kBlock) {
    const double w = gload(d.w, k);
    o[2LL * k] = (float)(w * m[2LL * k]);
    o[2LL * k + 1] = (float)(w * m[2LL * k + 1]);
  }
}

// Identity, diagonal limit, completion and the splits' sums (in order) of one body and right-hand
// side by one wave: task (item, body, rhs r, first rhs of its group | group size << 24).
template <bool STK>
__device__ __forceinline__ void finish_task(const int4 &t, const ItemDesc &d,
                                            bool mm, const double *__restrict__ mu,
                                            const double *__restrict__ partial,
                                            double *__restrict__ out) {
  const int lane = threadIdx.x & 63;
  constexpr int C = STK ? 2 : 1;
  const long long len = (long long)d.M * C;
  const int r0 = mm ? t.z / kMmGroup * kMmGroup : t.w & 0xffffff;
  const int R = mm ? min(kMmGroup, d.nrhs - r0) : t.w >> 24, S = mm ? d.Smm + 1 : d.S;
  const int k0 = gload(d.body_ptr, t.y), k1 = gload(d.body_ptr, t.y + 1);
  const double *m = mu + d.io + t.z * len;
  const double *part = partial + d.part + r0 * S * len + (t.z - r0) * len;
  double *o = out + d.io + t.z * len;
  double s[3] = {0.0, 0.0, 0.0};
  for (int k = k0 + lane; k < k1; k += 64) {
    const double w = gload(d.w, k);
    if (STK) {
      const double s1 = w * m[2 * k], s2 = w * m[2 * k + 1];
      s[0] += s1;
      s[1] += s2;
      s[2] += gload(d.px, k) * s1 + gload(d.py, k) * s2;
    } else {
      s[0] += w * m[k];
    }
  }
#pragma unroll
  for (int c = 0; c < (STK ? 3 : 1); ++c)
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s[c] += __shfl_xor(s[c], off, 64);
  for (int i = k0 + lane; i < k1; i += 64) {
    double far[C];
#pragma unroll
    for (int c = 0; c < C; ++c) far[c] = 0.0;
#pragma unroll 4
    for (int sp = 0; sp < S; ++sp)
#pragma unroll
      for (int c = 0; c < C; ++c) far[c] += part[(long long)sp * R * len + (long long)C * i + c];
    const double wi = gload(d.w, i), kap = gload(d.kappa, i);
    if constexpr (STK) {
      const double m1 = m[2 * i], m2 = m[2 * i + 1];
      const double t1 = -gload(d.ny, i), t2 = gload(d.nx, i);  // unit tangent
      const double dg = -kap / (2.0 * kPi) * (t1 * (wi * m1) + t2 * (wi * m2));
      o[2 * i] = 0.5 * m1 + dg * t1 + s[0] + gload(d.px, i) * s[2] + far[0];
      o[2 * i + 1] = 0.5 * m2 + dg * t2 + s[1] + gload(d.py, i) * s[2] + far[1];
    } else {
      const double mi = m[i];
      o[i] = 0.5 * mi - wi * mi * kap / (4.0 * kPi) + s[0] + far[0];
    }
  }
}

__global__ __launch_bounds__(kBlock) void k_multi_finish(int ntask, int nlap,
                                                         const int4 *__restrict__ tasks,
                                                         const ItemDesc *__restrict__ D,
                                                         const double *__restrict__ mu,
                                                         const ItemMask mm,
                                                         const double *__restrict__ partial,
                                                         double *__restrict__ out) {
  const int ti = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (ti >= ntask) return;
  const int4 t = tasks[ti];
  const ItemDesc &d = D[t.x];
  const bool f32 = d.mm && in_mask(mm, t.x);
  if (ti < nlap) finish_task<false>(t, d, f32, mu, partial, out);
  else finish_task<true>(t, d, f32, mu, partial, out);
}

// Source splits of an item whose targets make `tiles` workgroups, from the geometry alone: up to about
// 256 workgroups per rhs group (a batch has several groups and items to fill the compute units), and
// from 8,192 nodes on, where one item may be the whole batch, up to 1,024 with at least 2,048 sources
// each. Of these counts the one whose fullest compute unit is done first (within 3% the smallest),
// a lone workgroup running at 0.85 of the rate of several on a compute unit. One elastance request
// on 17,248 nodes 5.3 -> 3.1 ms per solve with 7 splits instead of one, 16 mobility ones 47 -> 30; on
// 8,416 nodes 1.4 with 3 splits (198 workgroups) and 1.6 with 4 (264).
int item_splits(int M, int tiles) {
  const int most = std::max(256 / tiles, std::min(1024 / tiles, M / 2048));
  int best = 1;
  double least = 1e300;
  for (int S = 1; S <= most; ++S) {
    const int n = (S * tiles + 255) / 256;
    const double time = n / (double)S / (n > 1 ? 1.0 : 0.85);
    if (time < 0.97 * least) {
      least = time;
      best = S;
    }
  }
  return best;
}

// The next right-hand side group of kind's items when `left` remain.
int next_group(int kind, int left) {
  int c = 0;
  while (kGroups[kind][c] > left) ++c;
  return kGroups[kind][c];
}

int build_plan(MultiPlan &P, const std::vector<MultiItem> &items, const std::vector<char> &active,
               hipStream_t s) {
  const int n = (int)items.size();
  std::vector<ItemDesc> desc(n);
  std::vector<int4> sweep[2], own[2], fin[2], mm[2], fr, pk, chunks;
  std::vector<int2> tiles16;
  std::vector<size_t> tile_at(n, 0), chunk_at(n, 0);
  long long part = 0, floats = 0;
  for (int i = 0; i < n; ++i) {
    const MultiItem &m = items[i];
    bie_geom *g = m.g;
    ItemDesc &d = desc[i];
    const int want = std::max(1, std::min(item_splits(g->M, (g->M + kSweepTile - 1) / kSweepTile),
                                          g->M / kBlock));
    d = ItemDesc{};
    d.M = g->M;
    d.N = g->N;
    d.nrhs = m.nrhs;
    d.per = (g->M + want - 1) / want;
    d.S = (g->M + d.per - 1) / d.per;  // no split is empty
    d.io = m.io;
    d.body_ptr = g->body_ptr;
    d.nx = g->nx; d.ny = g->ny; d.w = g->w; d.kappa = g->kappa;
    d.px = g->px; d.py = g->py; d.xy = g->xy;
    d.xr = g->xr; d.xc = g->xc; d.yc = g->yc;
    d.scale = g->pair_scale;
    d.away = g->pair_away;
    d.part = part;
    if (!active[i] || m.fmm) continue;
    const long long len = g->M * (m.kind == 0 ? 1LL : 2LL);
    const bool large = m.kind == 1 && g->M >= kFarNodes;
    const bool cores = !m.merged && m.nrhs >= (large ? kMmRhsLarge : kMmRhs[m.kind]) &&
                       (m.kind == 1 || g->M >= (long long)kMmNodes * g->N);
    const bool far = !cores && large;
    d.mm = cores || far;
    if (far) {
      d.body_of = g->body_of;
      d.split_body = g->split_body;
      d.Smm = g->nsplit;
      d.s32 = floats;
      floats += m.nrhs * len;
      for (int r0 = 0; r0 < m.nrhs; r0 += kFarGroup)
        for (int sp = 0; sp < d.Smm; ++sp)
          for (int k = 0; k < g->M; k += kBlock)
            fr.push_back(make_int4(i, r0 | std::min(kFarGroup, m.nrhs - r0) << 24, k, sp));
      for (int r = 0; r < m.nrhs; ++r)
        for (int k = 0; k < g->M; k += kPackNodes) pk.push_back(make_int4(i, r, k, 0));
    } else if (cores) {
      tile_at[i] = tiles16.size();
      chunk_at[i] = chunks.size();
      for (int b = 0; b < g->N; ++b) {
        const int b0 = g->h_body_ptr[b], b1 = g->h_body_ptr[b + 1];
        for (int k = b0; k < b1; k += 16) tiles16.push_back(make_int2(b, k));
        for (int k = b0; k < b1; k += kMmChunk)
          chunks.push_back(make_int4(b, k, std::min(kMmChunk, b1 - k), 0));
      }
      d.ntile = (int)(tiles16.size() - tile_at[i]);
      d.nchunk = (int)(chunks.size() - chunk_at[i]);
      const int wgs = (d.ntile + kMmTile / 16 - 1) / (kMmTile / 16);
      const int groups = (m.nrhs + kMmGroup - 1) / kMmGroup;  // (several fill the chip by themselves)
      const int smm = std::max(1, std::min(wgs * groups < 768 ? item_splits(g->M, wgs) : 256 / wgs,
                                           d.nchunk / 4));
      d.cper = (d.nchunk + smm - 1) / smm;
      d.Smm = (d.nchunk + d.cper - 1) / d.cper;
      for (int r0 = 0; r0 < m.nrhs; r0 += kMmGroup)
        for (int sp = 0; sp < d.Smm; ++sp)
          for (int t = 0; t < d.ntile; t += kMmTile / 16) mm[m.kind].push_back(make_int4(i, r0, t, sp));
    }
    if (d.mm) {
      // the bodies' own blocks in float64, in groups that stay within the groups of 16
      for (int r0 = 0; r0 < m.nrhs;) {
        const int left = std::min(m.nrhs, r0 / kMmGroup * kMmGroup + kMmGroup) - r0;
        const int R = next_group(m.kind, left);
        for (int b = 0; b < g->N; ++b)
          for (int k = g->h_body_ptr[b]; k < g->h_body_ptr[b + 1]; k += kSweepTile)
            own[m.kind].push_back(make_int4(i, r0, k, b | (16 * m.kind + R) << 20 | 1 << 26));
        r0 += R;
      }
    }
    part += m.nrhs * len * std::max(d.S, d.mm ? d.Smm + 1 : 0);
    for (int r0 = 0; r0 < m.nrhs;) {
      const int R = next_group(m.kind, m.nrhs - r0);
      for (int sp = 0; sp < d.S; ++sp)
        for (int k = 0; k < g->M; k += kSweepTile)
          sweep[m.kind].push_back(make_int4(i, r0, k, sp | (16 * m.kind + R) << 20));
      for (int b = 0; b < g->N; ++b)
        for (int r = r0; r < r0 + R; ++r) fin[m.kind].push_back(make_int4(i, b, r, r0 | R << 24));
      r0 += R;
    }
  }
  // the longest tasks (Stokes) first, so that the short ones fill the last round
  std::vector<int4> all(sweep[1]);
  auto append = [&](const std::vector<int4> &v) {
    all.insert(all.end(), v.begin(), v.end());
    return (int)v.size();
  };
  append(sweep[0]);
  append(own[1]);
  append(own[0]);
  P.nsweep = (int)all.size();
  P.nlap = append(fin[0]);
  P.nfin = P.nlap + append(fin[1]);
  for (int k = 0; k < 2; ++k) P.nmm[k] = append(mm[k]);
  P.nfar = append(fr);
  P.npack = append(pk);
  BIE_TRY(P.task_buf.reserve(all.size() * sizeof(int4) + 256));
  BIE_TRY(P.desc_buf.reserve(n * sizeof(ItemDesc) + 256));
  BIE_TRY(P.list_buf.reserve(chunks.size() * sizeof(int4) + tiles16.size() * sizeof(int2) + 256));
  P.sweep_task = P.task_buf.as<int4>();
  P.fin_task = P.sweep_task + P.nsweep;
  P.mm_task[0] = P.fin_task + P.nfin;
  P.mm_task[1] = P.mm_task[0] + P.nmm[0];
  P.far_task = P.mm_task[1] + P.nmm[1];
  P.pack_task = P.far_task + P.nfar;
  if (!all.empty())
    BIE_HIP_CHECK(hipMemcpyAsync(P.sweep_task, all.data(), all.size() * sizeof(int4),
                                 hipMemcpyHostToDevice, s));
  int4 *dch = P.list_buf.as<int4>();
  int2 *dti = reinterpret_cast<int2 *>(dch + chunks.size());
  if (!chunks.empty()) {
    BIE_HIP_CHECK(hipMemcpyAsync(dch, chunks.data(), chunks.size() * sizeof(int4),
                                 hipMemcpyHostToDevice, s));
    BIE_HIP_CHECK(hipMemcpyAsync(dti, tiles16.data(), tiles16.size() * sizeof(int2),
                                 hipMemcpyHostToDevice, s));
  }
  for (int i = 0; i < n; ++i) {
    desc[i].chunk = dch + chunk_at[i];
    desc[i].tile = dti + tile_at[i];
  }
  P.desc = P.desc_buf.as<ItemDesc>();
  BIE_HIP_CHECK(hipMemcpyAsync(P.desc, desc.data(), n * sizeof(ItemDesc), hipMemcpyHostToDevice, s));
  BIE_HIP_CHECK(hipStreamSynchronize(s));  // host vectors go out of scope
  P.npart = part;
  P.nfloat = floats;
  return BIE_OK;
}

}  // namespace

// out = (1/2 I + K + L) in for every active item (rhs blocks at items[i].io in flat vectors);
// inactive items get out = 0.
int multi_apply(MultiPlan *&P, const std::vector<MultiItem> &items, const std::vector<char> &active,
                int precision, const double *in, double *out, hipStream_t s,
                const std::vector<char> *item_f32) {
  if (!P) P = new MultiPlan();
  const int n = (int)items.size();
  if (item_f32 && ((int)item_f32->size() != n || n > kMaxPrecGroups)) {
    set_error("multi_apply: per-item precisions need one flag per item and at most 1024 items");
    return BIE_EINVAL;
  }
  auto f32_of = [&](int i) { return item_f32 ? (*item_f32)[i] != 0 : precision == BIE_MIXED; };
  bool same = P->valid && (int)P->key_gen.size() == n && P->key_active == active;
  for (int i = 0; same && i < n; ++i)
    same = P->key_gen[i] == items[i].g->gen && P->key_kind[i] == items[i].kind &&
           P->key_nrhs[i] == items[i].nrhs && P->key_fmm[i] == (char)items[i].fmm &&
           P->key_io[i] == items[i].io;
  if (!same) {
    P->valid = false;
    BIE_TRY(build_plan(*P, items, active, s));
    P->key_gen.resize(n);
    P->key_kind.resize(n);
    P->key_nrhs.resize(n);
    P->key_fmm.resize(n);
    P->key_io.resize(n);
    for (int i = 0; i < n; ++i) {
      P->key_gen[i] = items[i].g->gen;
      P->key_kind[i] = items[i].kind;
      P->key_nrhs[i] = items[i].nrhs;
      P->key_fmm[i] = (char)items[i].fmm;
      P->key_io[i] = items[i].io;
    }
    P->key_active = active;
    P->valid = true;
  }
  BIE_TRY(P->ws.reserve((size_t)P->npart * sizeof(double) + (size_t)P->nfloat * sizeof(float)));
  double *part = P->ws.as<double>();
  float *s32 = reinterpret_cast<float *>(part + P->npart);
  // inactive items (and FMM items, filled below) start from zero
  for (int i = 0; i < n; ++i)
    if (!active[i]) {
      const long long len = (long long)items[i].nrhs * items[i].g->M * (items[i].kind == 0 ? 1 : 2);
      BIE_HIP_CHECK(hipMemsetAsync(out + items[i].io, 0, len * sizeof(double), s));
    }
  if (P->nsweep > 0) {
    ItemMask mm{};
    mm.mode = item_f32 ? kBits : precision == BIE_MIXED ? kAll : kNone;
    bool any = mm.mode == kAll;
    for (int i = 0; item_f32 && i < n; ++i)
      if (f32_of(i)) {
        mm.w[i >> 6] |= 1ull << (i & 63);
        any = true;
      }
    for (int k = 1; any && k >= 0; --k) {
      if (P->nmm[k] == 0) continue;
      ProfScope prof(k ? BIE_K_FAR_STOKES_F32 : BIE_K_FAR_LAPLACE_F32, s, 0);
      if (k)
        hipLaunchKernelGGL(k_multi_mm<true>, dim3(P->nmm[k]), dim3(kBlock), 0, s, P->mm_task[k],
                           P->desc, in, mm, part);
      else
        hipLaunchKernelGGL(k_multi_mm<false>, dim3(P->nmm[k]), dim3(kBlock), 0, s, P->mm_task[k],
                           P->desc, in, mm, part);
    }
    if (any && P->nfar > 0) {
      ProfScope prof(BIE_K_FAR_STOKES_F32, s, 0);
      hipLaunchKernelGGL(k_multi_pack, dim3(P->npack), dim3(kBlock), 0, s, P->pack_task, P->desc, in,
                         mm, s32);
      hipLaunchKernelGGL(k_multi_far, dim3(P->nfar), dim3(kBlock), 0, s, P->far_task, P->desc, s32,
                         mm, part);
    }
    {
      ProfScope prof(P->nlap < P->nfin ? BIE_K_FAR_STOKES_F64 : BIE_K_FAR_LAPLACE_F64, s, 0);
      hipLaunchKernelGGL(k_multi_sweep, dim3(P->nsweep), dim3(kBlock), 0, s, P->sweep_task, P->desc,
                         in, mm, part);
    }
    ProfScope prof(BIE_K_EPILOGUE, s, 0);
    hipLaunchKernelGGL(k_multi_finish, dim3((P->nfin + 3) / 4), dim3(kBlock), 0, s, P->nfin,
                       P->nlap, P->fin_task, P->desc, in, mm, part, out);
  }
  BIE_HIP_CHECK(hipGetLastError());
  // FMM items: independent geometries overlap on the stream pool; items of one geometry share
  // its workspace and stay on one stream, in item order
  std::vector<const bie_geom *> gseen;
  std::vector<int> on(n, -1);
  for (int i = 0; i < n; ++i) {
    if (!active[i] || !items[i].fmm) continue;
    size_t gi = std::find(gseen.begin(), gseen.end(), items[i].g) - gseen.begin();
    if (gi == gseen.size()) gseen.push_back(items[i].g);
    on[i] = (int)(gi % kFmmStreams);
  }
  if (gseen.empty()) return BIE_OK;
  if (!P->fork) {
    // all streams are on one device: no system-scope fence at the event markers
    constexpr unsigned kFlags = hipEventDisableTiming | hipEventDisableSystemFence;
    BIE_HIP_CHECK(hipEventCreateWithFlags(&P->fork, kFlags));
    for (int k = 0; k < kFmmStreams; ++k) {
      BIE_HIP_CHECK(hipStreamCreateWithFlags(&P->pool[k], hipStreamNonBlocking));
      BIE_HIP_CHECK(hipEventCreateWithFlags(&P->join[k], kFlags));
    }
  }
  const int used = (int)std::min<size_t>(gseen.size(), kFmmStreams);
  BIE_HIP_CHECK(hipEventRecord(P->fork, s));
  for (int k = 0; k < used; ++k) BIE_HIP_CHECK(hipStreamWaitEvent(P->pool[k], P->fork, 0));
  int rc = BIE_OK;
  for (int i = 0; i < n && rc == BIE_OK; ++i)
    if (on[i] >= 0) {
      items[i].g->fmm_order = items[i].fmm_order;  // the caller's expansion order and leaf size
      items[i].g->fmm_leaf = items[i].fmm_leaf;
      rc = apply_operator(items[i].g, items[i].kind, f32_of(i) ? BIE_MIXED : BIE_FP64, BIE_FMM, 1,
                          1.0, items[i].nrhs, in + items[i].io, out + items[i].io, P->pool[on[i]],
                          items[i].merged);
    }
  for (int k = 0; k < used; ++k) {
    BIE_HIP_CHECK(hipEventRecord(P->join[k], P->pool[k]));
    BIE_HIP_CHECK(hipStreamWaitEvent(s, P->join[k], 0));
  }
  return rc;
}

}  // namespace bie

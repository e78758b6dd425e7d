// float64 vector kernels for the Arnoldi process over a set of independent systems ("segments")
// of possibly different lengths, stored back to back in flat vectors of Ntot entries. Work is
// cut into chunks that never straddle two systems; reductions are two-stage (per chunk, then per
// system in chunk order), so every result is bitwise reproducible run to run and independent of
// which other systems share the batch.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "internal.h"

namespace bie {
namespace {

__device__ inline double block_sum(double v, double *sh) {
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

// partial[l * C + c] = <V_l, w> over chunk c; grid (C, nvec), one workgroup per (chunk, vector)
__global__ __launch_bounds__(kBlock) void k_dots_stage1(int C, const long long *__restrict__ c0,
                                                       const long long *__restrict__ c1,
                                                       const double *__restrict__ V, long long vstride,
                                                       const double *__restrict__ w,
                                                       double *__restrict__ partial) {
  __shared__ double sh[4];
  const int c = blockIdx.x, l = blockIdx.y;
  const long long i0 = c0[c], i1 = c1[c];
  const double *v = V + l * vstride;
  double acc = 0.0;
  for (long long i = i0 + threadIdx.x; i < i1; i += kBlock) acc = fma(v[i], w[i], acc);
  const double t = block_sum(acc, sh);
  if (threadIdx.x == 0) partial[(long long)l * C + c] = t;
}

// h[s * hs + l] = sum over the chunks of system s (in order); sqrt for norms
__global__ __launch_bounds__(64) void k_dots_stage2(int C, const int *__restrict__ sys_chunk,
                                                   const double *__restrict__ partial,
                                                   double *__restrict__ h, long long hs, int do_sqrt) {
  const int l = blockIdx.x, s = blockIdx.y;
  const int a = sys_chunk[s], b = sys_chunk[s + 1];
  double acc = 0.0;
  for (int c = a + threadIdx.x; c < b; c += 64) acc += partial[(long long)l * C + c];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
  if (threadIdx.x == 0) h[s * hs + l] = do_sqrt ? sqrt(acc) : acc;
}

// w += sign * sum_l V_l h[s][l] on each chunk (s = system of the chunk); grid (C, kSub), each
// workgroup takes every kSub-th block of 256 entries of its chunk
__global__ __launch_bounds__(kBlock) void k_combination(int nvec, const int *__restrict__ csys,
                                                       const long long *__restrict__ c0,
                                                       const long long *__restrict__ c1,
                                                       const double *__restrict__ V, long long vstride,
                                                       const double *__restrict__ h, long long hs,
                                                       double *__restrict__ w, double sign) {
  const int c = blockIdx.x;
  const int s = csys[c];
  const double *hr = h + s * hs;
  for (long long i = c0[c] + blockIdx.y * kBlock + threadIdx.x; i < c1[c]; i += kSub * kBlock) {
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
    int l = 0;
    for (; l + 4 <= nvec; l += 4) {
      a0 = fma(V[l * vstride + i], hr[l], a0);
      a1 = fma(V[(l + 1) * vstride + i], hr[l + 1], a1);
      a2 = fma(V[(l + 2) * vstride + i], hr[l + 2], a2);
      a3 = fma(V[(l + 3) * vstride + i], hr[l + 3], a3);
    }
    // term l always goes to accumulator l mod 4, so trailing zero coefficients (a system frozen
    // inside a longer batch cycle) leave every sum unchanged
    if (l < nvec) a0 = fma(V[l * vstride + i], hr[l], a0);
    if (l + 1 < nvec) a1 = fma(V[(l + 1) * vstride + i], hr[l + 1], a1);
    if (l + 2 < nvec) a2 = fma(V[(l + 2) * vstride + i], hr[l + 2], a2);
    w[i] += sign * ((a0 + a1) + (a2 + a3));
  }
}

// The second Gram-Schmidt update fused with the norm of its result: as k_combination, and each
// workgroup (chunk c, part sub) writes the sum of squares of the entries it wrote to
// partial[c * kSub + sub].
__global__ __launch_bounds__(kBlock) void k_combination_nrm(
    int nvec, const int *__restrict__ csys, const long long *__restrict__ c0,
    const long long *__restrict__ c1, const double *__restrict__ V, long long vstride,
    const double *__restrict__ h, long long hs, double *__restrict__ w, double sign,
    double *__restrict__ partial) {
  __shared__ double sh[4];
  const int c = blockIdx.x;
  const int s = csys[c];
  const double *hr = h + s * hs;
  double sq = 0.0;
  for (long long i = c0[c] + blockIdx.y * kBlock + threadIdx.x; i < c1[c]; i += kSub * kBlock) {
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
    int l = 0;
    for (; l + 4 <= nvec; l += 4) {
      a0 = fma(V[l * vstride + i], hr[l], a0);
      a1 = fma(V[(l + 1) * vstride + i], hr[l + 1], a1);
      a2 = fma(V[(l + 2) * vstride + i], hr[l + 2], a2);
      a3 = fma(V[(l + 3) * vstride + i], hr[l + 3], a3);
    }
    if (l < nvec) a0 = fma(V[l * vstride + i], hr[l], a0);
    if (l + 1 < nvec) a1 = fma(V[(l + 1) * vstride + i], hr[l + 1], a1);
    if (l + 2 < nvec) a2 = fma(V[(l + 2) * vstride + i], hr[l + 2], a2);
    const double v = w[i] + sign * ((a0 + a1) + (a2 + a3));
    w[i] = v;
    sq = fma(v, v, sq);
  }
  const double t = block_sum(sq, sh);
  if (threadIdx.x == 0) partial[(long long)c * kSub + blockIdx.y] = t;
}

// Normalisation of the new Krylov vector, grid C + S: every workgroup of a system s sums s's
// partials in the same fixed order, so all of them form the same ||w||. Workgroup c < C writes
// v = w / ||w|| over chunk c; workgroup C + s completes the Hessenberg column,
// h2[s][0..cnt-1] += h1[s][...] and h2[s][cnt] = ||w||, stores ||w|| in nrm[s] and, when col_out
// is given (mapped host memory), writes the column there too, then (when flag is given) stores
// the tag of step *seq_base + seq_off in flag[s] once the column is visible to the host (the
// base is read when the kernel runs, so a captured graph of the step stays valid across
// cycles). What bounds it is that store's latency: one wave of a workgroup of its own releases
// its own stores, where a fence by all four waves of the system's first chunk also waited for
// that chunk of v (requests on 12 bodies of 96 nodes,
// 1,152 or 2,304 unknowns per system: 11.5 -> 5.4 us per step).
__global__ __launch_bounds__(kBlock) void k_normalize_column(
    int cnt, int C, const int *__restrict__ csys, const int *__restrict__ sys_chunk,
    const long long *__restrict__ c0, const long long *__restrict__ c1,
    const double *__restrict__ partial, const double *__restrict__ w, double *__restrict__ v,
    const double *__restrict__ h1, double *__restrict__ h2, long long hs,
    double *__restrict__ nrm, double *__restrict__ col_out, unsigned long long *flag,
    const unsigned long long *seq_base, unsigned long long seq_off) {
  __shared__ double sh[4];
  const int c = blockIdx.x, s = c < C ? csys[c] : c - C;
  const int a = sys_chunk[s] * kSub, b = sys_chunk[s + 1] * kSub;
  double acc = 0.0;
  for (int e = a + threadIdx.x; e < b; e += kBlock) acc += partial[e];
  const double n = sqrt(block_sum(acc, sh));
  if (c < C) {
    for (long long i = c0[c] + threadIdx.x; i < c1[c]; i += kBlock) v[i] = n > 0.0 ? w[i] / n : 0.0;
    return;
  }
  if (threadIdx.x >= 64) return;
  for (int l = threadIdx.x; l <= cnt; l += 64) {
    const double hv = l < cnt ? h2[s * hs + l] + h1[s * hs + l] : n;
    h2[s * hs + l] = hv;
    if (col_out) col_out[s * hs + l] = hv;
  }
  if (threadIdx.x == 0) nrm[s] = n;
  if (flag) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "");  // system scope
    if (threadIdx.x == 0)
      __hip_atomic_store(flag + s, column_tag(*seq_base + seq_off), __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

__global__ __launch_bounds__(kBlock) void k_scale_to(const int *__restrict__ csys,
                                                    const long long *__restrict__ c0,
                                                    const long long *__restrict__ c1,
                                                    const double *__restrict__ w,
                                                    const double *__restrict__ den,
                                                    double *__restrict__ v) {
  const int c = blockIdx.x;
  const double d = den[csys[c]];
  for (long long i = c0[c] + threadIdx.x; i < c1[c]; i += kBlock) v[i] = d > 0.0 ? w[i] / d : 0.0;
}

// ---- DCGS2 Arnoldi (classical Gram-Schmidt with delayed reorthogonalisation) ---------------
// Step j >= 1 works on U, the candidate for basis vector V_j after one projection, and
// Z = A U. One pass over V_0..V_{j-1} gives s = V^T U, t = V^T Z, U.U and U.Z (one reduction);
// from them a small per-system kernel finishes column j - 1 of the Hessenberg matrix (the first
// projection's coefficients plus s, and nu = sqrt(U.U - s.s) below the diagonal) and forms the
// coefficients of the next projection without another pass, using the Arnoldi relation
// A V_i = sum_k H[k][i] V_k: with V_j = (U - V s) / nu, A V_j = (Z - V (H s)) / nu, so
// V_k . A V_j = (t_k - (H s)_k) / nu (k < j) and ((U.Z - s.t) / nu - (H s)_j) / nu (k = j).
// A second pass writes V_j and the next candidate U' = A V_j - sum_{k<=j} g'_k V_k
// = Z / nu - sum_{k<=j} c_k V_k with c_k = (H s)_k / nu + g'_k.

// partial rows over chunk c: 2l = V_l . U and 2l + 1 = V_l . Z (l < nv); 2 nv = U . U and
// 2 nv + 1 = U . Z. Z NULL: the odd rows are zero. Grid (C, ceil((nv + 1) / kDotsVecs)): a
// workgroup holds its chunk of U and Z in registers (entries i0 + t + 256 k, k < kSub) and takes
// kDotsVecs of the vectors, so U and Z are read once per kDotsVecs vectors instead of once per
// vector. Each row's sum has the order of a one-vector reduction: per thread in entry order, the
// wave's shuffle tree, then the four waves as (w0 + w1) + (w2 + w3).
constexpr int kDotsVecs = 8;

__global__ __launch_bounds__(kBlock) void k_dots_uz(int C, const long long *__restrict__ c0,
                                                   const long long *__restrict__ c1, int nv,
                                                   const double *__restrict__ V, long long vstride,
                                                   const double *__restrict__ U,
                                                   const double *__restrict__ Z,
                                                   double *__restrict__ partial) {
  __shared__ double sh[4][2 * kDotsVecs];
  const int c = blockIdx.x, l0 = blockIdx.y * kDotsVecs;
  const int nl = min(kDotsVecs, nv + 1 - l0);
  const long long i0 = c0[c], i1 = c1[c], last = i1 > 0 ? i1 - 1 : 0;
  double u[kSub], z[kSub];
#pragma unroll
  for (int k = 0; k < kSub; ++k) {
    const long long i = i0 + threadIdx.x + (long long)k * kBlock;
    u[k] = i < i1 ? U[i] : 0.0;
    z[k] = (Z && i < i1) ? Z[i] : 0.0;
  }
  // every load of the workgroup's vectors is issued before the first product (places past the
  // last vector read U again, threads past the chunk's end its last entry against zeros): one
  // memory latency instead of one per vector (4,608 unknowns 7.8 -> 4.9 us per step, 256,000
  // unknowns 12.0 -> 7.5)
  double x[kDotsVecs][kSub];
#pragma unroll
  for (int q = 0; q < kDotsVecs; ++q) {
    const int l = l0 + q;
    const double *a = l < nv ? V + l * vstride : U;
#pragma unroll
    for (int k = 0; k < kSub; ++k) {
      const long long i = i0 + threadIdx.x + (long long)k * kBlock;
      x[q][k] = a[i < i1 ? i : last];
    }
  }
  double su[kDotsVecs], sz[kDotsVecs];
#pragma unroll
  for (int q = 0; q < kDotsVecs; ++q) {
    su[q] = sz[q] = 0.0;
#pragma unroll
    for (int k = 0; k < kSub; ++k) {
      su[q] = fma(x[q][k], u[k], su[q]);
      sz[q] = fma(x[q][k], z[k], sz[q]);
    }
  }
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < kDotsVecs; ++q) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      su[q] += __shfl_down(su[q], off, 64);
      sz[q] += __shfl_down(sz[q], off, 64);
    }
    if (lane == 0) {
      sh[wid][2 * q] = su[q];
      sh[wid][2 * q + 1] = sz[q];
    }
  }
  __syncthreads();
  if (threadIdx.x < 2 * nl) {
    const int x = threadIdx.x;
    const double t = (sh[0][x] + sh[1][x]) + (sh[2][x] + sh[3][x]);
    partial[(long long)(2 * l0 + x) * C + c] = t;
  }
}

// A finished column to the host: stored by one wave, whose flag store follows a release of its own
// stores only (a fence by every wave of the workgroup, ahead of the column's next use, cost about
// 3 us of each step).
__device__ __forceinline__ void notify_column(int cnt, const double *column, double *col_out,
                                              unsigned long long *flag,
                                              const unsigned long long *seq_base,
                                              unsigned long long seq_off) {
  const int lane = threadIdx.x & 63;
  for (int i = lane; i < cnt; i += 64) col_out[i] = column[i];
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "");  // system scope
  if (lane == 0)
    __hip_atomic_store(flag, column_tag(*seq_base + seq_off), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
}

// The sums of up to kFewChunks chunk sums in the order of k_dots_stage2's shuffle tree.
constexpr int kFewChunks = 8;
__device__ __forceinline__ double chunk_total(const double *p, long long stride, int C) {
  double x[kFewChunks];
#pragma unroll
  for (int c = 0; c < kFewChunks; ++c) x[c] = c < C ? p[c * stride] : 0.0;
  return ((x[0] + x[4]) + (x[2] + x[6])) + ((x[1] + x[5]) + (x[3] + x[7]));
}

// The small part of a DCGS2 step, for one system by one workgroup of T threads, from
// sv[i], tv[i] = s_i, t_i (i < j) and U.U, U.Z (i = j) in LDS: finishes column j - 1
// (col[i] = G[i] + s_i, col[j] = nu, also stored to the device copy Hd: column-major, leading
// dimension ldh) and, unless finalize, leaves the update's coefficients (s = sv for k < j,
// c_k = cc for k <= j, 1/nu returned) and G = g' (the first projection's coefficients of the next
// column). nu = 0 (breakdown) gives zero coefficients. Hl: step_h_lds(j) doubles of LDS with the
// columns of H before j - 1, which the product H s needs (HAhead: read while the reductions run).
constexpr int kHRead = 48;  // columns up to which H is read ahead into LDS
inline __host__ __device__ int step_h_lds(int j) { return j <= kHRead ? j * (j + 1) : 0; }

template <int T>
struct HAhead {
  static constexpr int N = (kHRead * (kHRead + 1) + T - 1) / T;
  double v[N];
  // columns 0 .. j - 2, rows 0 .. j of each (column i at i (j + 1))
  __device__ __forceinline__ void load(const double *H, long long ldh, int j) {
    if (j > kHRead) return;
#pragma unroll
    for (int e = 0; e < N; ++e) {
      const int x = threadIdx.x + e * T, i = x / (j + 1), k = x % (j + 1);
      if (x < (j - 1) * (j + 1)) v[e] = k <= i + 1 ? H[(long long)i * ldh + k] : 0.0;
    }
  }
  __device__ __forceinline__ void store(double *Hl, int j) const {
    if (j > kHRead) return;
#pragma unroll
    for (int e = 0; e < N; ++e) {
      const int x = threadIdx.x + e * T;
      if (x < (j - 1) * (j + 1)) Hl[x] = v[e];
    }
  }
};

template <int T>
__device__ __forceinline__ double dcgs_small_part(int j, bool finalize, const double *sv,
                                                  const double *tv, double *col, double *cc,
                                                  const double *Hl, double *red, double *G,
                                                  double *H, long long ldh) {
  const int t = threadIdx.x;
  // s.s and s.t in a fixed order (first wave: lanes stride, then the shuffle tree)
  if (t < 64) {
    double a = 0.0, b = 0.0;
    for (int i = t; i < j; i += 64) {
      a = fma(sv[i], sv[i], a);
      b = fma(sv[i], tv[i], b);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      a += __shfl_down(a, off, 64);
      b += __shfl_down(b, off, 64);
    }
    if (t == 0) {
      red[0] = a;
      red[1] = b;
    }
  }
  const double g0 = t < j ? G[t] : 0.0;
  __syncthreads();
  const double nu2 = sv[j] - red[0];
  const double nu = nu2 > 0.0 ? sqrt(nu2) : 0.0;
  for (int i = t; i <= j; i += T) {
    const double v = i < j ? (i < T ? g0 : G[i]) + sv[i] : nu;
    col[i] = v;
    H[(long long)(j - 1) * ldh + i] = v;
  }
  const double iv = nu > 0.0 ? 1.0 / nu : 0.0;
  __syncthreads();
  if (finalize) return iv;
  // (H s)_k = sum_{i < j} H[k][i] s_i, k = 0..j (H[k][i] = 0 for k > i + 1), in the order of i
  for (int k = t; k <= j; k += T) {
    double a = 0.0;
    int i = k > 0 ? k - 1 : 0;
    if (j <= kHRead) {
      for (; i < j - 1; ++i) a = fma(Hl[i * (j + 1) + k], sv[i], a);
    } else {
      for (; i + 8 <= j - 1; i += 8) {
        double h[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) h[e] = H[(long long)(i + e) * ldh + k];
#pragma unroll
        for (int e = 0; e < 8; ++e) a = fma(h[e], sv[i + e], a);
      }
      for (; i < j - 1; ++i) a = fma(H[(long long)i * ldh + k], sv[i], a);
    }
    a = fma(col[k], sv[j - 1], a);
    const double gn = k < j ? (tv[k] - a) * iv : ((tv[j] - red[1]) * iv - a) * iv;
    cc[k] = nu > 0.0 ? a * iv + gn : 0.0;
    G[k] = nu > 0.0 ? gn : 0.0;
  }
  __syncthreads();
  return iv;
}

// Per system (one workgroup): the small part of a step, from raw[s][2i], raw[s][2i + 1] or, with
// FEW (every system at most kFewChunks chunks), from the chunk sums themselves (partial, as
// k_dots_uz leaves them), which saves the launch that adds them. The update's coefficients go to
// sc, cc, inu; the column to the host with finalize only (else the update's launch sends it).
// Dynamic LDS: 4 (j + 1) + step_h_lds(j) doubles.
template <bool FEW>
__global__ __launch_bounds__(kBlock) void k_dcgs_small(
    int j, int finalize, const double *__restrict__ raw, long long rstride,
    const double *__restrict__ partial, int Ctot, const int *__restrict__ sys_chunk, double *G,
    double *Hd, long long ldh, long long hstride, double *__restrict__ sc,
    double *__restrict__ cc, double *__restrict__ inu, long long hs, double *__restrict__ col_out,
    unsigned long long *flag, const unsigned long long *seq_base, unsigned long long seq_off) {
  extern __shared__ double sm[];
  double *sv = sm, *tv = sm + (j + 1), *col = tv + (j + 1), *ccl = col + (j + 1), *Hl = ccl + (j + 1);
  __shared__ double red[2];
  const int s = blockIdx.x, t = threadIdx.x;
  double *H = Hd + s * hstride;
  HAhead<kBlock> ahead;
  if (!finalize) ahead.load(H, ldh, j);
  for (int r = t; r < 2 * (j + 1); r += kBlock) {
    double v;
    if (FEW) v = chunk_total(partial + (long long)r * Ctot + sys_chunk[s], 1, sys_chunk[s + 1] - sys_chunk[s]);
    else v = raw[s * rstride + r];
    ((r & 1) ? tv : sv)[r >> 1] = v;
  }
  if (!finalize) ahead.store(Hl, j);
  __syncthreads();
  const double iv = dcgs_small_part<kBlock>(j, finalize != 0, sv, tv, col, ccl, Hl, red,
                                            G + s * hs, H, ldh);
  if (finalize) {
    if (t < 64) notify_column(j + 1, col, col_out + s * hs, flag + s, seq_base, seq_off);
    return;
  }
  for (int k = t; k <= j; k += kBlock) {
    cc[s * hs + k] = ccl[k];
    if (k < j) sc[s * hs + k] = sv[k];
  }
  if (t == 0) inu[s] = iv;
}

// One entry of V_j = (U - sum_{k<j} sc_k V_k) / nu and of the next candidate
// U = Z / nu - sum_{k<j} cc_k V_k - cc_j V_j; term l goes to accumulator l mod 4. Eight entries of
// V are in flight at a time.
__device__ __forceinline__ void dcgs_entry(int j, const double *V, long long vstride, long long i,
                                           const double *sr, const double *cr, double iv, double u,
                                           double z, double &vj, double &unext) {
  double a[4] = {0.0, 0.0, 0.0, 0.0}, b[4] = {0.0, 0.0, 0.0, 0.0};
  int l = 0;
  for (; l + 8 <= j; l += 8) {
    double v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = V[(l + q) * vstride + i];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      a[q & 3] = fma(v[q], sr[l + q], a[q & 3]);
      b[q & 3] = fma(v[q], cr[l + q], b[q & 3]);
    }
  }
  if (l < j) {
    double v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = l + q < j ? V[(l + q) * vstride + i] : 0.0;
#pragma unroll
    for (int q = 0; q < 8; ++q)
      if (l + q < j) {
        a[q & 3] = fma(v[q], sr[l + q], a[q & 3]);
        b[q & 3] = fma(v[q], cr[l + q], b[q & 3]);
      }
  }
  vj = (u - ((a[0] + a[1]) + (a[2] + a[3]))) * iv;
  unext = z * iv - ((b[0] + b[1]) + (b[2] + b[3])) - cr[j] * vj;
}

// The update of a step, entry by entry (one pass over V_0..V_{j-1}); grid (C + S, kSub): chunk c's
// workgroups as k_combination, and workgroup (C + s, 0) sends system s's column j - 1 to the host
// meanwhile.
__global__ __launch_bounds__(kBlock) void k_dcgs_update(
    int j, int C, const int *__restrict__ csys, const long long *__restrict__ c0,
    const long long *__restrict__ c1, const double *__restrict__ V, long long vstride,
    const double *__restrict__ sc, const double *__restrict__ cc, const double *__restrict__ inu,
    long long hs, double *__restrict__ U, const double *__restrict__ Z, double *__restrict__ Vj,
    const double *__restrict__ Hd, long long ldh, long long hstride, double *__restrict__ col_out,
    unsigned long long *flag, const unsigned long long *seq_base, unsigned long long seq_off) {
  const int c = blockIdx.x;
  if (c >= C) {
    const int s = c - C;
    if (blockIdx.y == 0 && threadIdx.x < 64)
      notify_column(j + 1, Hd + s * hstride + (long long)(j - 1) * ldh, col_out + s * hs, flag + s,
                    seq_base, seq_off);
    return;
  }
  const int s = csys[c];
  const double iv = inu[s];
  for (long long i = c0[c] + blockIdx.y * kBlock + threadIdx.x; i < c1[c]; i += kSub * kBlock) {
    double vj, un;
    dcgs_entry(j, V, vstride, i, sc + s * hs, cc + s * hs, iv, U[i], Z[i], vj, un);
    Vj[i] = vj;
    U[i] = un;
  }
}

// ---- Arnoldi steps of small systems in one launch -------------------------------------------
// One workgroup per system of one chunk takes a whole Arnoldi step: the reductions, the small
// per-system part and the update, with the barriers of one workgroup where the separate kernels
// need launches. Every sum has the order of the separate kernels, so which of the two runs
// changes no bit and a batch may mix sizes. Bound by the latency of its phases; a longer system
// would be read through one compute unit (4,608 unknowns: 46 us per step at 20 vectors, the
// separate kernels 20), so only sets of one-chunk systems take it.
constexpr int kStepThreads = kChunk;
constexpr int kStepWaves = kStepThreads / 64;
constexpr int kStepVectors = kHRead;  // most basis vectors a fused step reads

// The sum that k_dots_stage1 / k_dots_uz forms over one chunk, by one wave: accumulator q stands for
// that kernel's wave q; x holds the vector (zero past the chunk's end).
__device__ __forceinline__ double chunk_dot(const double (&x)[kSub][4], const double *u) {
  const int lane = threadIdx.x & 63;
  double a[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    a[q] = 0.0;
#pragma unroll
    for (int k = 0; k < kSub; ++k) a[q] = fma(x[k][q], u[k * kBlock + q * 64 + lane], a[q]);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) a[q] += __shfl_down(a[q], off, 64);
  return (a[0] + a[1]) + (a[2] + a[3]);  // (valid in lane 0)
}

__device__ __forceinline__ void chunk_load(const double *v, int len, double (&x)[kSub][4]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int k = 0; k < kSub; ++k)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int e = k * kBlock + q * 64 + lane;
      x[k][q] = e < len ? v[e] : 0.0;
    }
}

// One DCGS2 step. Dynamic LDS: 4 (j + 1) + step_h_lds(j) doubles.
__global__ __launch_bounds__(kStepThreads) void k_dcgs_step(
    const int *__restrict__ sys_chunk, const long long *__restrict__ c0,
    const long long *__restrict__ c1, int j, int finalize, const double *__restrict__ V,
    long long vstride, double *G, double *Hd, long long ldh, long long hstride, long long hs,
    double *__restrict__ U, const double *__restrict__ Z, double *__restrict__ Vj,
    double *__restrict__ col_out, unsigned long long *flag, const unsigned long long *seq_base,
    unsigned long long seq_off) {
  extern __shared__ double sm[];
  __shared__ double us[kChunk], zs[kChunk], red[2];
  double *sv = sm, *tv = sv + (j + 1), *col = tv + (j + 1), *cc = col + (j + 1), *Hl = cc + (j + 1);
  const int s = blockIdx.x, t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const long long i0 = c0[sys_chunk[s]];
  const int len = (int)(c1[sys_chunk[s]] - i0);
  double *H = Hd + s * hstride;
  HAhead<kStepThreads> ahead;
  if (!finalize) ahead.load(H, ldh, j);
  const double ut = t < len ? U[i0 + t] : 0.0, zt = Z && t < len ? Z[i0 + t] : 0.0;
  double x[kSub][4];
  if (wv < j) chunk_load(V + wv * vstride + i0, len, x);
  us[t] = ut;
  zs[t] = zt;
  if (!finalize) ahead.store(Hl, j);
  __syncthreads();
  for (int l = wv; l <= j; l += kStepWaves) {
    if (l == j) {
#pragma unroll
      for (int k = 0; k < kSub; ++k)
#pragma unroll
        for (int q = 0; q < 4; ++q) x[k][q] = us[k * kBlock + q * 64 + lane];
    } else if (l != wv) {
      chunk_load(V + l * vstride + i0, len, x);
    }
#pragma unroll 1  // one at a time: both at once do not fit the registers of 16 waves
    for (int z = 0; z < 2; ++z) {
      const double a = chunk_dot(x, z ? zs : us);
      if (lane == 0) (z ? tv : sv)[l] = a;
    }
  }
  __syncthreads();
  const double iv = dcgs_small_part<kStepThreads>(j, finalize != 0, sv, tv, col, cc, Hl, red,
                                                  G + s * hs, H, ldh);
  if (!finalize && t < len) {
    double vj, un;
    dcgs_entry(j, V, vstride, i0 + t, sv, cc, iv, ut, zt, vj, un);
    Vj[i0 + t] = vj;
    U[i0 + t] = un;
  }
  if (wv == kStepWaves - 1) notify_column(j + 1, col, col_out + s * hs, flag + s, seq_base, seq_off);
}

// One classical Gram-Schmidt pass: h = V^T w (nv vectors), w -= V h, and with NORM the new basis
// vector vnext = w / ||w|| and the column (h, ||w||) (k_dots_stage1, k_dots_stage2,
// k_combination_nrm and k_normalize_column with a zero second pass); without, h is left in h_out
// (the first projection of a DCGS2 cycle).
template <bool NORM>
__global__ __launch_bounds__(kStepThreads) void k_cgs_step(
    const int *__restrict__ sys_chunk, const long long *__restrict__ c0,
    const long long *__restrict__ c1, int nv, const double *__restrict__ V, long long vstride,
    double *__restrict__ h_out, long long hs, double *__restrict__ w, double *__restrict__ nrm,
    double *__restrict__ vnext, double *__restrict__ col_out, unsigned long long *flag,
    const unsigned long long *seq_base, unsigned long long seq_off) {
  __shared__ double us[kChunk], ws[kStepWaves], h[kStepVectors + 1];
  const int s = blockIdx.x, t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const long long i0 = c0[sys_chunk[s]];
  const int len = (int)(c1[sys_chunk[s]] - i0);
  const double wt = t < len ? w[i0 + t] : 0.0;
  us[t] = wt;
  __syncthreads();
  for (int l = wv; l < nv; l += kStepWaves) {
    double x[kSub][4];
    chunk_load(V + l * vstride + i0, len, x);
    const double a = chunk_dot(x, us);
    if (lane == 0) h[l] = a;
  }
  __syncthreads();
  double v = 0.0;
  if (t < len) {
    double a[4] = {0.0, 0.0, 0.0, 0.0};
    for (int l = 0; l < nv; l += 8) {
      double y[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) y[q] = l + q < nv ? V[(l + q) * vstride + i0 + t] : 0.0;
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (l + q < nv) a[q & 3] = fma(y[q], h[l + q], a[q & 3]);
    }
    v = wt + -1.0 * ((a[0] + a[1]) + (a[2] + a[3]));
    w[i0 + t] = v;
  }
  for (int l = t; l < nv; l += kStepThreads) h_out[s * hs + l] = h[l];
  if (!NORM) return;
  double sq = t < len ? fma(v, v, 0.0) : 0.0;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) sq += __shfl_down(sq, off, 64);
  if (lane == 0) ws[wv] = sq;
  __syncthreads();
  // the four workgroups' parts of k_combination_nrm, added in k_normalize_column's tree
  double part[kSub];
#pragma unroll
  for (int q = 0; q < kSub; ++q)
    part[q] = (ws[4 * q] + ws[4 * q + 1]) + (ws[4 * q + 2] + ws[4 * q + 3]);
  const double n = sqrt((part[0] + part[2]) + (part[1] + part[3]));
  if (t < len) vnext[i0 + t] = n > 0.0 ? v / n : 0.0;
  if (t == 0) {
    nrm[s] = n;
    h_out[s * hs + nv] = n;
  }
  if (wv == kStepWaves - 1) {
    if (lane == 0) h[nv] = n;
    notify_column(nv + 1, h, col_out + s * hs, flag + s, seq_base, seq_off);
  }
}

__global__ void k_axpby(long long total, double a, const double *__restrict__ x, double b,
                        double *__restrict__ y) {
  const long long i = (long long)blockIdx.x * kBlock + threadIdx.x;
  if (i < total) y[i] = a * x[i] + b * y[i];
}

// A set of copies or sums of ranges (a request's part of a flat vector is one), grid (blocks of the
// longest, moves). The table travels with the launch. Each range's own copy or launch took 1.8 to
// 2.2 us and the gap behind it, whatever its 10 to 20 KB: 24 served requests issued about
// 300 and 75 (now 98 and 28), 4.30 -> 3.44 ms.
struct MoveTable {
  VecMove m[kMoves];
};

template <bool ADD>
__global__ __launch_bounds__(kBlock) void k_move(const MoveTable t) {
  const VecMove m = t.m[blockIdx.y];
  for (long long i = (long long)blockIdx.x * kBlock + threadIdx.x; i < m.n;
       i += (long long)gridDim.x * kBlock) {
    const double v = m.src ? m.src[i] : 0.0;
    m.dst[i] = ADD ? m.dst[i] + v : v;
  }
}

__global__ void k_add_h(int cnt, long long hs, const double *__restrict__ h1, double *__restrict__ h2) {
  const int s = blockIdx.x;
  for (int l = threadIdx.x; l < cnt; l += blockDim.x) h2[s * hs + l] += h1[s * hs + l];
}

// Sets whose systems all have few chunks: the consumer adds a reduction's chunk sums.
bool few_chunks(const Segments &sg) { return sg.max_len <= (long long)kFewChunks * kChunk; }

}  // namespace

int seg_dots(const Segments &sg, int nvec, const double *V, long long vstride, const double *w,
             double *h, long long hs, double *scratch, hipStream_t s) {
  if (nvec <= 0) return BIE_OK;
  hipLaunchKernelGGL(k_dots_stage1, dim3(sg.C, nvec), dim3(kBlock), 0, s, sg.C, sg.c0, sg.c1, V,
                     vstride, w, scratch);
  hipLaunchKernelGGL(k_dots_stage2, dim3(nvec, sg.S), dim3(64), 0, s, sg.C, sg.sys_chunk, scratch,
                     h, hs, 0);
  BIE_HIP_CHECK(hipGetLastError());
  return BIE_OK;
}

int seg_combination(const Segments &sg, int nvec, const double *V, long long vstride,
                    const double *h, long long hs, double *w, double sign, hipStream_t s) {
  if (nvec <= 0) return BIE_OK;
  hipLaunchKernelGGL(k_combination, dim3(sg.C, kSub), dim3(kBlock), 0, s, nvec, sg.csys, sg.c0,
                     sg.c1, V, vstride, h, hs, w, sign);
  BIE_HIP_CHECK(hipGetLastError());
  return BIE_OK;
}

int seg_nrm2(const Segments &sg, const double *w, double *out, double *scratch, hipStream_t s) {
  hipLaunchKernelGGL(k_dots_stage1, dim3(sg.C, 1), dim3(kBlock), 0, s, sg.C, sg.c0, sg.c1, w, 0LL,
                     w, scratch);
  hipLaunchKernelGGL(k_dots_stage2, dim3(1, sg.S), dim3(64), 0, s, sg.C, sg.sys_chunk, scratch, out,
                     1LL, 1);
  BIE_HIP_CHECK(hipGetLastError());
  return BIE_OK;
}

int seg_combination_column(const Segments &sg, int nvec, const double *V, long long vstride,
                           const double *h1, double *h2, long long hs, double *w, double *nrm,
                           double *vnext, double *col_out, unsigned long long *flag,
                           const unsigned long long *seq_base, unsigned long long seq_off,
                           double *scratch, hipStream_t s) {
  if (nvec <= 0) return BIE_OK;
  hipLaunchKernelGGL(k_combination_nrm, dim3(sg.C, kSub), dim3(kBlock), 0, s, nvec, sg.csys, sg.c0,
                     sg.c1, V, vstride, h2, hs, w, -1.0, scratch);
  hipLaunchKernelGGL(k_normalize_column, dim3(sg.C + sg.S), dim3(kBlock), 0, s, nvec, sg.C, sg.csys,
                     sg.sys_chunk, sg.c0, sg.c1, scratch, w, vnext, h1, h2, hs, nrm, col_out, flag,
                     seq_base, seq_off);
  BIE_HIP_CHECK(hipGetLastError());
  return BIE_OK;
}

int dcgs_dots(const Segments &sg, int nv, const double *V, long long vstride, const double *U,
              const double *Z, double *raw, long long rstride, double *scratch, hipStream_t s) {
  hipLaunchKernelGGL(k_dots_uz, dim3(sg.C, (nv + kDotsVecs) / kDotsVecs), dim3(kBlock), 0, s,
                     sg.C, sg.c0, sg.c1, nv, V, vstride, U, Z, scratch);
  if (!few_chunks(sg))  // else dcgs_small adds the chunk sums itself
    hipLaunchKernelGGL(k_dots_stage2, dim3(2 * nv + 2, sg.S), dim3(64), 0, s, sg.C, sg.sys_chunk,
                       scratch, raw, rstride, 0);
  BIE_HIP_CHECK(hipGetLastError());
  return BIE_OK;
}

int dcgs_small(const Segments &sg, int j, bool finalize, const double *raw, long long rstride,
               const double *scratch, double *G, double *Hd, long long ldh, long long hstride,
               double *sc, double *cc, double *inu, long long hs, double *col_out,
               unsigned long long *flag, const unsigned long long *seq_base,
               unsigned long long seq_off, hipStream_t s) {
  const size_t lds = (size_t)(4 * (j + 1) + step_h_lds(j)) * sizeof(double);
  if (few_chunks(sg))
    hipLaunchKernelGGL(k_dcgs_small<true>, dim3(sg.S), dim3(kBlock), lds, s, j, finalize ? 1 : 0,
                       raw, rstride, scratch, sg.C, sg.sys_chunk, G, Hd, ldh, hstride, sc, cc, inu,
                       hs, col_out, flag, seq_base, seq_off);
  else
    hipLaunchKernelGGL(k_dcgs_small<false>, dim3(sg.S), dim3(kBlock), lds, s, j, finalize ? 1 : 0,
                       raw, rstride, scratch, sg.C, sg.sys_chunk, G, Hd, ldh, hstride, sc, cc, inu,
                       hs, col_out, flag, seq_base, seq_off);
  BIE_HIP_CHECK(hipGetLastError());
  return BIE_OK;
}

int dcgs_update(const Segments &sg, int j, const double *V, long long vstride, const double *sc,
                const double *cc, const double *inu, long long hs, double *U, const double *Z,
                double *Vj, const double *Hd, long long ldh, long long hstride, double *col_out,
                unsigned long long *flag, const unsigned long long *seq_base,
                unsigned long long seq_off, hipStream_t s) {
  hipLaunchKernelGGL(k_dcgs_update, dim3(sg.C + sg.S, kSub), dim3(kBlock), 0, s, j, sg.C, sg.csys,
                     sg.c0, sg.c1, V, vstride, sc, cc, inu, hs, U, Z, Vj, Hd, ldh, hstride,
                     col_out, flag, seq_base, seq_off);
  BIE_HIP_CHECK(hipGetLastError());
  return BIE_OK;
}

bool step_is_small(const Segments &sg, int vectors) {
  return vectors <= kStepVectors && sg.max_len <= kChunk;
}

int dcgs_step(const Segments &sg, int j, bool finalize, const double *V, long long vstride,
              double *G, double *Hd, long long ldh, long long hstride, long long hs, double *U,
              const double *Z, double *Vj, double *col_out, unsigned long long *flag,
              const unsigned long long *seq_base, unsigned long long seq_off, hipStream_t s) {
  const size_t lds = (size_t)(4 * (j + 1) + step_h_lds(j)) * sizeof(double);
  hipLaunchKernelGGL(k_dcgs_step, dim3(sg.S), dim3(kStepThreads), lds, s, sg.sys_chunk, sg.c0,
                     sg.c1, j, finalize ? 1 : 0, V, vstride, G, Hd, ldh, hstride, hs, U, Z, Vj,
                     col_out, flag, seq_base, seq_off);
  BIE_HIP_CHECK(hipGetLastError());
  return BIE_OK;
}

int cgs_step(const Segments &sg, int nv, bool norm, const double *V, long long vstride, double *h,
             long long hs, double *w, double *nrm, double *vnext, double *col_out,
             unsigned long long *flag, const unsigned long long *seq_base,
             unsigned long long seq_off, hipStream_t s) {
  if (norm)
    hipLaunchKernelGGL(k_cgs_step<true>, dim3(sg.S), dim3(kStepThreads), 0, s, sg.sys_chunk, sg.c0,
                       sg.c1, nv, V, vstride, h, hs, w, nrm, vnext, col_out, flag, seq_base, seq_off);
  else
    hipLaunchKernelGGL(k_cgs_step<false>, dim3(sg.S), dim3(kStepThreads), 0, s, sg.sys_chunk, sg.c0,
                       sg.c1, nv, V, vstride, h, hs, w, nrm, vnext, col_out, flag, seq_base, seq_off);
  BIE_HIP_CHECK(hipGetLastError());
  return BIE_OK;
}

int seg_scale_to(const Segments &sg, const double *w, const double *den, double *v, hipStream_t s) {
  hipLaunchKernelGGL(k_scale_to, dim3(sg.C), dim3(kBlock), 0, s, sg.csys, sg.c0, sg.c1, w, den, v);
  BIE_HIP_CHECK(hipGetLastError());
  return BIE_OK;
}

int vec_axpby(long long total, double a, const double *x, double b, double *y, hipStream_t s) {
  hipLaunchKernelGGL(k_axpby, dim3((unsigned)((total + kBlock - 1) / kBlock)), dim3(kBlock), 0, s,
                     total, a, x, b, y);
  BIE_HIP_CHECK(hipGetLastError());
  return BIE_OK;
}

int vec_move(const std::vector<VecMove> &moves, bool add, hipStream_t s) {
  for (size_t at = 0; at < moves.size(); at += kMoves) {
    const size_t cnt = std::min<size_t>(kMoves, moves.size() - at);
    MoveTable t{};
    long long most = 0;
    for (size_t k = 0; k < cnt; ++k) {
      t.m[k] = moves[at + k];
      most = std::max(most, t.m[k].n);
    }
    if (most <= 0) continue;
    const dim3 grid((unsigned)std::min<long long>((most + kBlock - 1) / kBlock, 1024), (unsigned)cnt);
    if (add)
      hipLaunchKernelGGL(k_move<true>, grid, dim3(kBlock), 0, s, t);
    else
      hipLaunchKernelGGL(k_move<false>, grid, dim3(kBlock), 0, s, t);
  }
  BIE_HIP_CHECK(hipGetLastError());
  return BIE_OK;
}

int seg_add_h(int S, const double *h1, double *h2, int cnt, long long hs, hipStream_t s) {
  hipLaunchKernelGGL(k_add_h, dim3(S), dim3(64), 0, s, cnt, hs, h1, h2);
  BIE_HIP_CHECK(hipGetLastError());
  return BIE_OK;
}

// Chunk list of systems with the given lengths (flat, back to back).
int Segments::build(const std::vector<long long> &lens, hipStream_t s,
                    const std::vector<long long> *starts) {
  S = (int)lens.size();
  std::vector<long long> a, b;
  std::vector<int> cs, sc(1, 0);
  long long off = 0;
  h_off.assign(S + 1, 0);
  for (int k = 0; k < S; ++k) {
    const long long n = lens[k];
    if (starts) off = (*starts)[k];
    h_off[k] = off;
    const long long per = kChunk;  // chunk length
    for (long long i = 0; i < n; i += per) {
      a.push_back(off + i);
      b.push_back(off + std::min(n, i + per));
      cs.push_back(k);
    }
    if (n == 0) {  // keep one empty chunk so stage 2 sees the system
      a.push_back(off);
      b.push_back(off);
      cs.push_back(k);
    }
    sc.push_back((int)cs.size());
    off += n;
    h_off[k + 1] = off;
  }
  // h_off[k] is the start of system k; h_off[S] the end of the last one
  max_len = 0;
  for (long long n : lens) max_len = std::max(max_len, n);
  C = (int)cs.size();
  Ntot = off;
  const size_t bytes = (size_t)C * (8 + 8 + 4) + (S + 1) * 4 + 256;
  BIE_TRY(buf.reserve(bytes));
  char *q = buf.as<char>();
  c0 = (long long *)q;
  c1 = c0 + C;
  csys = (int *)(c1 + C);
  sys_chunk = csys + C;
  BIE_HIP_CHECK(hipMemcpyAsync(c0, a.data(), C * 8, hipMemcpyHostToDevice, s));
  BIE_HIP_CHECK(hipMemcpyAsync(c1, b.data(), C * 8, hipMemcpyHostToDevice, s));
  BIE_HIP_CHECK(hipMemcpyAsync(csys, cs.data(), C * 4, hipMemcpyHostToDevice, s));
  BIE_HIP_CHECK(hipMemcpyAsync(sys_chunk, sc.data(), (S + 1) * 4, hipMemcpyHostToDevice, s));
  BIE_HIP_CHECK(hipStreamSynchronize(s));
  return BIE_OK;
}

}  // namespace bie

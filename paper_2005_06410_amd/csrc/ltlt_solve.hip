// Solve X x = b with the factors of ltlt_factor.  With P X P^T = L T L^T,
// X x = b is L T L^T (P x) = P b, so (per right-hand side)
//   y = P b            y[i] = b[perm[i]], perm = the exchanges (i, ipiv[i])
//                      applied in order to the identity ordering;
//   z = L^{-1} y       forward substitution, L unit lower with L(:,0) = e_0
//                      and L(r, c) = A(r, c-1) for r >= c+1 (packed storage);
//   w = T^{-1} z       T skew tridiagonal, T(k+1,k) = alpha_k = A(k+1,k): row 0
//                      and the even rows give the odd unknowns forward, row
//                      n-1 and the odd rows the even unknowns backward;
//   u = L^{-T} w       backward substitution;
//   x = P^T u          x[perm[i]] = u[i].
//
// gfx950 mapping:
//  * perm: every row follows its own moves through the exchanges, in
//    parallel (the steps bucketed by the position they target);
//  * the inverses of the 64x64 unit lower diagonal blocks of L, and their
//    products with the nearest off-diagonal tile in each direction, are formed
//    first, all blocks at once (off the dependency chain);
//  * the triangular solves are persistent kernels over 64-row blocks,
//    left-looking: the waves of block b's workgroup stream their columns of
//    the 64x64 tiles of L to the left of its diagonal block (forward) or below
//    it (backward) through registers, each waiting for the stamped solution
//    words of the block a tile multiplies, except the nearest; then each wave
//    takes one right-hand side alone: the residual times the inverse of the
//    diagonal block (its transpose, backward), minus the precomputed product
//    with the nearest block's solution, waited for only then (one 64-term
//    product on the chain from block to block instead of a tile and a 64-step
//    substitution), and publishes its solution as stamped words.  A workgroup
//    takes its blocks in dependency order, so the earliest unfinished block
//    always has its inputs and the grid cannot deadlock; every wait is
//    bounded.  Each solve reads the lower triangle of L once;
//  * each recurrence of T (w_s = a_s w_{s-1} + b_s along one parity) runs
//    as a chunked scan: every thread of a workgroup composes the affine maps of
//    its chunk of steps, the workgroup scans the compositions, and every thread
//    then re-runs its chunk from its starting value with the recurrence as
//    written; one workgroup per (right-hand side, chain), the reciprocals of
//    alpha formed in parallel beforehand.
// Right-hand sides are taken kSolveRhs at a time, kSolveGroup to a workgroup.

#include "ltlt_device.h"
#include "ltlt_exchange.h"
#include "ltlt_internal.h"

#include <atomic>

namespace ltlt {

constexpr int kSB = 64;                // rows per block
constexpr int kSLd = kSB + 1;          // LDS stride of a tile column (bank spread)
constexpr int kSThreads = 256;         // 4 waves

// ---- permutation ----------------------------------------------------------
// perm[i] = index of the row at position i after the exchanges (i, ipiv[i]),
// i = 0 .. n-1 in order, with ipiv[i] >= i, so position i is final once step
// i is done.  Computed per row, in parallel: a row at position x at step t
// is moved next either by the first step s in [t, x) with ipiv[s] = x (it
// then lands at s, final), or, failing that, by step x itself (to ipiv[x],
// or it stays at x when ipiv[x] = x).  The steps are bucketed by the position
// they target (count, scan, scatter), then every row walks its positions.
__global__ void perm_count_kernel(int n, const int* ipiv, int* cnt) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s < n) {
    const int x = ipiv[s];
    if (x > s && x < n) atomicAdd(&cnt[x], 1);
  }
}

// exclusive prefix sum of cnt[0..n) into off[0..n] (one workgroup)
__global__ void __launch_bounds__(1024) perm_scan_kernel(int n, const int* cnt, int* off) {
  __shared__ int part[1024];
  const int t = threadIdx.x;
  const int per = (n + 1023) / 1024;
  const int lo = min(n, t * per), hi = min(n, lo + per);
  int sum = 0;
#pragma unroll 8
  for (int i = lo; i < hi; ++i) sum += cnt[i];
  part[t] = sum;
  __syncthreads();
  for (int d = 1; d < 1024; d <<= 1) {            // inclusive scan of the per-thread sums
    const int v = t >= d ? part[t - d] : 0;
    __syncthreads();
    part[t] += v;
    __syncthreads();
  }
  int run = part[t] - sum;
#pragma unroll 8
  for (int i = lo; i < hi; ++i) { off[i] = run; run += cnt[i]; }
  if (t == 1023) off[n] = part[1023];
}

__global__ void perm_scatter_kernel(int n, const int* ipiv, const int* off, int* fill, int* list) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s < n) {
    const int x = ipiv[s];
    if (x > s && x < n) list[off[x] + atomicAdd(&fill[x], 1)] = s;
  }
}

__global__ void perm_walk_kernel(int n, const int* ipiv, const int* off, const int* list, int* perm) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n) return;
  int x = r, t = 0;
  for (;;) {
    int first = INT32_MAX;                         // first step s in [t, x) targeting x
    for (int e = off[x]; e < off[x + 1]; ++e) {
      const int s = list[e];
      if (s >= t && s < first) first = s;
    }
    if (first != INT32_MAX) { x = first; break; }
    const int p = ipiv[x];
    if (p <= x || p >= n) break;                   // no move (ipiv[x] = x)
    t = x + 1;
    x = p;
  }
  perm[x] = r;
}

template <typename T>
__global__ void solve_gather_kernel(int n, int nr, const int* perm, const T* B, int64_t ldb, T* Y, int64_t ldy) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int q = blockIdx.y;
  if (i < n && q < nr) Y[(int64_t)i + (int64_t)q * ldy] = B[(int64_t)perm[i] + (int64_t)q * ldb];
}

template <typename T>
__global__ void solve_scatter_kernel(int n, int nr, const int* perm, const T* Y, int64_t ldy, T* B, int64_t ldb) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int q = blockIdx.y;
  if (i < n && q < nr) B[(int64_t)perm[i] + (int64_t)q * ldb] = Y[(int64_t)i + (int64_t)q * ldy];
}

// alpha_k = A(k+1, k) and its reciprocal, k < n-1
template <typename T>
__global__ void solve_alpha_kernel(int n, const T* A, int64_t lda, T* alpha, T* ralpha) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k + 1 < n) {
    const T a = A[(int64_t)(k + 1) + (int64_t)k * lda];
    alpha[k] = a;
    ralpha[k] = T(1) / a;
  }
}

__global__ void zero_ints_kernel(int* v, int count) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) v[i] = 0;
}

// ---- skew tridiagonal recurrences -----------------------------------------
// One workgroup per (right-hand side q, chain): even blocks run the odd unknowns
// forward, odd blocks the even unknowns backward.  Both chains are
// w_s = a_s w_{s-1} + b_s over s = 1 .. n/2 - 1 after a first value w_0:
//   odd:  i = 2s,        W[i+1] = (alpha_{i-1} W[i-1] - R[i]) / alpha_i,  w_0 = W[1] = -R[0] / alpha_0
//   even: i = n-1-2s,    W[i-1] = (R[i] + alpha_i W[i+1]) / alpha_{i-1},  w_0 = W[n-2] = R[n-1] / alpha_{n-2}
// Thread j takes the steps of chunk j (C consecutive steps): it composes their
// maps (A, B) with w_end = A w_start + B, the workgroup forms the exclusive
// prefix compositions (a shuffle scan in each wave, then over the waves), and
// each thread re-runs its chunk from w_start = A_prefix w_0 + B_prefix, writing
// every unknown with the recurrence as written above.  Each chain reads the
// other parity's inputs, so the result goes to a separate buffer W.  Bound by
// the serial chunk: 1024 threads per chain (8 steps at n = 16384) instead of
// one wave (128 steps) took it from 82 to 40 us.
template <typename T>
__device__ __forceinline__ void tri_step_coeffs(bool odd, int n, int s, const T* alpha, const T* ralpha, const T* R,
                                                T& ca, T& cb, T& cr, int& out) {
  if (odd) {                                       // i = 2s: W[i+1] = (alpha_{i-1} w - R[i]) * ralpha[i]
    const int i = 2 * s;
    ca = alpha[i - 1]; cb = R[i]; cr = ralpha[i]; out = i + 1;
  } else {                                         // i = n-1-2s: W[i-1] = (R[i] + alpha_i w) * ralpha[i-1]
    const int i = n - 1 - 2 * s;
    ca = alpha[i]; cb = R[i]; cr = ralpha[i - 1]; out = i - 1;
  }
}

constexpr int kTriWaves = 16;
template <typename T>
__global__ void __launch_bounds__(kTriWaves * kWave) solve_tridiag_kernel(int n, const T* alpha, const T* ralpha,
                                                                         const T* Y, T* W, int64_t ldy) {
  __shared__ T wa[kTriWaves], wb[kTriWaves];       // each wave's whole composition
  const int wave = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
  const int q = blockIdx.x >> 1;
  const bool odd = (blockIdx.x & 1) == 0;
  const T* R = Y + (int64_t)q * ldy;
  T* Wq = W + (int64_t)q * ldy;
  const int half = n / 2;                          // unknowns per chain
  const T w0 = odd ? -R[0] * ralpha[0] : R[n - 1] * ralpha[n - 2];
  if (threadIdx.x == 0) Wq[odd ? 1 : n - 2] = w0;
  const int steps = half - 1;                      // s = 1 .. half-1
  const int C = (steps + kTriWaves * kWave - 1) / (kTriWaves * kWave);   // steps per thread
  const int s_lo = 1 + threadIdx.x * C, s_hi = min(half, s_lo + C);
  // composition of this chunk's maps: w -> a w + b, a = ca cr (odd) / ca cr,
  // b = -cb cr (odd) / cb cr (even)
  T Ac = T(1), Bc = T(0);
#pragma unroll 8
  for (int s = s_lo; s < s_hi; ++s) {
    T ca, cb, cr;
    int out;
    tri_step_coeffs(odd, n, s, alpha, ralpha, R, ca, cb, cr, out);
    const T a = ca * cr, b = odd ? -cb * cr : cb * cr;
    Ac = a * Ac;
    Bc = fma(a, Bc, b);
  }
  // inclusive scan of the compositions in lane order (later maps applied
  // after earlier ones: (A2, B2) o (A1, B1) = (A2 A1, A2 B1 + B2))
  T Ai = Ac, Bi = Bc;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const T Ap = __shfl_up(Ai, off, kWave), Bp = __shfl_up(Bi, off, kWave);
    if (lane >= off) {
      Bi = fma(Ai, Bp, Bi);
      Ai = Ai * Ap;
    }
  }
  if (lane == kWave - 1) { wa[wave] = Ai; wb[wave] = Bi; }
  __syncthreads();
  // exclusive prefix: the earlier waves', then the inclusive one of the
  // previous lane
  T Ae = __shfl_up(Ai, 1, kWave), Be = __shfl_up(Bi, 1, kWave);
  if (lane == 0) { Ae = T(1); Be = T(0); }
  T w = w0;                                        // value entering this wave's chunks
  for (int v = 0; v < wave; ++v) w = fma(wa[v], w, wb[v]);
  w = fma(Ae, w, Be);                              // value entering this chunk
#pragma unroll 8
  for (int s = s_lo; s < s_hi; ++s) {
    T ca, cb, cr;
    int out;
    tri_step_coeffs(odd, n, s, alpha, ralpha, R, ca, cb, cr, out);
    w = odd ? (ca * w - cb) * cr : (cb + ca * w) * cr;
    Wq[out] = w;
  }
}

// ---- triangular solves ----------------------------------------------------
struct SolveTriArgs {
  const void* A;
  int64_t lda;
  int n;
  int nblk;
  void* Y;
  int64_t ldy;
  int nr;             // right-hand sides of this pass (<= kSolveRhs); a workgroup sees its group's
  uint64_t* box;      // [group][nblk][kSolveGroup][kSB][2] stamped solution words
  unsigned stamp;     // stamp of this launch (never 0)
  int* status;
  const void* Dinv;   // inverses of the diagonal blocks of L: [nblk][64 * 64], column-major
  const void* Mf;     // D_b^{-1} L_{b,b-1}: [nblk][64 * 64], column-major
  const void* Mb;     // D_b^{-T} L_{b+1,b}^T: [nblk][64 * 64], column-major
};

// A solution value crosses workgroups as two 64-bit words, each holding one
// 32-bit half of the value above the 32-bit stamp of the launch: naturally
// aligned 64-bit stores are single-copy atomic, so a reader that sees the
// stamp in both words has the value, without a separate flag (and the writer
// does not wait for its stores before signalling).  Words of an earlier
// launch carry an older stamp and never validate.
template <typename T>
__device__ __forceinline__ void box_put(uint64_t* w, T x, unsigned stamp) {
  unsigned hi, lo;
  if constexpr (sizeof(T) == 8) {
    hi = (unsigned)__double2hiint(x);
    lo = (unsigned)__double2loint(x);
  } else {
    hi = __float_as_uint(x);
    lo = 0u;
  }
  st_coh64(&w[0], ((uint64_t)hi << 32) | stamp);
  st_coh64(&w[1], ((uint64_t)lo << 32) | stamp);
}
template <typename T>
__device__ __forceinline__ bool box_get(const uint64_t* w, unsigned stamp, T& x) {
  const uint64_t w0 = ld_coh64(&w[0]), w1 = ld_coh64(&w[1]);
  if ((unsigned)w0 != stamp || (unsigned)w1 != stamp) return false;
  if constexpr (sizeof(T) == 8) x = __hiloint2double((int)(w0 >> 32), (int)(w1 >> 32));
  else x = __uint_as_float((unsigned)(w0 >> 32));
  return true;
}

// L(r, c) for global row r and column c: unit lower, L(:,0) = e_0,
// L(r, c) = A(r, c-1) below the diagonal.
template <typename T>
__device__ __forceinline__ T l_entry(const T* A, int64_t lda, int n, int r, int c) {
  if (r >= n || c >= n || r <= c || c == 0) return T(0);
  return A[(int64_t)r + (int64_t)(c - 1) * lda];
}

// Per 64-row block b: the inverse of its unit lower diagonal block D_b of L
// and the matrices that carry the nearest dependency of each substitution,
//   Mf_b = D_b^{-1} L_{b,b-1}        (forward, b >= 1),
//   Mb_b = D_b^{-T} L_{b+1,b}^T      (backward, b + 1 < nblk),
// so that z_b = D_b^{-1} r_b - Mf_b z_{b-1} and u_b = D_b^{-T} r_b - Mb_b u_{b+1},
// where r_b is the block's right-hand side less the contributions of every
// farther block.  All are stored column-major per block, X[b*64*64 + k*64 + r] =
// X(r, k); rows and columns past n give the identity (D_b^{-1}) or zeros (M),
// which the solves never use.

// D_b^{-1}, one wave per block: lane c forms column c by forward substitution,
// column k of D (from LDS by broadcast, two entries a read) applied to every
// later row at once, so that its products are independent.  Entry by entry,
// each a chain of products, it took 45 us at n = 16384; 23 now.
template <typename T>
__global__ void __launch_bounds__(kWave) solve_dinv_kernel(const T* A, int64_t lda, int n, T* Dinv) {
  __shared__ __align__(16) T d[kSB * kSB];         // D(r, c) at d[c * kSB + r]
  __shared__ T t[kSB * kSLd];                      // D^{-1}(r, c) at t[c * kSLd + r]
  const int b = blockIdx.x, lane = threadIdx.x;
  const int d0 = b * kSB;
  T x[kSB];
#pragma unroll
  for (int c = 0; c < kSB; ++c) x[c] = l_entry(A, lda, n, d0 + lane, d0 + c);
#pragma unroll
  for (int c = 0; c < kSB; ++c) d[c * kSB + lane] = x[c];
  wave_lds_sync();
#pragma unroll
  for (int r = 0; r < kSB; ++r) x[r] = r == lane ? T(1) : T(0);
#pragma unroll
  for (int k = 0; k < kSB - 1; ++k) {
#pragma unroll
    for (int r = k + 1; r < kSB; ++r) x[r] = fma(-d[k * kSB + r], x[k], x[r]);
    asm volatile("" ::: "memory");                 // a column's reads at a time
  }
#pragma unroll
  for (int r = 0; r < kSB; ++r) t[lane * kSLd + r] = x[r];
  wave_lds_sync();
  T* out = Dinv + (size_t)b * kSB * kSB;
#pragma unroll 4
  for (int cc = 0; cc < kSB; ++cc) out[cc * kSB + lane] = t[cc * kSLd + lane];
}

// Mf_b (blockIdx.y = 0) and Mb_b (1): 64 x 64 x 64 products on the matrix
// cores, wave w the rows 16w .. 16w+15.  (One lane per column with the inverse
// read by LDS broadcast took 91 us at n = 16384; 23 now.)
template <typename T>
__global__ void __launch_bounds__(kSThreads) solve_mmat_kernel(const T* A, int64_t lda, int n, int nblk,
                                                               const T* Dinv, T* Mf, T* Mb) {
  __shared__ T xa[kSB * kSLd];                     // X(r, j) at xa[j * kSLd + r]: D^{-1}, or its transpose
  __shared__ T lb[kSB * kSLd];                     // the tile's entry for (j, column) at lb[j * kSLd + column]
  const int b = blockIdx.x, tid = threadIdx.x;
  const bool fwd = blockIdx.y == 0;
  if (fwd ? b < 1 : b + 1 >= nblk) return;
  const int d0 = b * kSB, s0 = fwd ? d0 - kSB : d0 + kSB;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid & (kWave - 1);
  const size_t blk = (size_t)b * kSB * kSB;
  for (int c = wave; c < kSB; c += kSThreads / kWave) {
    const T x = Dinv[blk + c * kSB + lane];        // D^{-1}(lane, c)
    xa[fwd ? c * kSLd + lane : lane * kSLd + c] = x;
    // forward: column s0 + c of the tile's rows; backward: row s0 + lane, column d0 + c
    if (fwd) lb[lane * kSLd + c] = l_entry(A, lda, n, d0 + lane, s0 + c);
    else lb[c * kSLd + lane] = l_entry(A, lda, n, s0 + lane, d0 + c);
  }
  __syncthreads();
  typedef typename Mfma<T>::acc_t acc_t;
  acc_t acc[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) acc[t] = acc_t{T(0), T(0), T(0), T(0)};
  const int l16 = lane & 15, q = lane >> 4;
#pragma unroll
  for (int j = 0; j < kSB; j += 4) {
    const T x = xa[(j + q) * kSLd + 16 * wave + l16];
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = Mfma<T>::run(x, lb[(j + q) * kSLd + 16 * t + l16], acc[t]);
  }
  T* out = (fwd ? Mf : Mb) + blk;
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int v = 0; v < 4; ++v) out[(16 * t + l16) * kSB + 16 * wave + Mfma<T>::row(lane, v)] = acc[t][v];
}

// One wave polls entry `at` (per lane) of block sb for right-hand sides 0 ..
// NQ-1, reading the status word in the same round trip.  Blocks far from the
// one they wait for poll rarely (naps of 256 clocks), so that the next ones
// find the words' cache lines free.  Bounded: when the wait gives up (or an
// earlier wait already has) the status words are raised and the wave carries on
// with unspecified values, so that no wave leaves its workgroup's barriers.
template <typename T, int NQ>
__device__ __forceinline__ void wait_words(const SolveTriArgs& a, int sb, int at, int naps, T (&v)[NQ]) {
  const uint64_t* w = a.box + ((size_t)sb * kSolveGroup * kSB + at) * 2;
  const uint64_t t0 = wall_ticks();
  for (;;) {
    const int st = ld_coh(a.status);
    bool ok = true;
#pragma unroll
    for (int q = 0; q < NQ; ++q) ok = (q >= a.nr || box_get(w + (size_t)q * kSB * 2, a.stamp, v[q])) && ok;
    if (__ballot(!ok) == 0) return;
    if (__builtin_amdgcn_readfirstlane((st != 0 || wall_ticks() - t0 > kWaitLimitTicks) ? 1 : 0)) {
      if ((threadIdx.x & (kWave - 1)) == 0) raise_wait_status(a.status);
      return;
    }
    for (int i = 0; i < naps; ++i) __builtin_amdgcn_s_sleep(4);
  }
}

// 64 x 64 matrix times vector in one wave: m holds, for lane (p = lane/16, i =
// lane%16), X(16 e + i, 16 p + c) at m[(16 e + c) * 64 + lane]; v is lane k's
// entry k; lane r gets entry r of the product.  The vector reaches the FMAs
// through DPP row broadcasts (no LDS round trip for it), the four 16-lane rows
// sum a quarter of the columns each.
template <typename T>
__device__ __forceinline__ void load_mat(const T* m, int lane, T (&x)[kSB]) {
#pragma unroll
  for (int e = 0; e < kSB; ++e) x[e] = m[e * kWave + lane];
}
template <typename T>
__device__ __forceinline__ T mat_vec(const T (&x)[kSB], T v, int lane) {
  T s[4][4];
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int j = 0; j < 4; ++j) s[e][j] = T(0);
  refresh16<0>(s[0], v, x);
  refresh16<1>(s[1], v, x);
  refresh16<2>(s[2], v, x);
  refresh16<3>(s[3], v, x);
  T r = T(0);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const T sum = part_sum<4>((s[e][0] + s[e][1]) + (s[e][2] + s[e][3]));
    r = (lane >> 4) == e ? sum : r;
  }
  return r;
}

// Sums over the wave's 64 lanes of 16 values per lane: lane l with l % 16 == e
// gets, for e < 4, the sum of value e + 4 (l / 16 % 2) + 8 (l / 32).  Two
// exchange-and-add steps through the lane swaps halve the values and the
// lanes, then row rotations.
template <int CTRL>
__device__ __forceinline__ double ror_add(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, true);
  return v + __hiloint2double(hi, lo);
}
template <int CTRL>
__device__ __forceinline__ float ror_add(float v) {
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
// a's sum over the lane pairs in the even (lower) lanes, b's in the odd (upper)
template <int OFF>
__device__ __forceinline__ unsigned swap_halves(unsigned x, unsigned y, unsigned& other) {
  if constexpr (OFF == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(x, y, false, false);
    other = r[1];
    return r[0];
  } else {
    const auto r = __builtin_amdgcn_permlane32_swap(x, y, false, false);
    other = r[1];
    return r[0];
  }
}
template <int OFF>
__device__ __forceinline__ double pair_add(double a, double b) {
  unsigned lo1, hi1;
  const unsigned lo0 = swap_halves<OFF>((unsigned)__double2loint(a), (unsigned)__double2loint(b), lo1);
  const unsigned hi0 = swap_halves<OFF>((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), hi1);
  return __hiloint2double((int)hi0, (int)lo0) + __hiloint2double((int)hi1, (int)lo1);
}
template <int OFF>
__device__ __forceinline__ float pair_add(float a, float b) {
  unsigned o;
  const unsigned x = swap_halves<OFF>(__float_as_uint(a), __float_as_uint(b), o);
  return __uint_as_float(x) + __uint_as_float(o);
}
template <typename T>
__device__ __forceinline__ T lane_sums(const T (&v)[16], int lane) {
  T h[8], f[4];
#pragma unroll
  for (int c = 0; c < 8; ++c) h[c] = pair_add<32>(v[c], v[c + 8]);
#pragma unroll
  for (int c = 0; c < 4; ++c) f[c] = pair_add<16>(h[c], h[c + 4]);
  T r = T(0);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const T x = ror_add<0x121>(ror_add<0x122>(ror_add<0x124>(ror_add<0x128>(f[c]))));   // row_ror 8, 4, 2, 1
    r = (lane & 15) == c ? x : r;
  }
  return r;
}

// Forward (UPPER = false): z_b = D_b^{-1} r_b - Mf_b z_{b-1},
//   r_b = y_b - sum_{c<b-1} L_bc z_c.
// Backward (UPPER = true), blocks from the last one down:
//   u_b = D_b^{-T} r_b - Mb_b u_{b+1},  r_b = w_b - sum_{b'>b+1} L_{b'b}^T u_{b'}.
// The four waves of a workgroup take 16 columns each of the farther
// off-diagonal tiles of r_b and run through them without a barrier: every
// wave polls the solution words its tile needs straight into registers.
// Forward, a lane holds a row of the tile and the solution's entries reach the
// FMAs through DPP row broadcasts; backward, a lane holds a row as well (so
// that both directions read L's columns in runs), multiplies it by its own entry
// of the solution and keeps 16 sums, one per column, that meet once per block.
// Two tiles are in flight beside the two being used.  Then wave q takes
// right-hand side q alone: D_b^{-1} r_b, and, once the neighbouring block's
// solution arrives, M times it: the one product on the chain from block to
// block.  Bound by that chain, a block's words becoming visible and one 64 x 64
// product: one right-hand side at n = 16384 took 0.67 ms forward and 0.93 ms
// backward with a workgroup barrier or two per tile, the solution through
// LDS, eight right-hand-side slots always multiplied and the backward tiles
// read across columns; 0.35 and 0.41 now.
// Groups of four right-hand sides (blockIdx.y) are chains of their own, so they
// run side by side: MEASURED
template <typename T, bool UPPER, int NQ>
__global__ void __launch_bounds__(kSThreads, 1) solve_tri_kernel(SolveTriArgs a) {
  static_assert(NQ <= kSThreads / kWave && kSolveGroup <= kSThreads / kWave, "a wave solves one right-hand side");
  a.nr = min(a.nr - (int)blockIdx.y * kSolveGroup, NQ);
  a.Y = static_cast<T*>(a.Y) + (int64_t)blockIdx.y * kSolveGroup * a.ldy;
  a.box += (size_t)blockIdx.y * a.nblk * kSolveGroup * kSB * 2;
  extern __shared__ __align__(16) unsigned char smem[];
  T* dt = reinterpret_cast<T*>(smem);              // D_b^{-1} (forward) or D_b^{-T}, as load_mat reads it
  T* mt = dt + kSB * kSB;                          // Mf_b or Mb_b, likewise
  T* part = mt + kSB * kSB;                        // forward: [wave][NQ][64] partial sums; backward: [NQ][64] sums
  const T* A = static_cast<const T*>(a.A);
  T* Y = static_cast<T*>(a.Y);
  const T* Dinv = static_cast<const T*>(a.Dinv);
  const T* Mx = static_cast<const T*>(UPPER ? a.Mb : a.Mf);
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int g = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int i16 = lane & 15, p16 = lane >> 4;
  const int n = a.n, nr = a.nr, nblk = a.nblk;
  const int64_t lda = a.lda, ldy = a.ldy;
  for (int i = blockIdx.x; i < nblk; i += gridDim.x) {
    const int b = UPPER ? nblk - 1 - i : i;
    const int d0 = b * kSB;
    const int ntile = UPPER ? nblk - 1 - b : b;   // tiles of r_b and the chain's tile
    const int nfull = ntile > 1 ? ntile - 1 : 0;   // tiles the waves multiply
    // tile t multiplies the solution of block src(t): forward t, backward nblk-1-t
    auto src = [&](int t) { return UPPER ? nblk - 1 - t : t; };
    {
      T dv[16], mv[16];
      const size_t blk = (size_t)b * kSB * kSB;
#pragma unroll
      for (int c = 0; c < 16; ++c) {
        const int r = 16 * g + i16, k = 16 * p16 + c;
        dv[c] = Dinv[blk + (UPPER ? r * kSB + k : k * kSB + r)];
        mv[c] = ntile > 0 ? Mx[blk + k * kSB + r] : T(0);
      }
#pragma unroll
      for (int c = 0; c < 16; ++c) {
        dt[(16 * g + c) * kWave + lane] = dv[c];
        mt[(16 * g + c) * kWave + lane] = mv[c];
      }
    }
    const T ypre = (g < nr && d0 + lane < n) ? Y[(int64_t)(d0 + lane) + (int64_t)g * ldy] : T(0);
    // 16 columns of tile t, one row per lane: L(d0 + lane, s0 + 16g + c)
    // forward, L(s0 + lane, d0 + 16g + c) backward.  Rows past n read the last
    // row (forward such rows are never used, backward their solution is zero);
    // column 0 of L, e_0, is not stored: zeroed in the product.
    auto fetch = [&](int t, T(&x)[16]) {
      if (t >= nfull) return;
      const int s0 = src(t) * kSB;
      const int row = min((UPPER ? s0 : d0) + lane, n - 1), c0 = (UPPER ? d0 : s0) + 16 * g;
#pragma unroll
      for (int c = 0; c < 16; ++c) x[c] = A[(int64_t)row + (int64_t)max(c0 + c - 1, 0) * lda];
    };
    constexpr int NA = UPPER ? 16 : 4;
    T acc[NQ][NA];
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
      for (int c = 0; c < NA; ++c) acc[q][c] = T(0);
    auto use = [&](int t, T(&x)[16]) {
      if (t >= nfull) return;
      T v[NQ];
#pragma unroll
      for (int q = 0; q < NQ; ++q) v[q] = T(0);
      wait_words<T, NQ>(a, src(t), UPPER ? lane : 16 * g + i16, min(ntile - t, 32) - 3, v);
      if ((UPPER ? d0 : src(t) * kSB) + 16 * g == 0) x[0] = T(0);
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        if constexpr (UPPER) {
#pragma unroll
          for (int c = 0; c < 16; ++c) acc[q][c] = fma(x[c], v[q], acc[q][c]);
        } else {
          refresh16<0>(acc[q], v[q], x);
        }
      }
    };
    T r0[16], r1[16], r2[16], r3[16];
    fetch(0, r0);
    fetch(1, r1);
    for (int t = 0; t < nfull; t += 4) {
      fetch(t + 2, r2);
      fetch(t + 3, r3);
      use(t, r0);
      use(t + 1, r1);
      fetch(t + 4, r0);
      fetch(t + 5, r1);
      use(t + 2, r2);
      use(t + 3, r3);
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      if constexpr (UPPER) {
        const T x = lane_sums(acc[q], lane);
        if (i16 < 4) part[q * kSB + 16 * g + i16 + 4 * (p16 & 1) + 8 * (p16 >> 1)] = x;
      } else {
        part[(g * NQ + q) * kSB + lane] = (acc[q][0] + acc[q][1]) + (acc[q][2] + acc[q][3]);
      }
    }
    lds_barrier();
    if (g < nr) {                                  // wave q: right-hand side q
      T m[kSB];
      load_mat(dt, lane, m);
      T sum;
      if constexpr (UPPER) {
        sum = part[g * kSB + lane];
      } else {
        sum = T(0);
#pragma unroll
        for (int w = 0; w < kSThreads / kWave; ++w) sum += part[(w * NQ + g) * kSB + lane];
      }
      T x = mat_vec(m, d0 + lane < n ? ypre - sum : T(0), lane);
      if (ntile > 0) {
        load_mat(mt, lane, m);
        T near[1] = {T(0)};
        SolveTriArgs one = a;
        one.nr = 1;
        one.box += (size_t)g * kSB * 2;
        wait_words<T, 1>(one, src(ntile - 1), lane, 0, near);
        x -= mat_vec(m, near[0], lane);
      }
      if (d0 + lane < n) Y[(int64_t)(d0 + lane) + (int64_t)g * ldy] = x;
      box_put(&a.box[(((size_t)b * kSolveGroup + g) * kSB + lane) * 2], d0 + lane < n ? x : T(0), a.stamp);
    }
    lds_barrier();                                 // dt, mt and part are reused by the next block
  }
}

constexpr size_t solve_lds_bytes(int nq, size_t elem) { return (size_t)(2 * kSB * kSB + 4 * nq * kSB) * elem; }

// The substitution's workgroups wait on each other's blocks (bounded waits),
// so the grid never exceeds what the device holds at once; like the panels it
// is an ordinary launch unless ltlt_set_cooperative_panels(1) asks for the
// runtime's cooperative one.
template <typename T, bool UPPER, int NQ>
hipError_t launch_solve_tri_q(const SolveTriArgs& a, hipStream_t s) {
  const void* k = (const void*)solve_tri_kernel<T, UPPER, NQ>;
  const size_t lds = solve_lds_bytes(NQ, sizeof(T));
  hipError_t e = ensure_dynamic_lds(k, (int)lds);
  if (e != hipSuccess) return e;
  int dev = 0, per_cu = 0, cus = 0;
  if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
  if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
  if ((e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, kSThreads, lds)) != hipSuccess) return e;
  const int groups = (a.nr + NQ - 1) / NQ;         // NQ == kSolveGroup when there are two
  const int cap = per_cu * cus / groups;
  if (cap <= 0) return hipErrorInvalidValue;
  return launch_resident_grid(solve_tri_kernel<T, UPPER, NQ>, dim3((unsigned)(a.nblk < cap ? a.nblk : cap), groups),
                              kSThreads, lds, s, a);
}
template <typename T, bool UPPER>
hipError_t launch_solve_tri(const SolveTriArgs& a, hipStream_t s) {
  if (a.nr == 1) return launch_solve_tri_q<T, UPPER, 1>(a, s);
  if (a.nr == 2) return launch_solve_tri_q<T, UPPER, 2>(a, s);
  return launch_solve_tri_q<T, UPPER, kSolveGroup>(a, s);
}

// Stamps of the mailbox words: a process-wide counter that skips 0 (zeroed
// memory never validates).
unsigned next_stamp() {
  static std::atomic<unsigned> counter{0};
  unsigned v;
  do { v = counter.fetch_add(1) + 1; } while (v == 0);
  return v;
}

template <typename T>
hipError_t launch_solve(int n, const T* A, int64_t lda, const int* ipiv, int nrhs, T* B, int64_t ldb,
                        const SolveWork& w, hipStream_t s) {
  hipError_t e;
  {
    const int gb = (n + 255) / 256;
    hipLaunchKernelGGL(zero_ints_kernel, dim3((2 * n + 255) / 256), dim3(256), 0, s, w.cnt, 2 * n);
    hipLaunchKernelGGL(perm_count_kernel, dim3(gb), dim3(256), 0, s, n, ipiv, w.cnt);
    hipLaunchKernelGGL(perm_scan_kernel, dim3(1), dim3(1024), 0, s, n, w.cnt, w.off);
    hipLaunchKernelGGL(perm_scatter_kernel, dim3(gb), dim3(256), 0, s, n, ipiv, w.off, w.cnt + n, w.list);
    hipLaunchKernelGGL(perm_walk_kernel, dim3(gb), dim3(256), 0, s, n, ipiv, w.off, w.list, w.perm);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  T* alpha = static_cast<T*>(w.alpha);
  T* ralpha = static_cast<T*>(w.ralpha);
  T* Y = static_cast<T*>(w.Y);
  T* W = static_cast<T*>(w.W);
  hipLaunchKernelGGL(solve_alpha_kernel<T>, dim3((n + 255) / 256), dim3(256), 0, s, n, A, lda, alpha, ralpha);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const int nblk = (n + kSB - 1) / kSB;
  {
    // The solution words validate by the stamp of their launch, and stamps are
    // small integers: clear the words first, so that whatever an earlier call
    // left in this part of the workspace can never carry a current stamp.
    const int words = nblk * (nrhs > kSolveGroup ? kSolveRhs : kSolveGroup) * kSB * 2 * 2;   // as 32-bit halves
    hipLaunchKernelGGL(zero_ints_kernel, dim3((words + 255) / 256), dim3(256), 0, s, reinterpret_cast<int*>(w.box),
                       words);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  T* Dinv = static_cast<T*>(w.dinv);
  T* Mf = Dinv + (size_t)nblk * kSB * kSB;
  T* Mb = Mf + (size_t)nblk * kSB * kSB;
  hipLaunchKernelGGL(solve_dinv_kernel<T>, dim3(nblk), dim3(kWave), 0, s, A, lda, n, Dinv);
  hipLaunchKernelGGL(solve_mmat_kernel<T>, dim3(nblk, 2), dim3(kSThreads), 0, s, A, lda, n, nblk, Dinv, Mf, Mb);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  for (int q0 = 0; q0 < nrhs; q0 += kSolveRhs) {
    const int nr = nrhs - q0 < kSolveRhs ? nrhs - q0 : kSolveRhs;
    T* Bq = B + (int64_t)q0 * ldb;
    hipLaunchKernelGGL(solve_gather_kernel<T>, dim3((n + 255) / 256, nr), dim3(256), 0, s, n, nr, w.perm, Bq, ldb,
                       Y, w.ldy);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    SolveTriArgs ta{};
    ta.A = A; ta.lda = lda; ta.n = n; ta.nblk = nblk; ta.Y = Y; ta.ldy = w.ldy; ta.nr = nr;
    ta.box = w.box; ta.status = w.status; ta.Dinv = Dinv; ta.Mf = Mf; ta.Mb = Mb;
    ta.stamp = next_stamp();
    if ((e = launch_solve_tri<T, false>(ta, s)) != hipSuccess) return e;
    hipLaunchKernelGGL(solve_tridiag_kernel<T>, dim3(2 * nr), dim3(kTriWaves * kWave), 0, s, n, alpha, ralpha, Y, W,
                       w.ldy);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    ta.Y = W;
    ta.stamp = next_stamp();
    if ((e = launch_solve_tri<T, true>(ta, s)) != hipSuccess) return e;
    hipLaunchKernelGGL(solve_scatter_kernel<T>, dim3((n + 255) / 256, nr), dim3(256), 0, s, n, nr, w.perm, W, w.ldy,
                       Bq, ldb);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

template hipError_t launch_solve<double>(int, const double*, int64_t, const int*, int, double*, int64_t,
                                         const SolveWork&, hipStream_t);
template hipError_t launch_solve<float>(int, const float*, int64_t, const int*, int, float*, int64_t,
                                        const SolveWork&, hipStream_t);

}  // namespace ltlt

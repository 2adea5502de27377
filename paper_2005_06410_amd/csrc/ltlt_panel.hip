// Panel kernel: the column steps k = j .. j+bw-1 of one block of the pivoted
// skew-symmetric reduction P X P^T = L T L^T, run by P co-resident
// workgroups that together hold every row of the block (positions j+1..n-1).
//
// Thread layout: 512 threads (8 waves, two per SIMD) per workgroup, S lanes
// per row (S = 1, 2, 4 for blocks of up to 64, 128, 256 steps): the wave is
// split into S parts of 64/S consecutive lanes, part p holds the steps u with
// u % S == p of the same 64/S rows, so R = 512/S rows per workgroup and every
// 16-lane row of the wave belongs to one part.  A lane keeps its row's
// multipliers in registers: L[c] = multiplier of step j + c*S + p, c < 64.
//
// Rows never move between lanes.  Lane rows are the rows of the block-start
// matrix (block-start index `pos`, fixed); an exchange of positions k+1 and p
// only swaps the logical positions `lp` of the two lanes that hold them.  The
// row at position k+1 after the exchange is final from then on; the other one
// keeps its multipliers and column value where they are.
//
// What the other rows need of a row when it becomes the pivot -- its g
// coefficients, below, and its last two multipliers -- crosses workgroups
// through global memory, indexed by the block-start index; besides the
// exchange records it is the only data that does.  Two places:
//   * G, one row of TOT = 64 S values per row, g_u at group u / W, part u % S,
//     entry (u / S) % 4 with W = 4 S: the four values of a lane side by side, so
//     that a row is read with wide loads straight into the layout of the
//     refresh, and written once a group is full (every W steps);
//   * the tail, a ring of W entries (g_{s-1}, l_s) per row, one written at every
//     step, entry by entry over the rows, so that a wave's stores are one
//     contiguous run.  Writing both values to the row's place in G at every
//     step, a cache line per row, cost 10 of 97 ms at n = 16384.
//
// Column refresh.  The trailing matrix is stored as it was at block start
// (strict lower triangle), so the current column k is the stored column of
// the block-start index of position k, plus the not-yet-applied updates of
// steps j .. k-2.  Step s updates X(i,c) += l_i v_c - v_i l_c with v the
// column s+1 at step s, and v = alpha_{s+1} * L(:, s+2) below row s+2
// (column s+1 is the one step s+1 eliminates).  Summed over the block this is
// Lp Tx Lp^T with Tx skew tridiagonal, Tx[u,u+1] = alpha_{j+u+1}; the
// refresh of column k therefore needs only row k of Lp:
//   cv[i] = S(pos[i], pos[k]) + sum_{u<t} g_u Lp[u][i],
//   g_u = alpha_{j+u+1} Lrow[u+1] [u <= t-2] - alpha_{j+u} Lrow[u-1] [u >= 1],
//   Lrow[w] = Lp[w][k] (w <= t-2), Lrow[t-1] = 1 (unit diagonal of L),
// with S(a, b) = A(a, b) for a > b and -A(b, a) for a < b.
// Every row forms its own g as its multipliers appear: at step t, with l_t
// known, g_{t-1} = alpha_{j+t} l_t - alpha_{j+t-1} l_{t-2} is final.  A row that
// is the pivot of step t needs its last two multipliers as well, for the two
// coefficients that meet the unit diagonal of L: g_{t-1} = alpha_{j+t} -
// alpha_{j+t-1} l_{t-2} and g_t = -alpha_{j+t} l_{t-1}.  Wave 0, which learns the
// pivot first, fetches that row's values once for the workgroup, completes
// them and hands them out through LDS.  (Every wave gathering the multipliers
// for itself and forming g from LDS cost about 900 cycles a step, most of it
// LDS bandwidth, and every wave loading the finished g for itself kept the
// last wave as far behind the first at the CU's one address unit.)
// The g coefficients live in registers in "row broadcast" layout: register
// gr[k], lane l holds g of slot 4 (l % 16) + k of the lane's step slice, the
// same in each 16-lane row of that slice, and the refresh multiplies slot c
// by lane c / 4 of its own row through a DPP row broadcast, so no lane re-reads
// g from LDS.
//
// Exchange per step (one grid-wide round, no counters, no fences): every
// workgroup merges the candidates of its waves (one lane per wave) and the
// winning lane publishes the result as one record of two self-validating 64-bit words (each carries the step
// stamp); records sit 256 bytes apart.  Wave 0 of every workgroup polls all
// records until each carries the current stamp and reduces them (largest
// magnitude, then smallest position: the first maximum in position order), so
// all workgroups agree on the pivot p.  A barrier hands the result to the
// other waves, which load the next stored column (a strided row read for rows
// above the pivot, waited for only at the end of the refresh), form their
// multipliers and store what their rows may have to hand out; a second,
// LDS-only barrier hands them the pivot row's g.
// Values written to G at step k are read no earlier than step k+1; every wave
// waits for its own earlier stores to complete before the barrier that
// precedes the publication of the next record, so any record that validates
// implies that the winning row's values are visible.
//
// After the last step the carry column (column j+bw, refreshed) is formed and
// every lane writes its row of the block's outputs at its final position:
// Lx = [Lp, carry] (rows >= j+bw+1) feeds the trailing update as one
// rank-(bw+1) product with Bt = Lx Tx^T; the rows inside the block and the
// alphas are committed into A after that update.

//
// What bounds it: the step is one dependency chain (clock stamps, cycles, n =
// 16384 / n = 256): publish, poll and reduction of the records 3650 / 2640, the
// pivot row's values and the stored column 1000 / 600, everything local about
// 2300.  With the values handed out as above a step takes 3.6 -> 3.0 us at
// n = 16384 (factorization 97.4 -> 87.5 ms) and 2.9 -> 2.4 us at n = 2048
// (6.68 -> 5.57 ms), outputs bit-identical.

#include "ltlt_device.h"
#include "ltlt_exchange.h"
#include "ltlt_internal.h"

namespace ltlt {

int panel_rows(int bw) { return kPanelThreads / panel_split(bw); }
int panel_g_cols(int bw) { return KC * panel_split(bw); }
size_t panel_tail_elems(int bw, int64_t ldw) { return (size_t)(4 * panel_split(bw)) * 2 * (size_t)ldw; }

// Dynamic LDS: the pivot row's g, the block's alphas and pivots (TOT = steps a
// row can hold).
template <typename T>
size_t panel_lds_bytes(int bw, int /*R*/) {
  return (size_t)KC * panel_split(bw) * (2 * sizeof(T) + sizeof(int));
}

// Where step u of a row's g sits in its row of G.
template <int S>
__device__ __forceinline__ int g_at(int u) {
  return u / (4 * S) * (4 * S) + u % S * 4 + u / S % 4;
}
// Entry of the tail ring that step s writes (W = 4 S entries per row).
template <int S>
__device__ __forceinline__ int ring_at(int s) {
  return (s - 1) & (4 * S - 1);
}
// ONE: one workgroup holds every row (a.P == 1).
template <typename T, int S, bool ONE>
__global__ void __launch_bounds__(kPanelThreads, 1) panel_kernel(PanelArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int R = kPanelThreads / S;
  constexpr int RW = kWave / S;                    // rows per wave
  constexpr int W = 4 * S;                         // steps of a group of G (four per part)
  constexpr int TOT = KC * S;                      // steps a row can hold
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = tid / kWave;
  const int w = blockIdx.x;
  const int bw = a.bw, n = a.n, j = a.j;
  const int part = lane / RW;                      // step slice of this lane
  const int rloc = wave * RW + lane % RW;
  const int64_t lda = a.lda, ldw = a.ldw;
  const T* A = static_cast<const T*>(a.A);

  T* gl = reinterpret_cast<T*>(smem);              // the pivot row's g, as in its row of G
  T* alpha = gl + TOT;                             // alpha_{j+u}
  int* piv = reinterpret_cast<int*>(alpha + TOT);  // pivot position of step j+u
  __shared__ XRes s_x;                             // the agreement's result
  __shared__ Cand red[ONE ? 2 * kPanelWaves : kPanelWaves];

  if (ONE && ld_coh(a.status) != 0) return;        // the call has already failed
  const int row0 = j + 1 + w * R;                 // first block-start index held
  const int rows_here = max(0, min(R, n - row0));
  const bool my_row = rloc < rows_here;
  const int pos = row0 + rloc;                     // block-start index of this lane's row
  int lp = pos;                                    // its current position

  T L[KC], gr[4];
#pragma unroll
  for (int c = 0; c < KC; ++c) L[c] = T(0);
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) gr[kk] = T(0);
  T cv = T(0);
  T l1 = T(0), l2 = T(0), alph1 = T(0);            // multipliers of steps t-1, t-2; alpha_{j+t-1}
  const int posc = min(pos, n - 1);                // in range for lanes without a row too
  int64_t rowat = (int64_t)posc * lda;             // element (., posc)
  const int64_t at0 = (int64_t)(j + 1) + (int64_t)j * lda;
  // where this lane writes of its own row (gso: slots 4b .. 4b+3 of its part in
  // G; tso: the tail entry, part 0)
  constexpr unsigned TSZ = 2 * sizeof(T);
  const int b16 = lane & 15;
  const unsigned gso = (unsigned)((pos - (j + 1)) * TOT + part * 4) * (unsigned)sizeof(T);
  const unsigned tso = (unsigned)(pos - (j + 1)) * TSZ;
  const unsigned tstep = (unsigned)ldw * TSZ;      // bytes from one ring entry to the next
  const __amdgpu_buffer_rsrc_t grs =
      __builtin_amdgcn_make_buffer_rsrc(a.G, (short)0, (int)((unsigned)(n - 1 - j) * TOT * sizeof(T)), 0x00020000);
  const __amdgpu_buffer_rsrc_t trs = __builtin_amdgcn_make_buffer_rsrc(a.tail, (short)0, (int)(W * tstep), 0x00020000);
  T pg[4] = {T(0), T(0), T(0), T(0)};              // this part's g not yet in G
  // stored column value of this row (signed; zero past part 0).  First
  // column: index j, rows >= j+1 (lower part).
  T lvn = A[(int64_t)posc + (int64_t)j * lda];
  bool below = true;
  asm volatile("" : "+v"(lvn));                    // arrived: no wait for it inside the loop
  __syncthreads();

  for (int t = 0; t <= bw; ++t) {
    const int k = j + t;
    // ---- column refresh: cv = S(pos, q) + sum_u g_u L_u over rows at >= k+1 ----
    const bool active = my_row && lp >= k + 1;
    {
      T acc[4] = {T(0), T(0), T(0), T(0)};
      refresh_slots(acc, gr, L, (t + S - 1) / S);
      // the stored value, waited for only here (one part adds it)
      const T lv = part == 0 ? (below ? lvn : -lvn) : T(0);
      const T sum = part_sum<S>(lv + ((acc[0] + acc[1]) + (acc[2] + acc[3])));
      if (active) cv = sum;
    }
    if (t == bw) break;                           // carry column formed

    // ---- this wave's pivot candidate: (|cv|, position), first maximum; one
    //      lane per row, NaN is never a candidate ----
    Cand* wred = ONE ? red + (t & 1) * kPanelWaves : red;
    {
      const double m = (double)fabs(cv);
      wave_candidate(wred, wave, make_cand(active && part == 0 && m == m, m, cv < T(0), pos, lp));
    }
    // Wave 0 fetches what the column needs of the pivot row, for all waves, as
    // soon as it knows the row: g from G up to the last full group, the ring.
    constexpr int GL = (TOT * (int)sizeof(T) + 1023) / 1024;   // 16-byte loads per lane
    const int full = max(t - 1, 0) / W * W;        // steps whose g is in G
    u32x4 gq[GL];
    Pair<T> tq;
    auto fetch = [&](int row) {
      const unsigned r = (unsigned)(row - (j + 1));
#pragma unroll
      for (int q = 0; q < GL; ++q) {
        const unsigned off = (unsigned)(q * 1024 + lane * 16);
        gq[q] = buf_load16<ONE>(grs, off < (unsigned)(full * sizeof(T)) ? off : kSkip, r * (unsigned)(TOT * sizeof(T)));
      }
      tq = buf_load2<ONE>(T(0), trs, lane < W ? (unsigned)lane * tstep : kSkip, r * TSZ);
    };
    XRes xr;
    if constexpr (ONE) {
      xr = exchange_one(k, wave, lane, wred, fetch);
    } else {
      exchange_pivot(a, k + 1, k, wave, lane, w, red, s_x, fetch);
      xr = s_x;
    }
    const T alph = (T)xr.alpha;
    const int p = __builtin_amdgcn_readfirstlane(xr.p);
    const int posw = __builtin_amdgcn_readfirstlane(xr.posw);   // block-start index of the pivot row
    if (p < 0) return;

    // ---- the next stored column S(pos, posw) = +A(pos, posw) below the
    //      diagonal, -A(posw, pos) above; waited for in its refresh.  The lanes
    //      of the pivot row itself (and lanes without a row, standing in for the
    //      last one) read the block's first entry: never the diagonal, which may
    //      not be the caller's memory ----
    int64_t at1 = (int64_t)posw * lda + posc, at2 = rowat + posw;
    asm volatile("" : "+v"(at1), "+v"(at2));       // both formed, one selected: no branch
    below = pos > posw;
    const int64_t at = below ? at1 : at2;
    lvn = A[posc == posw ? at0 : at];
    __builtin_amdgcn_sched_barrier(0);             // keep the loads ahead of the work below

    // ---- exchange positions k+1 and p (logical only); multiplier of step k;
    //      into its slot; this row's g_{t-1} ----
    lp = lp == p ? k + 1 : (lp == k + 1 ? p : lp);
    const bool next = my_row && lp >= k + 2;      // rows still to be eliminated
    T l = cv / alph;
    l = next && alph != T(0) ? l : T(0);
    set_slot(L, t / S, part == t % S, l);
    if (tid == 0) {
      alpha[t] = alph;
      piv[t] = p;
    }
    const T gown = fma(-alph1, l2, alph * l);
    const int u = max(t - 1, 0);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) pg[kk] = (u % S == part && (u / S) % 4 == kk) ? gown : pg[kk];
    buf_store2<ONE>(gown, l, trs, next && part == 0 ? tso : kSkip, (unsigned)ring_at<S>(t) * tstep);
    if (u % W == W - 1) {                          // a full group: this part's four values
      const unsigned to = next ? gso : kSkip, at = (unsigned)(u / W) * (unsigned)(W * sizeof(T));
      buf_store2<ONE>(pg[0], pg[1], grs, to, at);
      buf_store2<ONE>(pg[2], pg[3], grs, to + 2 * (unsigned)sizeof(T), at);
    }

    // ---- g of the next column, through LDS: from G, from the ring, zeros past
    //      it, then the two coefficients that meet the unit diagonal of L.
    //      One wave's LDS writes take effect in their order. ----
    if (wave == 0) {
#pragma unroll
      for (int q = 0; q < GL; ++q) put16(gl, (q * kWave + lane) * (16 / (int)sizeof(T)), TOT, gq[q]);
      if (lane < W) gl[full + (lane % S) * 4 + lane / S] = full + lane < t - 1 ? tq.a : T(0);
      if (lane == ring_at<S>(t - 2) && t >= 1) gl[g_at<S>(t - 1)] = fma(-alph1, t < 2 ? T(0) : tq.b, alph);
      if (lane == ring_at<S>(t - 1)) gl[g_at<S>(t)] = t < 1 ? T(0) : -alph * tq.b;
    }
    lds_barrier();
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) gr[kk] = gl[(b16 * S + part) * 4 + kk];
    l2 = l1;
    l1 = l;
    alph1 = alph;
  }
  __syncthreads();                                 // the alphas and pivots in LDS

  // ---- outputs, by final position, straight from registers.  Rows at
  //      positions j+1 .. j+bw hold the multipliers of the steps before they
  //      became final (zeros after); trailing rows hold all of them and the
  //      carry. ----
  T* PO = static_cast<T*>(a.PO);
  T* Bm = static_cast<T*>(a.Bm);
  const int tr0 = j + bw + 1;                      // first trailing position
  const bool trailing = my_row && lp >= tr0;
  const T carry = trailing ? cv : T(0);
  if (my_row) {
    const int64_t ro = lp - (j + 1);
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      const int u = c * S + part;
      if (u < bw) PO[ro + (int64_t)u * ldw] = L[c];
    }
    if (part == 0) PO[ro + (int64_t)bw * ldw] = carry;
  }
  // Bt = Lx Tx^T: column u = a_u Lx_{u+1} - a_{u-1} Lx_{u-1},
  // a_u = alpha_{j+u+1} (u <= bw-2), a_{bw-1} = 1, Lx_bw = carry.
  // Step u = c*S + part; step u+1 lives in the next part (lane + RW), slot c
  // (slot c+1 when this is the last part), step u-1 in the previous part
  // (lane - RW), slot c (slot c-1 when this is part 0).  The owner lane hands
  // out the slot its requester needs.
  const int up_src = (lane + RW) % kWave, dn_src = (lane + kWave - RW) % kWave;
#pragma unroll
  for (int c = 0; c < KC; ++c) {
    const T give_up = (part == 0 && c + 1 < KC) ? L[c + 1 < KC ? c + 1 : c] : (part == 0 ? T(0) : L[c]);
    const T give_dn = (part == S - 1) ? (c >= 1 ? L[c >= 1 ? c - 1 : 0] : T(0)) : L[c];
    const T xp0 = S == 1 ? give_up : __shfl(give_up, up_src, kWave);
    const T xm = S == 1 ? give_dn : __shfl(give_dn, dn_src, kWave);
    const int u = c * S + part;
    if (trailing && u <= bw) {
      T v = T(0);
      if (u <= bw - 1) {
        const T au = (u <= bw - 2) ? alpha[u + 1] : T(1);
        v += au * (u + 1 == bw ? carry : xp0);
      }
      if (u >= 1) {
        const T am = (u - 1 <= bw - 2) ? alpha[u] : T(1);
        v -= am * xm;
      }
      Bm[(int64_t)(lp - tr0) + (int64_t)u * ldw] = v;
    }
  }
  // column bw when it lies past the slots (bw == TOT): -Lx_{bw-1}, step TOT-1
  // is slot KC-1 of the last part
  {
    const T last = __shfl(L[KC - 1], (lane % RW) + (S - 1) * RW, kWave);
    if (trailing && bw == TOT && part == 0) Bm[(int64_t)(lp - tr0) + (int64_t)bw * ldw] = -last;
  }
  if (my_row && part == 0) a.perm[lp] = pos;
  if (w == 0 && wave == 0) {
    T* al = static_cast<T*>(a.alpha);
    for (int u = lane; u < bw; u += kWave) {
      al[u] = alpha[u];
      a.ipiv[j + u + 1] = piv[u];
    }
  }
}

template <typename T, int S>
hipError_t launch_panel_s(const PanelArgs& a, size_t lds, hipStream_t st) {
  if (a.P == 1) return launch_resident_grid(panel_kernel<T, S, true>, 1u, kPanelThreads, lds, st, a);
  return launch_resident_grid(panel_kernel<T, S, false>, (unsigned)a.P, kPanelThreads, lds, st, a);
}

template <typename T>
hipError_t launch_panel(const PanelArgs& a, size_t lds, hipStream_t st) {
  if (a.P > kMaxPanelRecords || a.P > a.nrec || a.R != panel_rows(a.bw)) return hipErrorInvalidValue;
  switch (panel_split(a.bw)) {
    case 1: return launch_panel_s<T, 1>(a, lds, st);
    case 2: return launch_panel_s<T, 2>(a, lds, st);
    case 4: return launch_panel_s<T, 4>(a, lds, st);
    default: return hipErrorInvalidValue;
  }
}

template <typename T, int S>
int panel_max_blocks_s(size_t lds) {
  int dev = 0, per_cu = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)panel_kernel<T, S, false>, kPanelThreads, lds) !=
      hipSuccess)
    return 0;
  return per_cu * cus;
}

// Co-resident workgroups for a block of width bw (capped by the records one
// poll covers).
template <typename T>
int panel_max_blocks(int bw, size_t lds) {
  int cap;
  switch (panel_split(bw)) {
    case 1: cap = panel_max_blocks_s<T, 1>(lds); break;
    case 2: cap = panel_max_blocks_s<T, 2>(lds); break;
    case 4: cap = panel_max_blocks_s<T, 4>(lds); break;
    default: return 0;
  }
  return cap < kMaxPanelRecords ? cap : kMaxPanelRecords;
}

// Exchange records start with stamps that can never validate: word B stamp 0,
// and word A epoch opposite to that of the first stamp using the slot
// (slot 1 first holds s = 1, epoch 0; slot 0 first holds s = 2, epoch 1).
__global__ void rec_init_kernel(uint64_t* rec, int nrec) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= 2 * kRecStride * nrec) return;
  const int slot = i / (kRecStride * nrec);
  const int word = i % kRecStride;
  rec[i] = (word == 0 && slot == 1) ? (1ull << 63) : 0ull;
}

hipError_t launch_rec_init(uint64_t* rec, int nrec_per_slot, hipStream_t s) {
  const int tot = 2 * kRecStride * nrec_per_slot;
  hipLaunchKernelGGL(rec_init_kernel, dim3((tot + 255) / 256), dim3(256), 0, s, rec, nrec_per_slot);
  return hipGetLastError();
}

template int panel_max_blocks<double>(int, size_t);
template int panel_max_blocks<float>(int, size_t);
template size_t panel_lds_bytes<double>(int, int);
template size_t panel_lds_bytes<float>(int, int);
template hipError_t launch_panel<double>(const PanelArgs&, size_t, hipStream_t);
template hipError_t launch_panel<float>(const PanelArgs&, size_t, hipStream_t);

}  // namespace ltlt

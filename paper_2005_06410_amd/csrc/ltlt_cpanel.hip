// Complex panel kernel: the column steps k = j .. j+bw-1 of one block of the
// pivoted reduction P X P^T = L T L^T of a complex skew-symmetric X
// (X^T = -X, a transpose without conjugation), held as two real planes.
//
// The algorithm, thread layout, exchange and output order are those of the
// real panel (ltlt_panel.hip); what changes:
//  * a lane keeps KCC = 32 complex multipliers of its row (real and
//    imaginary parts in registers, 128 VGPRs in fp64, as the real panel's 64
//    real slots), so S = 1, 2, 4 lanes share a row for blocks of up to 32,
//    64, 128 steps;
//  * the refresh cv = S(pos, q) + sum_u g_u L_u takes four DPP row-broadcast
//    FMA passes per 16 slots: Re += gr Lr + (-gi) Li, Im += gr Li + gi Lr;
//  * the pivot search compares |re| + |im| (the magnitude of the BLAS complex
//    i_amax); the exchange record carries that magnitude, so the pivot value
//    itself goes through a per-row slot V[idx - j - 1] that each wave's
//    candidate lane writes before its workgroup publishes, and every wave
//    loads the winner's V right after the agreement (a validated record
//    implies the slot is visible, as for G and the tail);
//  * G and the tail hold complex values: groups of W = 2 S steps (two per
//    part), tail entries (g_{s-1}, l_s).  Handing the pivot row's g out like
//    the real panel took n = 1501 complex128 from 7.17 to 6.69 ms, n = 9000 from
//    65.2 to 62.2 ms and n = 128 (one workgroup) from 486 to 355 us;
//  * multipliers l = cv / alpha by Smith's quotient;
//  * outputs: LL = [Lr | Li | Lr] and the two right operands
//    BtA = [Btr | -Bti], BtB = [Btr | Bti] (Bt = Lx Tx^T), so that each
//    plane's trailing update is one real product of depth 2(bw+1).

#include "ltlt_device.h"
#include "ltlt_exchange.h"
#include "ltlt_internal.h"

namespace ltlt {

constexpr int KCC = 32;                          // complex multiplier slots per lane

inline int cpanel_split(int bw) { return bw <= KCC ? 1 : (bw <= 2 * KCC ? 2 : 4); }
int cpanel_rows(int bw) { return kPanelThreads / cpanel_split(bw); }

int cpanel_g_cols(int bw) { return 2 * KCC * cpanel_split(bw); }
size_t cpanel_tail_elems(int bw, int64_t ldw) { return (size_t)(2 * cpanel_split(bw)) * 4 * (size_t)ldw; }

// Dynamic LDS: the pivot row's g, the block's alphas (complex) and pivots.
template <typename T>
size_t cpanel_lds_bytes(int bw) {
  return (size_t)KCC * cpanel_split(bw) * (4 * sizeof(T) + sizeof(int));
}

// Smith's quotient x / y (y != 0).
template <typename T>
__device__ __forceinline__ void cdiv(T xr, T xi, T yr, T yi, T& zr, T& zi) {
  if (fabs(yr) >= fabs(yi)) {
    const T r = yi / yr, den = yr + yi * r;
    zr = (xr + xi * r) / den;
    zi = (xi - xr * r) / den;
  } else {
    const T r = yr / yi, den = yi + yr * r;
    zr = (xr * r + xi) / den;
    zi = (xi * r - xr) / den;
  }
}

// The 16 slots c = 16 K .. 16 K + 15 of the refresh, four passes: ar += gr Lr, ar +=
// (-gi) Li, ai += gr Li, ai += gi Lr; slot c takes g register c % 2 of lane c / 2
// of its 16-lane row (DPP row broadcast) and sum c % 4.  Only the first eight of
// each pass when no more are in use (c < nslots; the others hold zeros).
#define LTLT_CF(OP, acc, g, l, b) OP " %[" #acc "], %[" #g "], %[" #l "] row_newbcast:" b " row_mask:0xf bank_mask:0xf\n"
#define LTLT_CFMAS(OP, B0, B1, B2, B3, B4, B5, B6, B7) \
  LTLT_CF(OP, ar0, re0, r0, B0) LTLT_CF(OP, ar1, re1, r1, B0) \
  LTLT_CF(OP, ar2, re0, r2, B1) LTLT_CF(OP, ar3, re1, r3, B1) \
  LTLT_CF(OP, ar0, re0, r4, B2) LTLT_CF(OP, ar1, re1, r5, B2) \
  LTLT_CF(OP, ar2, re0, r6, B3) LTLT_CF(OP, ar3, re1, r7, B3) \
  "s_cbranch_scc1 LTLT_carre%=\n" \
  LTLT_CF(OP, ar0, re0, r8, B4) LTLT_CF(OP, ar1, re1, r9, B4) \
  LTLT_CF(OP, ar2, re0, r10, B5) LTLT_CF(OP, ar3, re1, r11, B5) \
  LTLT_CF(OP, ar0, re0, r12, B6) LTLT_CF(OP, ar1, re1, r13, B6) \
  LTLT_CF(OP, ar2, re0, r14, B7) LTLT_CF(OP, ar3, re1, r15, B7) \
  "LTLT_carre%=:\n" \
  LTLT_CF(OP, ar0, ni0, i0, B0) LTLT_CF(OP, ar1, ni1, i1, B0) \
  LTLT_CF(OP, ar2, ni0, i2, B1) LTLT_CF(OP, ar3, ni1, i3, B1) \
  LTLT_CF(OP, ar0, ni0, i4, B2) LTLT_CF(OP, ar1, ni1, i5, B2) \
  LTLT_CF(OP, ar2, ni0, i6, B3) LTLT_CF(OP, ar3, ni1, i7, B3) \
  "s_cbranch_scc1 LTLT_carni%=\n" \
  LTLT_CF(OP, ar0, ni0, i8, B4) LTLT_CF(OP, ar1, ni1, i9, B4) \
  LTLT_CF(OP, ar2, ni0, i10, B5) LTLT_CF(OP, ar3, ni1, i11, B5) \
  LTLT_CF(OP, ar0, ni0, i12, B6) LTLT_CF(OP, ar1, ni1, i13, B6) \
  LTLT_CF(OP, ar2, ni0, i14, B7) LTLT_CF(OP, ar3, ni1, i15, B7) \
  "LTLT_carni%=:\n" \
  LTLT_CF(OP, ai0, re0, i0, B0) LTLT_CF(OP, ai1, re1, i1, B0) \
  LTLT_CF(OP, ai2, re0, i2, B1) LTLT_CF(OP, ai3, re1, i3, B1) \
  LTLT_CF(OP, ai0, re0, i4, B2) LTLT_CF(OP, ai1, re1, i5, B2) \
  LTLT_CF(OP, ai2, re0, i6, B3) LTLT_CF(OP, ai3, re1, i7, B3) \
  "s_cbranch_scc1 LTLT_caire%=\n" \
  LTLT_CF(OP, ai0, re0, i8, B4) LTLT_CF(OP, ai1, re1, i9, B4) \
  LTLT_CF(OP, ai2, re0, i10, B5) LTLT_CF(OP, ai3, re1, i11, B5) \
  LTLT_CF(OP, ai0, re0, i12, B6) LTLT_CF(OP, ai1, re1, i13, B6) \
  LTLT_CF(OP, ai2, re0, i14, B7) LTLT_CF(OP, ai3, re1, i15, B7) \
  "LTLT_caire%=:\n" \
  LTLT_CF(OP, ai0, im0, r0, B0) LTLT_CF(OP, ai1, im1, r1, B0) \
  LTLT_CF(OP, ai2, im0, r2, B1) LTLT_CF(OP, ai3, im1, r3, B1) \
  LTLT_CF(OP, ai0, im0, r4, B2) LTLT_CF(OP, ai1, im1, r5, B2) \
  LTLT_CF(OP, ai2, im0, r6, B3) LTLT_CF(OP, ai3, im1, r7, B3) \
  "s_cbranch_scc1 LTLT_caiim%=\n" \
  LTLT_CF(OP, ai0, im0, r8, B4) LTLT_CF(OP, ai1, im1, r9, B4) \
  LTLT_CF(OP, ai2, im0, r10, B5) LTLT_CF(OP, ai3, im1, r11, B5) \
  LTLT_CF(OP, ai0, im0, r12, B6) LTLT_CF(OP, ai1, im1, r13, B6) \
  LTLT_CF(OP, ai2, im0, r14, B7) LTLT_CF(OP, ai3, im1, r15, B7) \
  "LTLT_caiim%=:\n"
#define LTLT_CREFRESH(OP, HALF, ...) \
  asm volatile("s_nop 1\ns_cmp_le_i32 %[ns], " HALF "\n" LTLT_CFMAS(OP, __VA_ARGS__) \
               : [ar0] "+v"(ar[0]), [ar1] "+v"(ar[1]), [ar2] "+v"(ar[2]), [ar3] "+v"(ar[3]), [ai0] "+v"(ai[0]), \
                 [ai1] "+v"(ai[1]), [ai2] "+v"(ai[2]), [ai3] "+v"(ai[3]) \
               : [ns] "s"(nslots), [re0] "v"(gre[0]), [re1] "v"(gre[1]), [im0] "v"(gim[0]), [im1] "v"(gim[1]), \
                 [ni0] "v"(gni[0]), [ni1] "v"(gni[1]), \
                 [r0] "v"(Lr[16 * K + 0]), [i0] "v"(Li[16 * K + 0]), [r1] "v"(Lr[16 * K + 1]), [i1] "v"(Li[16 * K + 1]), \
                 [r2] "v"(Lr[16 * K + 2]), [i2] "v"(Li[16 * K + 2]), [r3] "v"(Lr[16 * K + 3]), [i3] "v"(Li[16 * K + 3]), \
                 [r4] "v"(Lr[16 * K + 4]), [i4] "v"(Li[16 * K + 4]), [r5] "v"(Lr[16 * K + 5]), [i5] "v"(Li[16 * K + 5]), \
                 [r6] "v"(Lr[16 * K + 6]), [i6] "v"(Li[16 * K + 6]), [r7] "v"(Lr[16 * K + 7]), [i7] "v"(Li[16 * K + 7]), \
                 [r8] "v"(Lr[16 * K + 8]), [i8] "v"(Li[16 * K + 8]), [r9] "v"(Lr[16 * K + 9]), [i9] "v"(Li[16 * K + 9]), \
                 [r10] "v"(Lr[16 * K + 10]), [i10] "v"(Li[16 * K + 10]), [r11] "v"(Lr[16 * K + 11]), [i11] "v"(Li[16 * K + 11]), \
                 [r12] "v"(Lr[16 * K + 12]), [i12] "v"(Li[16 * K + 12]), [r13] "v"(Lr[16 * K + 13]), [i13] "v"(Li[16 * K + 13]), \
                 [r14] "v"(Lr[16 * K + 14]), [i14] "v"(Li[16 * K + 14]), [r15] "v"(Lr[16 * K + 15]), [i15] "v"(Li[16 * K + 15]) \
               : "scc")
#define LTLT_CREFRESH_FN(T, OP) \
  template <int K> \
  __device__ __forceinline__ void crefresh(T (&ar)[4], T (&ai)[4], const T (&gre)[2], const T (&gim)[2], \
                                           const T (&gni)[2], const T (&Lr)[KCC], const T (&Li)[KCC], int nslots) { \
    if constexpr (K == 0) LTLT_CREFRESH(OP, "8", "0", "1", "2", "3", "4", "5", "6", "7"); \
    else LTLT_CREFRESH(OP, "24", "8", "9", "10", "11", "12", "13", "14", "15"); \
  }
LTLT_CREFRESH_FN(double, "v_fmac_f64_dpp")
LTLT_CREFRESH_FN(float, "v_fmac_f32_dpp")
#undef LTLT_CREFRESH_FN
#undef LTLT_CREFRESH
#undef LTLT_CFMAS
#undef LTLT_CF

// Lr[c] = vr, Li[c] = vi in the lanes of `on`, for a wave-uniform slot 0 <= c <
// 32, by a jump straight to the slot's moves (16 bytes an entry, the first one
// 12 bytes past the address s_getpc returns).
#define LTLT_CM(OP, c) OP " %[r" #c "], %[vr]\n" OP " %[i" #c "], %[vi]\ns_branch LTLT_cs%=\ns_nop 0\n"
#define LTLT_CMOVS(OP) \
  LTLT_CM(OP, 0) LTLT_CM(OP, 1) LTLT_CM(OP, 2) LTLT_CM(OP, 3) \
  LTLT_CM(OP, 4) LTLT_CM(OP, 5) LTLT_CM(OP, 6) LTLT_CM(OP, 7) \
  LTLT_CM(OP, 8) LTLT_CM(OP, 9) LTLT_CM(OP, 10) LTLT_CM(OP, 11) \
  LTLT_CM(OP, 12) LTLT_CM(OP, 13) LTLT_CM(OP, 14) LTLT_CM(OP, 15) \
  LTLT_CM(OP, 16) LTLT_CM(OP, 17) LTLT_CM(OP, 18) LTLT_CM(OP, 19) \
  LTLT_CM(OP, 20) LTLT_CM(OP, 21) LTLT_CM(OP, 22) LTLT_CM(OP, 23) \
  LTLT_CM(OP, 24) LTLT_CM(OP, 25) LTLT_CM(OP, 26) LTLT_CM(OP, 27) \
  LTLT_CM(OP, 28) LTLT_CM(OP, 29) LTLT_CM(OP, 30) LTLT_CM(OP, 31)
#define LTLT_CSET(OP) \
  uint64_t keep; \
  asm volatile("s_and_saveexec_b64 %[keep], %[on]\n" \
               "s_getpc_b64 vcc\n" \
               "s_add_u32 vcc_lo, vcc_lo, %[off]\n" \
               "s_addc_u32 vcc_hi, vcc_hi, 0\n" \
               "s_setpc_b64 vcc\n" LTLT_CMOVS(OP) \
               "LTLT_cs%=:\n" \
               "s_mov_b64 exec, %[keep]\n" \
               : [keep] "=&s"(keep), \
                 [r0] "+v"(Lr[0]), [i0] "+v"(Li[0]), [r1] "+v"(Lr[1]), [i1] "+v"(Li[1]), \
                 [r2] "+v"(Lr[2]), [i2] "+v"(Li[2]), [r3] "+v"(Lr[3]), [i3] "+v"(Li[3]), \
                 [r4] "+v"(Lr[4]), [i4] "+v"(Li[4]), [r5] "+v"(Lr[5]), [i5] "+v"(Li[5]), \
                 [r6] "+v"(Lr[6]), [i6] "+v"(Li[6]), [r7] "+v"(Lr[7]), [i7] "+v"(Li[7]), \
                 [r8] "+v"(Lr[8]), [i8] "+v"(Li[8]), [r9] "+v"(Lr[9]), [i9] "+v"(Li[9]), \
                 [r10] "+v"(Lr[10]), [i10] "+v"(Li[10]), [r11] "+v"(Lr[11]), [i11] "+v"(Li[11]), \
                 [r12] "+v"(Lr[12]), [i12] "+v"(Li[12]), [r13] "+v"(Lr[13]), [i13] "+v"(Li[13]), \
                 [r14] "+v"(Lr[14]), [i14] "+v"(Li[14]), [r15] "+v"(Lr[15]), [i15] "+v"(Li[15]), \
                 [r16] "+v"(Lr[16]), [i16] "+v"(Li[16]), [r17] "+v"(Lr[17]), [i17] "+v"(Li[17]), \
                 [r18] "+v"(Lr[18]), [i18] "+v"(Li[18]), [r19] "+v"(Lr[19]), [i19] "+v"(Li[19]), \
                 [r20] "+v"(Lr[20]), [i20] "+v"(Li[20]), [r21] "+v"(Lr[21]), [i21] "+v"(Li[21]), \
                 [r22] "+v"(Lr[22]), [i22] "+v"(Li[22]), [r23] "+v"(Lr[23]), [i23] "+v"(Li[23]), \
                 [r24] "+v"(Lr[24]), [i24] "+v"(Li[24]), [r25] "+v"(Lr[25]), [i25] "+v"(Li[25]), \
                 [r26] "+v"(Lr[26]), [i26] "+v"(Li[26]), [r27] "+v"(Lr[27]), [i27] "+v"(Li[27]), \
                 [r28] "+v"(Lr[28]), [i28] "+v"(Li[28]), [r29] "+v"(Lr[29]), [i29] "+v"(Li[29]), \
                 [r30] "+v"(Lr[30]), [i30] "+v"(Li[30]), [r31] "+v"(Lr[31]), [i31] "+v"(Li[31]) \
               : [off] "s"(12 + 16 * c), [on] "s"(mask), [vr] "v"(vr), [vi] "v"(vi) \
               : "vcc", "scc")
__device__ __forceinline__ void cset_slot(double (&Lr)[KCC], double (&Li)[KCC], int c, bool on, double vr, double vi) {
  static_assert(KCC == 32, "32 slots");
  const uint64_t mask = __ballot(on);
  LTLT_CSET("v_mov_b64_e32");
}
__device__ __forceinline__ void cset_slot(float (&Lr)[KCC], float (&Li)[KCC], int c, bool on, float vr, float vi) {
  const uint64_t mask = __ballot(on);
  LTLT_CSET("v_mov_b32_e32");
}
#undef LTLT_CSET
#undef LTLT_CMOVS
#undef LTLT_CM

// Where step u of a row's g sits in its row of G (in complex values): the two
// of a lane side by side, W = 2 S steps a group.
template <int S>
__device__ __forceinline__ int cg_at(int u) {
  return u / (2 * S) * (2 * S) + u % S * 2 + u / S % 2;
}
// Entry of the tail ring that step s writes.
template <int S>
__device__ __forceinline__ int cring_at(int s) {
  return (s - 1) & (2 * S - 1);
}

// ONE: one workgroup holds every row (P == 1).
template <typename T, int S, bool ONE>
__global__ void __launch_bounds__(kPanelThreads, 1) cpanel_kernel(CPanelArgs ca) {
  extern __shared__ __align__(16) unsigned char smem[];
  const PanelArgs& a = ca.b;
  constexpr int R = kPanelThreads / S;
  constexpr int RW = kWave / S;                    // rows per wave
  constexpr int TOT = KCC * S;                     // steps a row can hold
  constexpr int W = 2 * S;                         // steps of a group of G (two per part)
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = tid / kWave;
  const int w = blockIdx.x;
  const int bw = a.bw, n = a.n, j = a.j;
  const int part = lane / RW;
  const int rloc = wave * RW + lane % RW;
  const int64_t lda = a.lda, ldw = a.ldw;
  const T* Ar = static_cast<const T*>(a.A);
  const T* Ai = static_cast<const T*>(ca.Ai);
  T* Vr = static_cast<T*>(ca.Vr);
  T* Vi = static_cast<T*>(ca.Vi);

  T* gl = reinterpret_cast<T*>(smem);              // the pivot row's g (re, im), as in its row of G
  T* my_ar = gl + 2 * TOT;                         // alpha_{j+u}
  T* my_ai = my_ar + TOT;
  int* piv = reinterpret_cast<int*>(my_ai + TOT);  // pivot position of step j+u
  __shared__ XRes s_x;                             // alpha NaN: no finite candidate at this step
  __shared__ Cand red[ONE ? 2 * kPanelWaves : kPanelWaves];
  if (ONE && ld_coh(a.status) != 0) return;        // the call has already failed

  const int row0 = j + 1 + w * R;
  const int rows_here = max(0, min(R, n - row0));
  const bool my_row = rloc < rows_here;
  const int pos = row0 + rloc;
  int lp = pos;

  T Lr[KCC], Li[KCC], gre[2], gim[2], gni[2];
#pragma unroll
  for (int c = 0; c < KCC; ++c) { Lr[c] = T(0); Li[c] = T(0); }
#pragma unroll
  for (int k = 0; k < 2; ++k) { gre[k] = T(0); gim[k] = T(0); gni[k] = T(0); }
  T cvr = T(0), cvi = T(0);
  T l1r = T(0), l1i = T(0), l2r = T(0), l2i = T(0), alr1 = T(0), ali1 = T(0);   // steps t-1, t-2
  const int posc = min(pos, n - 1);                // in range for lanes without a row too
  int64_t rowat = (int64_t)posc * lda;             // element (., posc)
  constexpr unsigned TSZ = 4 * sizeof(T);
  const int b16 = lane & 15;
  const unsigned gso = (unsigned)((pos - (j + 1)) * 2 * TOT + part * 4) * (unsigned)sizeof(T);
  const unsigned tso = (unsigned)(pos - (j + 1)) * TSZ;
  const unsigned tstep = (unsigned)ldw * TSZ;      // bytes from one ring entry to the next
  const __amdgpu_buffer_rsrc_t grs =
      __builtin_amdgcn_make_buffer_rsrc(a.G, (short)0, (int)((unsigned)(n - 1 - j) * 2 * TOT * sizeof(T)), 0x00020000);
  const __amdgpu_buffer_rsrc_t trs = __builtin_amdgcn_make_buffer_rsrc(a.tail, (short)0, (int)(W * tstep), 0x00020000);
  T pg[4] = {T(0), T(0), T(0), T(0)};              // this part's g (re, im, re, im) not yet in G
  T lvrn = Ar[(int64_t)posc + (int64_t)j * lda], lvin = Ai[(int64_t)posc + (int64_t)j * lda];
  bool below = true;
  asm volatile("" : "+v"(lvrn), "+v"(lvin));       // arrived: no wait for it inside the loop
  __syncthreads();

  for (int t = 0; t <= bw; ++t) {
    const int k = j + t;
    const bool active = my_row && lp >= k + 1;
    {
      T ar[4] = {T(0), T(0), T(0), T(0)}, ai[4] = {T(0), T(0), T(0), T(0)};
      const int nslots = (t + S - 1) / S;
      if (nslots > 0) crefresh<0>(ar, ai, gre, gim, gni, Lr, Li, nslots);
      if (nslots > 16) crefresh<1>(ar, ai, gre, gim, gni, Lr, Li, nslots);
      // the stored value, waited for only here (one part adds it)
      const T lvr = part == 0 ? (below ? lvrn : -lvrn) : T(0), lvi = part == 0 ? (below ? lvin : -lvin) : T(0);
      const T sr = part_sum<S>(lvr + ((ar[0] + ar[1]) + (ar[2] + ar[3])));
      const T si = part_sum<S>(lvi + ((ai[0] + ai[1]) + (ai[2] + ai[3])));
      if (active) { cvr = sr; cvi = si; }
    }
    if (t == bw) break;

    // ---- this wave's candidate: (|re| + |im|, position), first maximum; the
    //      candidate lane leaves its value in V for the agreement ----
    Cand* wred = ONE ? red + (t & 1) * kPanelWaves : red;
    {
      const double m = (double)(fabs(cvr) + fabs(cvi));
      const Cand c = make_cand(active && part == 0 && m == m, m, false, pos, lp);
      if (first_max_lane<false>(c, true)) {
        wred[wave] = c;
        if (cand_lp(c) != (unsigned)kIdxNone) {
          st_coh_t(&Vr[pos - (j + 1)], cvr);
          st_coh_t(&Vi[pos - (j + 1)], cvi);
        }
      }
    }
    // Wave 0 fetches the pivot row's g and ring for all waves as soon as it
    // knows the row.
    constexpr int GL = (2 * TOT * (int)sizeof(T) + 1023) / 1024;   // 16-byte loads per lane
    const int full = max(t - 1, 0) / W * W;        // steps whose g is in G
    u32x4 gq[GL];
    T tq[4];
    auto fetch = [&](int row) {
      const unsigned r = (unsigned)(row - (j + 1));
#pragma unroll
      for (int q = 0; q < GL; ++q) {
        const unsigned off = (unsigned)(q * 1024 + lane * 16);
        gq[q] = buf_load16<ONE>(grs, off < (unsigned)(full * 2 * sizeof(T)) ? off : kSkip,
                                r * (unsigned)(2 * TOT * sizeof(T)));
      }
      buf_load4<ONE>(tq, trs, lane < W ? (unsigned)lane * tstep : kSkip, r * TSZ);
    };
    XRes xr;
    if constexpr (ONE) {
      xr = exchange_one(k, wave, lane, wred, fetch);
    } else {
      exchange_pivot(a, k + 1, k, wave, lane, w, red, s_x, fetch);
      xr = s_x;
    }
    const int p = __builtin_amdgcn_readfirstlane(xr.p);
    const int posw = __builtin_amdgcn_readfirstlane(xr.posw);
    const bool none = xr.alpha != xr.alpha;
    if (p < 0) return;

    // ---- the pivot value, then the next stored column, waited for in its
    //      refresh (every lane loads, so the waits count exactly) ----
    T alr = ld_coh_t(&Vr[posw - (j + 1)]), ali = ld_coh_t(&Vi[posw - (j + 1)]);
    int64_t at1 = (int64_t)posw * lda + posc, at2 = rowat + posw;
    asm volatile("" : "+v"(at1), "+v"(at2));       // both formed, one selected: no branch
    below = pos > posw;
    lvrn = Ar[below ? at1 : at2];
    lvin = Ai[below ? at1 : at2];
    __builtin_amdgcn_sched_barrier(0);             // keep the loads ahead of the work below

    // ---- exchange positions k+1 and p (logical only); multiplier of step k
    //      into its slot; this row's g_{t-1} ----
    lp = lp == p ? k + 1 : (lp == k + 1 ? p : lp);
    const bool next = my_row && lp >= k + 2;
    alr = none ? T(NAN) : alr;
    ali = none ? T(NAN) : ali;
    T lr = T(0), li = T(0);
    cdiv(cvr, cvi, alr, ali, lr, li);
    const bool div = next && (alr != T(0) || ali != T(0));
    lr = div ? lr : T(0);
    li = div ? li : T(0);
    cset_slot(Lr, Li, t / S, part == t % S, lr, li);
    if (tid == 0) {
      my_ar[t] = alr; my_ai[t] = ali;
      piv[t] = p;
    }
    T gr = alr * lr - ali * li, gi = alr * li + ali * lr;
    if (t >= 2) { gr -= alr1 * l2r - ali1 * l2i; gi -= alr1 * l2i + ali1 * l2r; }
    const int u = max(t - 1, 0);
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      const bool mine = u % S == part && (u / S) % 2 == kk;
      pg[2 * kk] = mine ? gr : pg[2 * kk];
      pg[2 * kk + 1] = mine ? gi : pg[2 * kk + 1];
    }
    buf_store4<ONE>(gr, gi, lr, li, trs, next && part == 0 ? tso : kSkip, (unsigned)cring_at<S>(t) * tstep);
    if (u % W == W - 1)                            // a full group: this part's two values
      buf_store4<ONE>(pg[0], pg[1], pg[2], pg[3], grs, next ? gso : kSkip,
                      (unsigned)(u / W) * (unsigned)(2 * W * sizeof(T)));

    // ---- g of the next column, through LDS: from G, from the ring, zeros past
    //      it, then the two coefficients that meet the unit diagonal of L:
    //      g_u = alpha_{u+1} Lrow[u+1] [u <= t-1] - alpha_u Lrow[u-1] [u >= 1].
    //      One wave's LDS writes take effect in their order. ----
    if (wave == 0) {
#pragma unroll
      for (int q = 0; q < GL; ++q) put16(gl, (q * kWave + lane) * (16 / (int)sizeof(T)), 2 * TOT, gq[q]);
      if (lane < W) {
        const bool has = full + lane < t - 1;
        const int at = 2 * (full + (lane % S) * 2 + lane / S);
        gl[at] = has ? tq[0] : T(0);
        gl[at + 1] = has ? tq[1] : T(0);
      }
      if (lane == cring_at<S>(t - 2) && t >= 1) {
        T hr = alr, hi = ali;
        if (t >= 2) { hr -= alr1 * tq[2] - ali1 * tq[3]; hi -= alr1 * tq[3] + ali1 * tq[2]; }
        const int at = 2 * cg_at<S>(t - 1);
        gl[at] = hr;
        gl[at + 1] = hi;
      }
      if (lane == cring_at<S>(t - 1)) {
        T hr = T(0), hi = T(0);
        if (t >= 1) { hr -= alr * tq[2] - ali * tq[3]; hi -= alr * tq[3] + ali * tq[2]; }
        const int at = 2 * cg_at<S>(t);
        gl[at] = hr;
        gl[at + 1] = hi;
      }
    }
    lds_barrier();
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      gre[kk] = gl[(b16 * S + part) * 4 + 2 * kk];
      gim[kk] = gl[(b16 * S + part) * 4 + 2 * kk + 1];
      gni[kk] = -gim[kk];
    }
    l2r = l1r; l2i = l1i;
    l1r = lr; l1i = li;
    alr1 = alr; ali1 = ali;
  }
  __syncthreads();                                 // the alphas and pivots in LDS

  // ---- outputs by final position, straight from registers ----
  const int K = bw + 1;
  T* LLr = static_cast<T*>(ca.LL);
  T* LLi = LLr + (int64_t)K * ldw;
  T* LLr2 = LLi + (int64_t)K * ldw;
  T* BAr = static_cast<T*>(ca.BtA);                // Btr
  T* BAi = BAr + (int64_t)K * ldw;                 // -Bti
  T* BBr = static_cast<T*>(ca.BtB);                // Btr
  T* BBi = BBr + (int64_t)K * ldw;                 // Bti
  const int tr0 = j + bw + 1;
  const bool trailing = my_row && lp >= tr0;
  const T carr = trailing ? cvr : T(0), cari = trailing ? cvi : T(0);
  if (my_row) {
    const int64_t ro = lp - (j + 1);
#pragma unroll
    for (int c = 0; c < KCC; ++c) {
      const int u = c * S + part;
      if (u < bw) {
        LLr[ro + (int64_t)u * ldw] = Lr[c];
        LLi[ro + (int64_t)u * ldw] = Li[c];
        LLr2[ro + (int64_t)u * ldw] = Lr[c];
      }
    }
    if (part == 0) {
      LLr[ro + (int64_t)bw * ldw] = carr;
      LLi[ro + (int64_t)bw * ldw] = cari;
      LLr2[ro + (int64_t)bw * ldw] = carr;
    }
  }
  // Bt = Lx Tx^T: column u = a_u Lx_{u+1} - a_{u-1} Lx_{u-1},
  // a_u = alpha_{j+u+1} (u <= bw-2), a_{bw-1} = 1, Lx_bw = carry; the
  // neighbouring steps come from the neighbouring parts as in the real panel.
  const int up_src = (lane + RW) % kWave, dn_src = (lane + kWave - RW) % kWave;
#pragma unroll
  for (int c = 0; c < KCC; ++c) {
    const int cu = c + 1 < KCC ? c + 1 : c, cd = c >= 1 ? c - 1 : 0;
    const T gur = (part == 0 && c + 1 < KCC) ? Lr[cu] : (part == 0 ? T(0) : Lr[c]);
    const T gui = (part == 0 && c + 1 < KCC) ? Li[cu] : (part == 0 ? T(0) : Li[c]);
    const T gdr = (part == S - 1) ? (c >= 1 ? Lr[cd] : T(0)) : Lr[c];
    const T gdi = (part == S - 1) ? (c >= 1 ? Li[cd] : T(0)) : Li[c];
    const T xpr = S == 1 ? gur : __shfl(gur, up_src, kWave);
    const T xpi = S == 1 ? gui : __shfl(gui, up_src, kWave);
    const T xmr = S == 1 ? gdr : __shfl(gdr, dn_src, kWave);
    const T xmi = S == 1 ? gdi : __shfl(gdi, dn_src, kWave);
    const int u = c * S + part;
    if (trailing && u <= bw) {
      T vr = T(0), vi = T(0);
      if (u <= bw - 1) {
        const bool last = u + 1 == bw;
        const T br = last ? carr : xpr, bi = last ? cari : xpi;
        if (u <= bw - 2) {
          const T aur = my_ar[u + 1], aui = my_ai[u + 1];
          vr += aur * br - aui * bi;
          vi += aur * bi + aui * br;
        } else {
          vr += br;
          vi += bi;
        }
      }
      if (u >= 1) {
        if (u - 1 <= bw - 2) {
          const T amr = my_ar[u], ami = my_ai[u];
          vr -= amr * xmr - ami * xmi;
          vi -= amr * xmi + ami * xmr;
        } else {
          vr -= xmr;
          vi -= xmi;
        }
      }
      const int64_t at = (int64_t)(lp - tr0) + (int64_t)u * ldw;
      BAr[at] = vr;
      BAi[at] = -vi;
      BBr[at] = vr;
      BBi[at] = vi;
    }
  }
  // column bw when it lies past the slots (bw == TOT): -Lx_{bw-1}
  {
    const int src = (lane % RW) + (S - 1) * RW;
    const T lr_last = __shfl(Lr[KCC - 1], src, kWave);
    const T li_last = __shfl(Li[KCC - 1], src, kWave);
    if (trailing && bw == TOT && part == 0) {
      const int64_t at = (int64_t)(lp - tr0) + (int64_t)bw * ldw;
      BAr[at] = -lr_last;
      BAi[at] = li_last;
      BBr[at] = -lr_last;
      BBi[at] = -li_last;
    }
  }
  if (my_row && part == 0) a.perm[lp] = pos;
  if (w == 0 && wave == 0) {
    T* alr_out = static_cast<T*>(a.alpha);
    T* ali_out = static_cast<T*>(ca.alpha_i);
    for (int u = lane; u < bw; u += kWave) {
      alr_out[u] = my_ar[u];
      ali_out[u] = my_ai[u];
      a.ipiv[j + u + 1] = piv[u];
    }
  }
}

template <typename T, int S>
hipError_t launch_cpanel_s(const CPanelArgs& a, size_t lds, hipStream_t st) {
  if (a.b.P == 1) return launch_resident_grid(cpanel_kernel<T, S, true>, 1u, kPanelThreads, lds, st, a);
  return launch_resident_grid(cpanel_kernel<T, S, false>, (unsigned)a.b.P, kPanelThreads, lds, st, a);
}

template <typename T>
hipError_t launch_cpanel(const CPanelArgs& a, size_t lds, hipStream_t st) {
  if (a.b.P > kMaxPanelRecords || a.b.P > a.b.nrec || a.b.R != cpanel_rows(a.b.bw) || a.b.bw > 4 * KCC)
    return hipErrorInvalidValue;
  switch (cpanel_split(a.b.bw)) {
    case 1: return launch_cpanel_s<T, 1>(a, lds, st);
    case 2: return launch_cpanel_s<T, 2>(a, lds, st);
    case 4: return launch_cpanel_s<T, 4>(a, lds, st);
    default: return hipErrorInvalidValue;
  }
}

template <typename T, int S>
int cpanel_max_blocks_s(size_t lds) {
  int dev = 0, per_cu = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)cpanel_kernel<T, S, false>, kPanelThreads, lds) !=
      hipSuccess)
    return 0;
  return per_cu * cus;
}

template <typename T>
int cpanel_max_blocks(int bw, size_t lds) {
  int cap;
  switch (cpanel_split(bw)) {
    case 1: cap = cpanel_max_blocks_s<T, 1>(lds); break;
    case 2: cap = cpanel_max_blocks_s<T, 2>(lds); break;
    case 4: cap = cpanel_max_blocks_s<T, 4>(lds); break;
    default: return 0;
  }
  return cap < kMaxPanelRecords ? cap : kMaxPanelRecords;
}

// ---------------------------------------------------------------------------
// Interleaved complex <-> two real planes, strict lower triangle only.  One
// workgroup per column (grid-stride over columns), rows across the threads.
template <typename T>
__global__ void __launch_bounds__(256) cplx_split_kernel(int n, const T* A, int64_t lda, T* Pr, T* Pi, int64_t ldp) {
  for (int c = blockIdx.x; c < n; c += gridDim.x) {
    const T* col = A + 2 * (int64_t)c * lda;
    for (int i = c + 1 + threadIdx.x; i < n; i += blockDim.x) {
      const T re = col[2 * (int64_t)i], im = col[2 * (int64_t)i + 1];
      Pr[(int64_t)i + (int64_t)c * ldp] = re;
      Pi[(int64_t)i + (int64_t)c * ldp] = im;
    }
  }
}

template <typename T>
__global__ void __launch_bounds__(256) cplx_merge_kernel(int n, T* A, int64_t lda, const T* Pr, const T* Pi,
                                                         int64_t ldp) {
  for (int c = blockIdx.x; c < n; c += gridDim.x) {
    T* col = A + 2 * (int64_t)c * lda;
    for (int i = c + 1 + threadIdx.x; i < n; i += blockDim.x) {
      col[2 * (int64_t)i] = Pr[(int64_t)i + (int64_t)c * ldp];
      col[2 * (int64_t)i + 1] = Pi[(int64_t)i + (int64_t)c * ldp];
    }
  }
}

template <typename T>
hipError_t launch_cplx_split(int n, const void* A, int64_t lda, T* Pr, T* Pi, int64_t ldp, hipStream_t s) {
  if (n <= 1) return hipSuccess;
  const int g = n < 4096 ? n : 4096;
  hipLaunchKernelGGL(cplx_split_kernel<T>, dim3(g), dim3(256), 0, s, n, static_cast<const T*>(A), lda, Pr, Pi, ldp);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_cplx_merge(int n, void* A, int64_t lda, const T* Pr, const T* Pi, int64_t ldp, hipStream_t s) {
  if (n <= 1) return hipSuccess;
  const int g = n < 4096 ? n : 4096;
  hipLaunchKernelGGL(cplx_merge_kernel<T>, dim3(g), dim3(256), 0, s, n, static_cast<T*>(A), lda, Pr, Pi, ldp);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Complex Pfaffian from the (interleaved) factors: log|Pf| = sum_j log|alpha_{2j}| (fp64,
// |z| by hypot) and the phase Pf/|Pf| = det(P) prod_j (-alpha_{2j})/|alpha_{2j}|,
// both by one fixed-order tree reduction (sums of logs, products of unit
// complex numbers).
// A raised abort flag (status[0]) gives log|Pf| = NaN and phase 0.
template <typename T>
__global__ void __launch_bounds__(1024) cpfaffian_kernel(int n, const T* A, int64_t lda, const int* ipiv,
                                                         double* logabs, double* phase, const int* status) {
  __shared__ double s_log[1024], s_pr[1024], s_pi[1024];
  __shared__ int s_zero[1024];
  const int tid = threadIdx.x;
  double lg = 0.0, pr = 1.0, pi = 0.0;
  int zero = 0, neg = 0;
  const int half = n / 2;
  if ((n & 1) == 0) {
    for (int jj = tid; jj < half; jj += 1024) {
      const int64_t at = 2 * ((int64_t)(2 * jj + 1) + (int64_t)(2 * jj) * lda);   // (re, im) pairs
      const double ar = (double)A[at], ai = (double)A[at + 1];
      const double mag = hypot(ar, ai);
      if (mag == 0.0) zero = 1;
      else {
        lg += log(mag);
        const double ur = -ar / mag, ui = -ai / mag;   // factor T(2j,2j+1) = -alpha_{2j}
        const double tr = pr * ur - pi * ui;
        pi = pr * ui + pi * ur;
        pr = tr;
      }
    }
    for (int i = tid; i < n; i += 1024)
      if (ipiv[i] != i) neg ^= 1;
    if (neg) { pr = -pr; pi = -pi; }
  }
  s_log[tid] = lg; s_pr[tid] = pr; s_pi[tid] = pi; s_zero[tid] = zero;
  __syncthreads();
  for (int st = 512; st >= 1; st >>= 1) {
    if (tid < st) {
      s_log[tid] += s_log[tid + st];
      const double ar = s_pr[tid], ai = s_pi[tid], br = s_pr[tid + st], bi = s_pi[tid + st];
      s_pr[tid] = ar * br - ai * bi;
      s_pi[tid] = ar * bi + ai * br;
      s_zero[tid] |= s_zero[tid + st];
    }
    __syncthreads();
  }
  if (tid == 0) {
    if (status[0] != 0) { *logabs = NAN; phase[0] = 0.0; phase[1] = 0.0; }
    else if ((n & 1) || s_zero[0]) { *logabs = -INFINITY; phase[0] = 0.0; phase[1] = 0.0; }
    else {
      // renormalise the product of unit factors (rounding drift only)
      const double m = hypot(s_pr[0], s_pi[0]);
      *logabs = s_log[0];
      phase[0] = s_pr[0] / m;
      phase[1] = s_pi[0] / m;
    }
  }
}

template <typename T>
hipError_t launch_cpfaffian(int n, const void* A, int64_t lda, const int* ipiv, double* logabs, double* phase,
                            const int* status, hipStream_t s) {
  hipLaunchKernelGGL(cpfaffian_kernel<T>, dim3(1), dim3(1024), 0, s, n, static_cast<const T*>(A), lda, ipiv, logabs,
                     phase, status);
  return hipGetLastError();
}

#define LTLT_CINST(T)                                                                                        \
  template size_t cpanel_lds_bytes<T>(int);                                                                 \
  template int cpanel_max_blocks<T>(int, size_t);                                                           \
  template hipError_t launch_cpanel<T>(const CPanelArgs&, size_t, hipStream_t);                             \
  template hipError_t launch_cplx_split<T>(int, const void*, int64_t, T*, T*, int64_t, hipStream_t);        \
  template hipError_t launch_cplx_merge<T>(int, void*, int64_t, const T*, const T*, int64_t, hipStream_t);  \
  template hipError_t launch_cpfaffian<T>(int, const void*, int64_t, const int*, double*, double*, const int*,  \
                                          hipStream_t);
LTLT_CINST(double)
LTLT_CINST(float)
#undef LTLT_CINST

}  // namespace ltlt

// Exchange machinery shared by the panel kernels: the per-step pivot
// agreement between the co-resident workgroups of a panel (records, poll,
// reduction), the register-slot helpers and the part sums of a row.
#pragma once

#include "ltlt_device.h"
#include "ltlt_internal.h"

namespace ltlt {

constexpr int kPollPerLane = kMaxPanelRecords / kWave;   // records per polling lane
constexpr int KC = 64;                                   // multiplier slots per lane

// Lanes per row and register slots per lane for a block of width bw.
inline int panel_split(int bw) { return bw <= KC ? 1 : (bw <= 2 * KC ? 2 : 4); }

// A pivot candidate on its way from lanes to waves to workgroups:
//   v = bits(|cv|) (a non-negative double)
//   w = (sign(cv) << 42) | (pos << 21) | lp;  lp = kIdxNone: no candidate, v = 0
// Record words.  s is the step stamp (1 <= s < 2^21; it grows by one per
// exchange, so consecutive exchanges use alternate record slots).
//   word A = v | epoch(s) << 63,   epoch(s) = (s >> 1) & 1
//   word B = (s << 43) | w
// A record slot alternates with s & 1 and every record location is written at
// every step of its slot, so a slot holds stamp s or s-2 and the epoch bit
// alone tells them apart in word A; word B carries the full stamp.
constexpr uint64_t kIdxNone = 0x1FFFFFull;
struct __align__(16) Cand {
  uint64_t v, w;
};
__device__ __forceinline__ Cand make_cand(bool on, double absv, bool neg, int pos, int lp) {
  Cand c;
  c.v = on ? (uint64_t)__double_as_longlong(absv) : 0ull;
  c.w = on ? ((uint64_t)(((unsigned)neg << 10) | ((unsigned)pos >> 11)) << 32) | (((unsigned)pos << 21) | (unsigned)lp) : kIdxNone;
  return c;
}
__device__ __forceinline__ unsigned cand_lp(const Cand& c) { return (unsigned)c.w & (unsigned)kIdxNone; }
__device__ __forceinline__ uint64_t rec_epoch(int s) { return (uint64_t)((s >> 1) & 1) << 63; }
__device__ __forceinline__ bool rec_valid(uint64_t a, uint64_t b, int s) {
  return (int)(a >> 63) == ((s >> 1) & 1) && (int)(b >> 43) == s;
}
__device__ __forceinline__ uint64_t ld_coh64(const uint64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_coh64(uint64_t* p, uint64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void st_coh_t(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ T ld_coh_t(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// LDS written by some lanes of a wave is read by other lanes of the same wave:
// wait for the wave's LDS operations and keep the compiler from moving memory
// accesses across this point.
__device__ __forceinline__ void wave_lds_sync() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// acc[c % 4] += g[c % 4](lane (lane & ~15) + c / 4) * L[c] for the slots c <
// nslots (wave-uniform, 0 <= nslots <= 64; up to the next multiple of 8, where
// the slots hold zeros), oldest first, through v_fmac with a DPP row broadcast
// (row_newbcast, gfx950).  One asm block with its own exits: groups of 16 behind
// branches that the compiler lays out cost a jump out and back each.  It is led
// by the two wait states a DPP read needs after a vector write of its source.
#define LTLT_SLOT_FMA(OP, c, k, b) \
  OP " %[a" #k "], %[g" #k "], %[l" #c "] row_newbcast:" #b " row_mask:0xf bank_mask:0xf\n"
#define LTLT_SLOT_END(c) "s_cmp_le_i32 %[ns], " #c "\ns_cbranch_scc1 LTLT_fma%=\n"
#define LTLT_SLOT_FMAS(OP) \
  LTLT_SLOT_FMA(OP, 0, 0, 0) LTLT_SLOT_FMA(OP, 1, 1, 0) LTLT_SLOT_FMA(OP, 2, 2, 0) LTLT_SLOT_FMA(OP, 3, 3, 0) \
  LTLT_SLOT_FMA(OP, 4, 0, 1) LTLT_SLOT_FMA(OP, 5, 1, 1) LTLT_SLOT_FMA(OP, 6, 2, 1) LTLT_SLOT_FMA(OP, 7, 3, 1) \
  LTLT_SLOT_END(8) \
  LTLT_SLOT_FMA(OP, 8, 0, 2) LTLT_SLOT_FMA(OP, 9, 1, 2) LTLT_SLOT_FMA(OP, 10, 2, 2) LTLT_SLOT_FMA(OP, 11, 3, 2) \
  LTLT_SLOT_FMA(OP, 12, 0, 3) LTLT_SLOT_FMA(OP, 13, 1, 3) LTLT_SLOT_FMA(OP, 14, 2, 3) LTLT_SLOT_FMA(OP, 15, 3, 3) \
  LTLT_SLOT_END(16) \
  LTLT_SLOT_FMA(OP, 16, 0, 4) LTLT_SLOT_FMA(OP, 17, 1, 4) LTLT_SLOT_FMA(OP, 18, 2, 4) LTLT_SLOT_FMA(OP, 19, 3, 4) \
  LTLT_SLOT_FMA(OP, 20, 0, 5) LTLT_SLOT_FMA(OP, 21, 1, 5) LTLT_SLOT_FMA(OP, 22, 2, 5) LTLT_SLOT_FMA(OP, 23, 3, 5) \
  LTLT_SLOT_END(24) \
  LTLT_SLOT_FMA(OP, 24, 0, 6) LTLT_SLOT_FMA(OP, 25, 1, 6) LTLT_SLOT_FMA(OP, 26, 2, 6) LTLT_SLOT_FMA(OP, 27, 3, 6) \
  LTLT_SLOT_FMA(OP, 28, 0, 7) LTLT_SLOT_FMA(OP, 29, 1, 7) LTLT_SLOT_FMA(OP, 30, 2, 7) LTLT_SLOT_FMA(OP, 31, 3, 7) \
  LTLT_SLOT_END(32) \
  LTLT_SLOT_FMA(OP, 32, 0, 8) LTLT_SLOT_FMA(OP, 33, 1, 8) LTLT_SLOT_FMA(OP, 34, 2, 8) LTLT_SLOT_FMA(OP, 35, 3, 8) \
  LTLT_SLOT_FMA(OP, 36, 0, 9) LTLT_SLOT_FMA(OP, 37, 1, 9) LTLT_SLOT_FMA(OP, 38, 2, 9) LTLT_SLOT_FMA(OP, 39, 3, 9) \
  LTLT_SLOT_END(40) \
  LTLT_SLOT_FMA(OP, 40, 0, 10) LTLT_SLOT_FMA(OP, 41, 1, 10) LTLT_SLOT_FMA(OP, 42, 2, 10) LTLT_SLOT_FMA(OP, 43, 3, 10) \
  LTLT_SLOT_FMA(OP, 44, 0, 11) LTLT_SLOT_FMA(OP, 45, 1, 11) LTLT_SLOT_FMA(OP, 46, 2, 11) LTLT_SLOT_FMA(OP, 47, 3, 11) \
  LTLT_SLOT_END(48) \
  LTLT_SLOT_FMA(OP, 48, 0, 12) LTLT_SLOT_FMA(OP, 49, 1, 12) LTLT_SLOT_FMA(OP, 50, 2, 12) LTLT_SLOT_FMA(OP, 51, 3, 12) \
  LTLT_SLOT_FMA(OP, 52, 0, 13) LTLT_SLOT_FMA(OP, 53, 1, 13) LTLT_SLOT_FMA(OP, 54, 2, 13) LTLT_SLOT_FMA(OP, 55, 3, 13) \
  LTLT_SLOT_END(56) \
  LTLT_SLOT_FMA(OP, 56, 0, 14) LTLT_SLOT_FMA(OP, 57, 1, 14) LTLT_SLOT_FMA(OP, 58, 2, 14) LTLT_SLOT_FMA(OP, 59, 3, 14) \
  LTLT_SLOT_FMA(OP, 60, 0, 15) LTLT_SLOT_FMA(OP, 61, 1, 15) LTLT_SLOT_FMA(OP, 62, 2, 15) LTLT_SLOT_FMA(OP, 63, 3, 15)
#define LTLT_REFRESH(OP) \
  asm volatile("s_nop 1\n" LTLT_SLOT_END(0) LTLT_SLOT_FMAS(OP) \
               "LTLT_fma%=:\n" \
               : [a0] "+v"(acc[0]), [a1] "+v"(acc[1]), [a2] "+v"(acc[2]), [a3] "+v"(acc[3]) \
               : [ns] "s"(nslots), [g0] "v"(g[0]), [g1] "v"(g[1]), [g2] "v"(g[2]), [g3] "v"(g[3]), \
                 [l0] "v"(L[0]), [l1] "v"(L[1]), [l2] "v"(L[2]), [l3] "v"(L[3]), \
                 [l4] "v"(L[4]), [l5] "v"(L[5]), [l6] "v"(L[6]), [l7] "v"(L[7]), \
                 [l8] "v"(L[8]), [l9] "v"(L[9]), [l10] "v"(L[10]), [l11] "v"(L[11]), \
                 [l12] "v"(L[12]), [l13] "v"(L[13]), [l14] "v"(L[14]), [l15] "v"(L[15]), \
                 [l16] "v"(L[16]), [l17] "v"(L[17]), [l18] "v"(L[18]), [l19] "v"(L[19]), \
                 [l20] "v"(L[20]), [l21] "v"(L[21]), [l22] "v"(L[22]), [l23] "v"(L[23]), \
                 [l24] "v"(L[24]), [l25] "v"(L[25]), [l26] "v"(L[26]), [l27] "v"(L[27]), \
                 [l28] "v"(L[28]), [l29] "v"(L[29]), [l30] "v"(L[30]), [l31] "v"(L[31]), \
                 [l32] "v"(L[32]), [l33] "v"(L[33]), [l34] "v"(L[34]), [l35] "v"(L[35]), \
                 [l36] "v"(L[36]), [l37] "v"(L[37]), [l38] "v"(L[38]), [l39] "v"(L[39]), \
                 [l40] "v"(L[40]), [l41] "v"(L[41]), [l42] "v"(L[42]), [l43] "v"(L[43]), \
                 [l44] "v"(L[44]), [l45] "v"(L[45]), [l46] "v"(L[46]), [l47] "v"(L[47]), \
                 [l48] "v"(L[48]), [l49] "v"(L[49]), [l50] "v"(L[50]), [l51] "v"(L[51]), \
                 [l52] "v"(L[52]), [l53] "v"(L[53]), [l54] "v"(L[54]), [l55] "v"(L[55]), \
                 [l56] "v"(L[56]), [l57] "v"(L[57]), [l58] "v"(L[58]), [l59] "v"(L[59]), \
                 [l60] "v"(L[60]), [l61] "v"(L[61]), [l62] "v"(L[62]), [l63] "v"(L[63]) \
               : "scc")
__device__ __forceinline__ void refresh_slots(double (&acc)[4], const double (&g)[4], const double (&L)[KC],
                                              int nslots) {
  static_assert(KC == 64, "64 slots");
  LTLT_REFRESH("v_fmac_f64_dpp");
}
__device__ __forceinline__ void refresh_slots(float (&acc)[4], const float (&g)[4], const float (&L)[KC], int nslots) {
  LTLT_REFRESH("v_fmac_f32_dpp");
}
#undef LTLT_REFRESH
#undef LTLT_SLOT_FMAS
#undef LTLT_SLOT_END
#undef LTLT_SLOT_FMA

// L[c] = v in the lanes of `on`, for a wave-uniform slot 0 <= c < 64, by a jump
// straight to the slot's move (s_getpc + offset; every entry is 8 bytes, the
// first one 12 bytes past the address s_getpc returns).  A switch over 64 slots
// compiles to a tree of some twelve taken branches (570 cycles a step,
// measured).
#define LTLT_SLOT_MOV(OP, c) OP " %[l" #c "], %[v]\ns_branch LTLT_slot%=\n"
#define LTLT_SLOT_MOVS(OP) \
  LTLT_SLOT_MOV(OP, 0) LTLT_SLOT_MOV(OP, 1) LTLT_SLOT_MOV(OP, 2) LTLT_SLOT_MOV(OP, 3) \
  LTLT_SLOT_MOV(OP, 4) LTLT_SLOT_MOV(OP, 5) LTLT_SLOT_MOV(OP, 6) LTLT_SLOT_MOV(OP, 7) \
  LTLT_SLOT_MOV(OP, 8) LTLT_SLOT_MOV(OP, 9) LTLT_SLOT_MOV(OP, 10) LTLT_SLOT_MOV(OP, 11) \
  LTLT_SLOT_MOV(OP, 12) LTLT_SLOT_MOV(OP, 13) LTLT_SLOT_MOV(OP, 14) LTLT_SLOT_MOV(OP, 15) \
  LTLT_SLOT_MOV(OP, 16) LTLT_SLOT_MOV(OP, 17) LTLT_SLOT_MOV(OP, 18) LTLT_SLOT_MOV(OP, 19) \
  LTLT_SLOT_MOV(OP, 20) LTLT_SLOT_MOV(OP, 21) LTLT_SLOT_MOV(OP, 22) LTLT_SLOT_MOV(OP, 23) \
  LTLT_SLOT_MOV(OP, 24) LTLT_SLOT_MOV(OP, 25) LTLT_SLOT_MOV(OP, 26) LTLT_SLOT_MOV(OP, 27) \
  LTLT_SLOT_MOV(OP, 28) LTLT_SLOT_MOV(OP, 29) LTLT_SLOT_MOV(OP, 30) LTLT_SLOT_MOV(OP, 31) \
  LTLT_SLOT_MOV(OP, 32) LTLT_SLOT_MOV(OP, 33) LTLT_SLOT_MOV(OP, 34) LTLT_SLOT_MOV(OP, 35) \
  LTLT_SLOT_MOV(OP, 36) LTLT_SLOT_MOV(OP, 37) LTLT_SLOT_MOV(OP, 38) LTLT_SLOT_MOV(OP, 39) \
  LTLT_SLOT_MOV(OP, 40) LTLT_SLOT_MOV(OP, 41) LTLT_SLOT_MOV(OP, 42) LTLT_SLOT_MOV(OP, 43) \
  LTLT_SLOT_MOV(OP, 44) LTLT_SLOT_MOV(OP, 45) LTLT_SLOT_MOV(OP, 46) LTLT_SLOT_MOV(OP, 47) \
  LTLT_SLOT_MOV(OP, 48) LTLT_SLOT_MOV(OP, 49) LTLT_SLOT_MOV(OP, 50) LTLT_SLOT_MOV(OP, 51) \
  LTLT_SLOT_MOV(OP, 52) LTLT_SLOT_MOV(OP, 53) LTLT_SLOT_MOV(OP, 54) LTLT_SLOT_MOV(OP, 55) \
  LTLT_SLOT_MOV(OP, 56) LTLT_SLOT_MOV(OP, 57) LTLT_SLOT_MOV(OP, 58) LTLT_SLOT_MOV(OP, 59) \
  LTLT_SLOT_MOV(OP, 60) LTLT_SLOT_MOV(OP, 61) LTLT_SLOT_MOV(OP, 62) LTLT_SLOT_MOV(OP, 63)                     
#define LTLT_SLOT_SET(OP) \
  uint64_t keep; \
  asm volatile("s_and_saveexec_b64 %[keep], %[on]\n" \
               "s_getpc_b64 vcc\n" \
               "s_add_u32 vcc_lo, vcc_lo, %[off]\n" \
               "s_addc_u32 vcc_hi, vcc_hi, 0\n" \
               "s_setpc_b64 vcc\n" LTLT_SLOT_MOVS(OP) \
               "LTLT_slot%=:\n" \
               "s_mov_b64 exec, %[keep]\n" \
               : [keep] "=&s"(keep), \
      [l0] "+v"(L[0]), [l1] "+v"(L[1]), [l2] "+v"(L[2]), [l3] "+v"(L[3])                            , \
      [l4] "+v"(L[4]), [l5] "+v"(L[5]), [l6] "+v"(L[6]), [l7] "+v"(L[7])                            , \
      [l8] "+v"(L[8]), [l9] "+v"(L[9]), [l10] "+v"(L[10]), [l11] "+v"(L[11])                        , \
      [l12] "+v"(L[12]), [l13] "+v"(L[13]), [l14] "+v"(L[14]), [l15] "+v"(L[15])                    , \
      [l16] "+v"(L[16]), [l17] "+v"(L[17]), [l18] "+v"(L[18]), [l19] "+v"(L[19])                    , \
      [l20] "+v"(L[20]), [l21] "+v"(L[21]), [l22] "+v"(L[22]), [l23] "+v"(L[23])                    , \
      [l24] "+v"(L[24]), [l25] "+v"(L[25]), [l26] "+v"(L[26]), [l27] "+v"(L[27])                    , \
      [l28] "+v"(L[28]), [l29] "+v"(L[29]), [l30] "+v"(L[30]), [l31] "+v"(L[31])                    , \
      [l32] "+v"(L[32]), [l33] "+v"(L[33]), [l34] "+v"(L[34]), [l35] "+v"(L[35])                    , \
      [l36] "+v"(L[36]), [l37] "+v"(L[37]), [l38] "+v"(L[38]), [l39] "+v"(L[39])                    , \
      [l40] "+v"(L[40]), [l41] "+v"(L[41]), [l42] "+v"(L[42]), [l43] "+v"(L[43])                    , \
      [l44] "+v"(L[44]), [l45] "+v"(L[45]), [l46] "+v"(L[46]), [l47] "+v"(L[47])                    , \
      [l48] "+v"(L[48]), [l49] "+v"(L[49]), [l50] "+v"(L[50]), [l51] "+v"(L[51])                    , \
      [l52] "+v"(L[52]), [l53] "+v"(L[53]), [l54] "+v"(L[54]), [l55] "+v"(L[55])                    , \
      [l56] "+v"(L[56]), [l57] "+v"(L[57]), [l58] "+v"(L[58]), [l59] "+v"(L[59])                    , \
      [l60] "+v"(L[60]), [l61] "+v"(L[61]), [l62] "+v"(L[62]), [l63] "+v"(L[63]) \
               : [off] "s"(12 + 8 * c), [on] "s"(mask), [v] "v"(v) \
               : "vcc", "scc")
__device__ __forceinline__ void set_slot(double (&L)[KC], int c, bool on, double v) {
  const uint64_t mask = __ballot(on);
  LTLT_SLOT_SET("v_mov_b64_e32");
}
__device__ __forceinline__ void set_slot(float (&L)[KC], int c, bool on, float v) {
  const uint64_t mask = __ballot(on);
  LTLT_SLOT_SET("v_mov_b32_e32");
}
#undef LTLT_SLOT_SET
#undef LTLT_SLOT_MOVS
#undef LTLT_SLOT_MOV

// v + (v of lane ^ 16) or v + (v of lane ^ 32) through the gfx950 lane
// swaps (no LDS crossbar round trip): with both operands v, permlane16_swap
// returns in every 16-lane row the values of the even row of its pair and
// of the odd row (permlane32_swap: of the lower and the upper half), whose
// sum has the same two terms as v + shfl_xor(v, 16 | 32), bit for bit.
template <int OFF>
__device__ __forceinline__ unsigned xor_pair(unsigned x, unsigned& other) {
  if constexpr (OFF == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    other = r[1];
    return r[0];
  } else {
    const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    other = r[1];
    return r[0];
  }
}
template <int OFF>
__device__ __forceinline__ double xor_add(double v) {
  unsigned lo1, hi1;
  const unsigned lo0 = xor_pair<OFF>((unsigned)__double2loint(v), lo1);
  const unsigned hi0 = xor_pair<OFF>((unsigned)__double2hiint(v), hi1);
  return __hiloint2double((int)hi0, (int)lo0) + __hiloint2double((int)hi1, (int)lo1);
}
template <int OFF>
__device__ __forceinline__ float xor_add(float v) {
  unsigned o;
  const unsigned a = xor_pair<OFF>(__float_as_uint(v), o);
  return __uint_as_float(a) + __uint_as_float(o);
}
// Sum of v over the S parts of a row (lanes lane ^ 16, lane ^ 32).
template <int S, typename T>
__device__ __forceinline__ T part_sum(T v) {
  if constexpr (S == 4) v = xor_add<16>(v);
  if constexpr (S >= 2) v = xor_add<32>(v);
  return v;
}

// Maximum of an unsigned key over lanes 0-7 (DPP row shifts 1, 2, 4; the
// result sits in lane 7).
__device__ __forceinline__ unsigned oct_umax(unsigned x) {
  asm volatile(
      "s_nop 1\n"
      "v_max_u32_dpp %0, %0, %0 row_shr:1 row_mask:0xf bank_mask:0xf\n"
      "s_nop 1\n"
      "v_max_u32_dpp %0, %0, %0 row_shr:2 row_mask:0xf bank_mask:0xf\n"
      "s_nop 1\n"
      "v_max_u32_dpp %0, %0, %0 row_shr:4 row_mask:0xf bank_mask:0xf\n"
      "s_nop 1\n"
      : "+v"(x));
  return (unsigned)__builtin_amdgcn_readlane((int)x, 7);
}

// True in the lane (among those with `in`) that holds the first maximum: the
// largest v, and among equal ones the smallest lp.  When no lane has a
// candidate it is true in every `in` lane (they hold the same "none").  The
// maximum is taken over the high words of v (order-preserving, +1 so that 0
// means none); lanes that tie there are resolved by two more reductions, over
// the low words and then the positions.  The winner is left as a lane mask, not
// read out to scalars: the lane itself stores its candidate where it is
// needed, which keeps the chain of lane reads (each waits for the vector unit)
// off the step.  The step is bound by such chains, not by memory alone: clock
// stamps gave about 900 cycles to a wave's own maximum, 700 to the merge of
// the eight waves one after the other and 700 to the reduction of the records;
// with lane-resident winners and the eight waves merged across lanes a column
// step takes 3.26 -> 2.60 us with one workgroup and the n = 16384
// factorization 107.4 -> 97.4 ms (complex n = 1501: 8.44 -> 7.41 ms), factors
// bit-identical.
template <bool OCT>
__device__ __forceinline__ bool first_max_lane(const Cand& c, bool in) {
  const bool some = in && cand_lp(c) != (unsigned)kIdxNone;
  const unsigned hk = some ? (unsigned)(c.v >> 32) + 1u : 0u;
  const unsigned mh = OCT ? oct_umax(hk) : wave_umax(hk);
  bool tie = in && hk == mh;
  const unsigned long long b = __ballot(tie);
  if (__builtin_expect((b & (b - 1)) != 0 && mh != 0, 0)) {
    const unsigned lo = (unsigned)c.v;
    const unsigned ml = OCT ? oct_umax(tie ? lo : 0u) : wave_umax(tie ? lo : 0u);
    tie = tie && lo == ml;
    const unsigned nk = tie ? ~cand_lp(c) : 0u;
    const unsigned mk = OCT ? oct_umax(nk) : wave_umax(nk);
    tie = tie && nk == mk;
  }
  return tie;
}

// This wave's candidate: the first maximum of its lanes' goes into red[wave].
__device__ __forceinline__ void wave_candidate(Cand* red, int wave, const Cand& c) {
  if (first_max_lane<false>(c, true)) red[wave] = c;
}

// One grid-wide pivot agreement, in two halves called by every thread of the
// workgroup (work that does not depend on the pivot may run in between).
// Each wave has put its candidate in red (wave_candidate).
// exchange_publish: every wave waits for its own earlier stores (so a
// validated record implies they are visible), a barrier, then wave 0 merges
// the waves (lane i takes wave i's candidate) and the winning lane stores the
// workgroup's record for stamp s.
// exchange_collect: wave 0 polls every record until all carry stamp s and
// reduces them (largest magnitude, then smallest position); the result lands
// in res: p (pivot position), posw (its block-start index) and alpha (signed
// pivot value; NaN and p = posw = k+1 when no finite candidate exists), handed
// to the other waves by a barrier.  A wait that exceeds its bound, or finds the
// call's abort flag raised, raises the status words and leaves p = -1.
// early(posw) runs in wave 0 alone as soon as it knows the pivot row, ahead of
// the barrier: a place to issue loads of that row's data (a row in range, even
// if the call is being aborted).
struct __align__(16) XRes {
  double alpha;
  int p, posw;
};

__device__ __forceinline__ void exchange_publish(const PanelArgs& a, int s, int wave, int lane, int w,
                                                 const Cand* red) {
  uint64_t* recs = a.rec + (size_t)(s & 1) * (size_t)a.nrec * kRecStride;
  wait_stores();
  __syncthreads();
  if (wave == 0) {
    const Cand c = red[lane & (kPanelWaves - 1)];
    if (first_max_lane<true>(c, lane < kPanelWaves)) {
      st_coh64(&recs[(size_t)kRecStride * w + 0], c.v | rec_epoch(s));
      st_coh64(&recs[(size_t)kRecStride * w + 1], c.w | ((uint64_t)s << 43));
    }
  }
}

template <typename F>
__device__ __forceinline__ void exchange_collect(const PanelArgs& a, int s, int k, int wave, int lane, XRes& res,
                                                 F&& early) {
  const int P = a.P;
  const uint64_t* recs = a.rec + (size_t)(s & 1) * (size_t)a.nrec * kRecStride;
  if (wave == 0) {
    const uint64_t t0 = wall_ticks();
    bool gave_up = false;
    Cand c{0ull, kIdxNone};
    if (P <= kWave) {
      // one record per lane (lanes past P read the last one and drop it):
      // both words and the abort flag in one round trip
      const uint64_t* rp = &recs[(size_t)kRecStride * min(lane, P - 1)];
      uint64_t ra, rb;
      for (;;) {
        int stv;
        asm volatile(
            "global_load_dwordx2 %0, %3, off sc1\n"
            "global_load_dwordx2 %1, %3, off offset:8 sc1\n"
            "global_load_dword %2, %4, %5 sc1\n"
            "s_waitcnt vmcnt(0)"
            : "=&v"(ra), "=&v"(rb), "=&v"(stv)
            : "v"(rp), "v"(0), "s"(a.status)
            : "memory");
        const bool all = __ballot(!rec_valid(ra, rb, s)) == 0;
        const bool stop = __builtin_amdgcn_readfirstlane(stv) != 0;
        // a wait of this call that gave up elsewhere ends this one too, even
        // when every record has arrived
        if (__builtin_expect(stop || (!all && wall_ticks() - t0 > kWaitLimitTicks), 0)) {
          if (lane == 0) raise_wait_status(a.status);
          gave_up = true;
          break;
        }
        if (all) break;
      }
      if (lane < P) c = Cand{ra & 0x7FFFFFFFFFFFFFFFull, rb & 0x7FFFFFFFFFFull};
    } else {
      const int q_n = (P + kWave - 1) / kWave;
      uint64_t ra[kPollPerLane], rb[kPollPerLane];
      for (;;) {
#pragma unroll
        for (int q = 0; q < kPollPerLane; ++q) {
          const int u = q * kWave + lane;
          if (q < q_n && u < P) {
            ra[q] = ld_coh64(&recs[(size_t)kRecStride * u + 0]);
            rb[q] = ld_coh64(&recs[(size_t)kRecStride * u + 1]);
          }
        }
        const int stv = ld_coh(a.status);         // same round trip as the records
        bool ok = true;
#pragma unroll
        for (int q = 0; q < kPollPerLane; ++q) {
          const int u = q * kWave + lane;
          if (q < q_n && u < P) ok = ok && rec_valid(ra[q], rb[q], s);
        }
        const bool all = __ballot(!ok) == 0;
        if (stv != 0 || (!all && wall_ticks() - t0 > kWaitLimitTicks)) {
          if (lane == 0) raise_wait_status(a.status);
          gave_up = true;
          break;
        }
        if (all) break;
      }
      // this lane's best of its records (lane, lane + 64, ...)
#pragma unroll
      for (int q = 0; q < kPollPerLane; ++q) {
        const int u = q * kWave + lane;
        if (q < q_n && u < P) {
          const Cand o{ra[q] & 0x7FFFFFFFFFFFFFFFull, rb[q] & 0x7FFFFFFFFFFull};
          const bool take = q == 0 || o.v > c.v || (o.v == c.v && cand_lp(o) < cand_lp(c));
          c.v = take ? o.v : c.v;
          c.w = take ? o.w : c.w;
        }
      }
    }
    const bool first = first_max_lane<false>(c, true);
    const bool none = cand_lp(c) == (unsigned)kIdxNone;     // no finite candidate: no exchange
    const double v = __longlong_as_double((long long)c.v);
    XRes r;
    r.alpha = none ? (double)NAN : ((c.w >> 42) & 1 ? -v : v);
    r.p = gave_up ? -1 : (none ? k + 1 : (int)cand_lp(c));
    r.posw = none || gave_up ? k + 1 : (int)((c.w >> 21) & kIdxNone);
    early(__builtin_amdgcn_readlane(r.posw, __ffsll(__ballot(first)) - 1));
    if (first) res = r;
  }
  __syncthreads();
}

// Both halves back to back.
template <typename F>
__device__ __forceinline__ void exchange_pivot(const PanelArgs& a, int s, int k, int wave, int lane, int w,
                                               const Cand* red, XRes& res, F&& early) {
  exchange_publish(a, s, wave, lane, w, red);
  exchange_collect(a, s, k, wave, lane, res, early);
}

// The agreement when one workgroup holds every row: no records.  After one
// barrier every wave reduces the waves' candidates for itself (red alternates
// between two sets, so the next step's writes never meet a slow reader).  The
// values are uniform; none: alpha NaN, p = posw = k+1.  Against one record that the
// workgroup polls back from memory (about 1600 cycles), n = 256 takes 585 -> 416 us.
template <typename F>
__device__ __forceinline__ XRes exchange_one(int k, int wave, int lane, const Cand* red, F&& early) {
  wait_stores();
  __syncthreads();
  const Cand c = red[lane & (kPanelWaves - 1)];
  const int src = __ffsll(__ballot(first_max_lane<true>(c, lane < kPanelWaves))) - 1;
  const unsigned wlo = __builtin_amdgcn_readlane((unsigned)c.w, src);
  const unsigned whi = __builtin_amdgcn_readlane((unsigned)(c.w >> 32), src);
  const uint64_t w = ((uint64_t)whi << 32) | wlo;
  const bool none = (w & kIdxNone) == kIdxNone;
  XRes r;
  r.p = none ? k + 1 : (int)(w & kIdxNone);
  r.posw = none ? k + 1 : (int)((w >> 21) & kIdxNone);
  if (wave == 0) early(r.posw);
  const unsigned vlo = __builtin_amdgcn_readlane((unsigned)c.v, src);
  const unsigned vhi = __builtin_amdgcn_readlane((unsigned)(c.v >> 32), src) | ((unsigned)(w >> 42) & 1u) << 31;
  r.alpha = none ? (double)NAN : __hiloint2double((int)vhi, (int)vlo);
  return r;
}

// Buffer accesses; a lane whose offset is kSkip is out of
// the buffer's range: its load returns 0 and its store is dropped, without a
// branch, so that the waits for earlier loads count exactly the accesses
// issued after them.
constexpr unsigned kSkip = 0x80000000u;            // buffers are smaller than this
// Buffer cache policy: device scope (sc1) between workgroups; within one, whose
// waves share a CU and its L1, plain accesses (L2 hits instead of trips past it).
template <bool ONE>
constexpr int kPolicy = ONE ? 0 : 16;
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
template <typename T>
struct Pair { T a, b; };
template <bool ONE>
__device__ __forceinline__ void buf_store2(double a, double b, __amdgpu_buffer_rsrc_t rs, unsigned off, unsigned base) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, Pair<double>{a, b}), rs, off, base, kPolicy<ONE>);
}
template <bool ONE>
__device__ __forceinline__ void buf_store2(float a, float b, __amdgpu_buffer_rsrc_t rs, unsigned off, unsigned base) {
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, Pair<float>{a, b}), rs, off, base, kPolicy<ONE>);
}
template <bool ONE>
__device__ __forceinline__ u32x4 buf_load16(__amdgpu_buffer_rsrc_t rs, unsigned off, unsigned base) {
  return __builtin_amdgcn_raw_buffer_load_b128(rs, off, base, kPolicy<ONE>);
}
// 16 loaded bytes into v[at ..] (unless they lie past its n values).
__device__ __forceinline__ void put16(double* v, int at, int n, u32x4 x) {
  const auto d = __builtin_bit_cast(Pair<double>, x);
  if (at < n) { v[at] = d.a; v[at + 1] = d.b; }
}
__device__ __forceinline__ void put16(float* v, int at, int n, u32x4 x) {
  struct Four { float a, b, c, d; };
  const auto f = __builtin_bit_cast(Four, x);
  if (at < n) { v[at] = f.a; v[at + 1] = f.b; v[at + 2] = f.c; v[at + 3] = f.d; }
}
// One tail entry (two values).
template <bool ONE>
__device__ __forceinline__ Pair<double> buf_load2(double, __amdgpu_buffer_rsrc_t rs, unsigned off, unsigned base) {
  return __builtin_bit_cast(Pair<double>, __builtin_amdgcn_raw_buffer_load_b128(rs, off, base, kPolicy<ONE>));
}
template <bool ONE>
__device__ __forceinline__ Pair<float> buf_load2(float, __amdgpu_buffer_rsrc_t rs, unsigned off, unsigned base) {
  return __builtin_bit_cast(Pair<float>, __builtin_amdgcn_raw_buffer_load_b64(rs, off, base, kPolicy<ONE>));
}

// Four values: one complex tail entry, or a lane's two complex g.
template <bool ONE>
__device__ __forceinline__ void buf_store4(double a, double b, double c, double d, __amdgpu_buffer_rsrc_t rs,
                                           unsigned off, unsigned base) {
  buf_store2<ONE>(a, b, rs, off, base);
  buf_store2<ONE>(c, d, rs, off + 16, base);
}
template <bool ONE>
__device__ __forceinline__ void buf_store4(float a, float b, float c, float d, __amdgpu_buffer_rsrc_t rs, unsigned off,
                                           unsigned base) {
  struct Four { float a, b, c, d; };
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, Four{a, b, c, d}), rs, off, base, kPolicy<ONE>);
}
template <bool ONE>
__device__ __forceinline__ void buf_load4(double (&v)[4], __amdgpu_buffer_rsrc_t rs, unsigned off, unsigned base) {
  const auto x = __builtin_bit_cast(Pair<double>, buf_load16<ONE>(rs, off, base));
  const auto y = __builtin_bit_cast(Pair<double>, buf_load16<ONE>(rs, off + 16, base));
  v[0] = x.a; v[1] = x.b; v[2] = y.a; v[3] = y.b;
}
template <bool ONE>
__device__ __forceinline__ void buf_load4(float (&v)[4], __amdgpu_buffer_rsrc_t rs, unsigned off, unsigned base) {
  struct Four { float a, b, c, d; };
  const auto x = __builtin_bit_cast(Four, buf_load16<ONE>(rs, off, base));
  v[0] = x.a; v[1] = x.b; v[2] = x.c; v[3] = x.d;
}

// Workgroup barrier for LDS only: it waits for this wave's LDS operations
// but not for its outstanding global loads (__syncthreads does, and with
// them every tile and solution prefetch in flight).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

}  // namespace ltlt

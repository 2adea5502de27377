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

// L[c] = v where `on`, for a wave-uniform slot c: a uniform branch on the
// group of 16 slots, then selects inside the group, so that register indices
// stay static and the other 48 slots are untouched.
#define LTLT_SET_GROUP(G0)                                                       \
  if ((c >> 4) == (G0) / 16) {                                                  \
    _Pragma("unroll") for (int i = 0; i < 16; ++i) L[(G0) + i] = (on && c == (G0) + i) ? v : L[(G0) + i]; \
  }

// L[c] = v where `on`, for a wave-uniform slot c < KC: a uniform jump to the
// one slot (register indices stay static and only that slot is written),
// instead of LTLT_SET_GROUP's selects over a whole group of 16.  Measured
// faster in the two- and four-lane-per-row panels; with one lane per row the
// jump table's control flow pushed the kernel past its register budget, so
// that panel keeps the group form.
#define LTLT_SLOT_CASE(i) \
  case (i): L[(i)] = on ? v : L[(i)]; break;
#define LTLT_SLOT_CASE4(i) LTLT_SLOT_CASE(i) LTLT_SLOT_CASE((i) + 1) LTLT_SLOT_CASE((i) + 2) LTLT_SLOT_CASE((i) + 3)
#define LTLT_SLOT_CASE16(i) \
  LTLT_SLOT_CASE4(i) LTLT_SLOT_CASE4((i) + 4) LTLT_SLOT_CASE4((i) + 8) LTLT_SLOT_CASE4((i) + 12)
template <typename T>
__device__ __forceinline__ void set_slot(T (&L)[KC], int c, bool on, T v) {
  static_assert(KC == 64, "64 slots");
  switch (c) {
    LTLT_SLOT_CASE16(0) LTLT_SLOT_CASE16(16) LTLT_SLOT_CASE16(32) LTLT_SLOT_CASE16(48)
    default: break;
  }
}
#undef LTLT_SLOT_CASE16
#undef LTLT_SLOT_CASE4
#undef LTLT_SLOT_CASE

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

__device__ __forceinline__ void exchange_collect(const PanelArgs& a, int s, int k, int wave, int lane, XRes& res) {
  const int P = a.P;
  const uint64_t* recs = a.rec + (size_t)(s & 1) * (size_t)a.nrec * kRecStride;
  if (wave == 0) {
    const int q_n = (P + kWave - 1) / kWave;
    const uint64_t t0 = wall_ticks();
    uint64_t ra[kPollPerLane], rb[kPollPerLane];
    bool gave_up = false;
    for (;;) {
#pragma unroll
      for (int q = 0; q < kPollPerLane; ++q) {
        const int u = q * kWave + lane;
        if (q < q_n && u < P) {
          ra[q] = ld_coh64(&recs[(size_t)kRecStride * u + 0]);
          rb[q] = ld_coh64(&recs[(size_t)kRecStride * u + 1]);
        }
      }
      const int stv = ld_coh(a.status);           // same round trip as the records
      bool ok = true;
#pragma unroll
      for (int q = 0; q < kPollPerLane; ++q) {
        const int u = q * kWave + lane;
        if (q < q_n && u < P) ok = ok && rec_valid(ra[q], rb[q], s);
      }
      // a wait of this call that gave up elsewhere ends this one too, even
      // when every record has arrived
      const bool all = __ballot(!ok) == 0;
      if (stv != 0 || (!all && wall_ticks() - t0 > kWaitLimitTicks)) {
        if (lane == 0) raise_wait_status(a.status);
        gave_up = true;
        break;
      }
      if (all) break;
      __builtin_amdgcn_s_sleep(0);
    }
    // this lane's best of its records (lane, lane + 64, ...): positions rise
    // with neither, so ties compare them
    Cand c{0ull, kIdxNone};
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
    if (first_max_lane<false>(c, true)) {
      const bool none = cand_lp(c) == (unsigned)kIdxNone;   // no finite candidate: no exchange
      const double v = __longlong_as_double((long long)c.v);
      XRes r;
      r.alpha = none ? (double)NAN : ((c.w >> 42) & 1 ? -v : v);
      r.p = gave_up ? -1 : (none ? k + 1 : (int)cand_lp(c));
      r.posw = none ? k + 1 : (int)((c.w >> 21) & kIdxNone);
      res = r;
    }
  }
  __syncthreads();
}

// Both halves back to back.
__device__ __forceinline__ void exchange_pivot(const PanelArgs& a, int s, int k, int wave, int lane, int w,
                                               const Cand* red, XRes& res) {
  exchange_publish(a, s, wave, lane, w, red);
  exchange_collect(a, s, k, wave, lane, res);
}

}  // namespace ltlt

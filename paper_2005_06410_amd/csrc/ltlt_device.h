// Device-side helpers shared by the gfx950 kernels of the LTL^T library.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ltlt {

constexpr int kWave = 64;            // CDNA wavefront width

// ---------------------------------------------------------------------------
// Coherent (agent-scope) relaxed accesses.  On gfx950 these compile to
// global loads/stores with the sc1 bit: they bypass the non-coherent part of
// the per-XCD L2, so data written this way by one workgroup is seen by any
// other workgroup that reads it this way, without the full-L2 writeback /
// invalidate that an agent-scope release/acquire fence costs.  Ordering
// between a workgroup's data stores and its later flag update comes from
// waiting for the stores to complete (s_waitcnt vmcnt(0)) before the flag.
// ---------------------------------------------------------------------------
__device__ __forceinline__ double ld_coh(const double* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int ld_coh(const int* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned ld_coh(const unsigned* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_coh(double* p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_coh(int* p, int v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void wait_stores() {
  // vmcnt(0) expcnt(0) lgkmcnt(0): every earlier memory operation of this
  // wave has completed.
  __builtin_amdgcn_s_waitcnt(0);
}

// Wall clock for bounded device-side waits (constant 100 MHz counter).
__device__ __forceinline__ uint64_t wall_ticks() { return __builtin_amdgcn_s_memrealtime(); }
constexpr uint64_t kWaitLimitTicks = 200000000ull;   // 2 s at 100 MHz

// Bounded-wait status, two words per device:
//   status[0]  this call's abort flag: cleared when a call starts, raised when
//              one of its waits gives up; every later wait of the call gives up
//              at once, and the kernels that write results (commit, Pfaffian)
//              write NaN / sign 0 instead;
//   status[1]  sticky: raised together with status[0], cleared only when the
//              host reads it (ltlt_device_status), so a failed call is seen
//              even if later calls succeed.
__device__ __forceinline__ void raise_wait_status(int* status) {
  atomicOr(status, 1);
  atomicOr(status + 1, 1);
}

// ---------------------------------------------------------------------------
// Register-resident column refresh and wave-wide maximum, shared by the
// panel and the batched kernels.
// ---------------------------------------------------------------------------

// The 16 slots of one g register: acc[c % 4] += g(lane (lane & ~15) + c) * L[c0 + c]
// through v_fmac with a DPP row broadcast (row_newbcast, gfx950).  One asm
// block, led by the two wait states a DPP read needs after a VALU write of its
// source, so that no compiler-inserted copy of g can sit in between.
#define LTLT_FMAC16(OP)                                                                                  \
  asm volatile("s_nop 1\n"                                                                               \
               OP " %0, %4, %5 row_newbcast:0 row_mask:0xf bank_mask:0xf\n"                              \
               OP " %1, %4, %6 row_newbcast:1 row_mask:0xf bank_mask:0xf\n"                              \
               OP " %2, %4, %7 row_newbcast:2 row_mask:0xf bank_mask:0xf\n"                              \
               OP " %3, %4, %8 row_newbcast:3 row_mask:0xf bank_mask:0xf\n"                              \
               OP " %0, %4, %9 row_newbcast:4 row_mask:0xf bank_mask:0xf\n"                              \
               OP " %1, %4, %10 row_newbcast:5 row_mask:0xf bank_mask:0xf\n"                             \
               OP " %2, %4, %11 row_newbcast:6 row_mask:0xf bank_mask:0xf\n"                             \
               OP " %3, %4, %12 row_newbcast:7 row_mask:0xf bank_mask:0xf\n"                             \
               OP " %0, %4, %13 row_newbcast:8 row_mask:0xf bank_mask:0xf\n"                             \
               OP " %1, %4, %14 row_newbcast:9 row_mask:0xf bank_mask:0xf\n"                             \
               OP " %2, %4, %15 row_newbcast:10 row_mask:0xf bank_mask:0xf\n"                            \
               OP " %3, %4, %16 row_newbcast:11 row_mask:0xf bank_mask:0xf\n"                            \
               OP " %0, %4, %17 row_newbcast:12 row_mask:0xf bank_mask:0xf\n"                            \
               OP " %1, %4, %18 row_newbcast:13 row_mask:0xf bank_mask:0xf\n"                            \
               OP " %2, %4, %19 row_newbcast:14 row_mask:0xf bank_mask:0xf\n"                            \
               OP " %3, %4, %20 row_newbcast:15 row_mask:0xf bank_mask:0xf\n"                            \
               : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3])                                  \
               : "v"(g), "v"(L[c0 + 0]), "v"(L[c0 + 1]), "v"(L[c0 + 2]), "v"(L[c0 + 3]), "v"(L[c0 + 4]), \
                 "v"(L[c0 + 5]), "v"(L[c0 + 6]), "v"(L[c0 + 7]), "v"(L[c0 + 8]), "v"(L[c0 + 9]),         \
                 "v"(L[c0 + 10]), "v"(L[c0 + 11]), "v"(L[c0 + 12]), "v"(L[c0 + 13]), "v"(L[c0 + 14]),    \
                 "v"(L[c0 + 15]))
template <int K, int NS>
__device__ __forceinline__ void refresh16(double (&acc)[4], double g, const double (&L)[NS]) {
  constexpr int c0 = 16 * K;
  LTLT_FMAC16("v_fmac_f64_dpp");
}
template <int K, int NS>
__device__ __forceinline__ void refresh16(float (&acc)[4], float g, const float (&L)[NS]) {
  constexpr int c0 = 16 * K;
  LTLT_FMAC16("v_fmac_f32_dpp");
}
#undef LTLT_FMAC16

// The 16 x 16 x 4 matrix instructions: lane l gives A(l%16, l/16) and B(l/16, l%16).
typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

template <typename T> struct Mfma;
template <> struct Mfma<double> {
  typedef v4d acc_t;
  static __device__ __forceinline__ acc_t run(double a, double b, acc_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  // output element v of lane l sits at row (l/16) + 4v, column l%16
  static __device__ __forceinline__ int row(int l, int v) { return (l >> 4) + 4 * v; }
};
template <> struct Mfma<float> {
  typedef v4f acc_t;
  static __device__ __forceinline__ acc_t run(float a, float b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  // output element v of lane l sits at row 4(l/16) + v, column l%16
  static __device__ __forceinline__ int row(int l, int v) { return 4 * (l >> 4) + v; }
};

// Wave-wide maximum of an unsigned key (every lane gets it): DPP row shifts
// and row broadcasts folded into v_max_u32 (a lane without a source is not
// written and keeps its key), two wait states before each DPP read; lane 63
// ends with the maximum.
__device__ __forceinline__ unsigned wave_umax(unsigned x) {
  asm volatile(
      "s_nop 1\n"
      "v_max_u32_dpp %0, %0, %0 row_shr:1 row_mask:0xf bank_mask:0xf\n"
      "s_nop 1\n"
      "v_max_u32_dpp %0, %0, %0 row_shr:2 row_mask:0xf bank_mask:0xf\n"
      "s_nop 1\n"
      "v_max_u32_dpp %0, %0, %0 row_shr:4 row_mask:0xf bank_mask:0xf\n"
      "s_nop 1\n"
      "v_max_u32_dpp %0, %0, %0 row_shr:8 row_mask:0xf bank_mask:0xf\n"
      "s_nop 1\n"
      "v_max_u32_dpp %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0xf\n"
      "s_nop 1\n"
      "v_max_u32_dpp %0, %0, %0 row_bcast:31 row_mask:0xc bank_mask:0xf\n"
      "s_nop 1\n"
      : "+v"(x));
  return (unsigned)__builtin_amdgcn_readlane((int)x, 63);
}
}  // namespace ltlt

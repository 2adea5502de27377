// CONVGEMM on gfx950: the convolution O = conv(F, I) as one fp32 matrix product
// O^ = F^ . im2col(I) whose second operand is gathered from the input tensor
// while it is staged into LDS (the paper's section 4, Figure 6: im2col folded
// into the packing of the GEMM's B operand, so the augmented matrix of
// section 3 is never formed in memory).
//
// Four kernels, chosen by choose() below: the LDS-staged gather described here
// (any layer), a register-direct one (no padding), channel blocks (the usual
// layers of eleven channels and more) and runs of taps (strided first layers),
// each described where it stands.
//
// The LDS-staged gather.  One workgroup (4 waves, 2 x 2) owns an MT x NT tile of O^
// (MT filters x NT output positions).  The contraction runs in chunks of
// KC = 16 or 32 rows of im2col(I) (= columns of F^):
//   * F^ chunk (MT x KC): coalesced loads along the filter index, kept in LDS
//     as rows of KC contraction values per filter;
//   * im2col chunk (KC x NT): each thread owns one output position (column)
//     of the tile, decoded once into (oh, ow, n), and walks its contraction
//     rows r -> (y, x, c) incrementally; the value is I at
//     (s*oh + y - p, s*ow + x - p, c, n) or zero outside the input, exactly
//     Figure 6's index maps.  Neighbouring threads hold neighbouring output
//     positions, so each load instruction reads a contiguous (stride s) run of
//     one input row.  Stored in LDS as KC contraction values per column;
//   * v_mfma_f32_16x16x4_f32 on 16 x 16 blocks.  Because the contraction may
//     be taken in any order, lane group q of a wave (lanes 16q .. 16q+15)
//     takes contraction rows 4q .. 4q+3 of each group of 16 for that group's
//     four MFMAs, so one ds_read_b128 feeds four MFMAs;
//   * two LDS buffers: the next chunk's global loads are issued before the
//     current chunk's MFMAs and written to the other buffer after them, one
//     barrier per chunk.
// Tiles are handed out XCD-aware: consecutive workgroup ids go to different
// XCDs (round-robin), so ids are remapped to give each XCD a contiguous range of
// tiles, filter tiles fastest; tiles that share output positions (and the input
// rows they read) then run on the same XCD and share its L2.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "convgemm.h"

namespace convgemm {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
constexpr int kDirectMaxK = 16384;   // register-direct kernel: its row table (4 bytes a row) fits 64 KiB of LDS

struct Geometry {
    int M, K, N;        // kn, kh*kw*ci, ho*wo*b
    int ci;
    int kh, khw;        // kh, kh*kw
    int kw;
    int hi, wi, hiwi;   // input height, width, hi*wi
    int ho, hw;         // ho, ho*wo
    int s, p;
    int64_t sample;     // hi*wi*ci: input floats per batch entry
    uint32_t ibytes;    // bytes of I (< 2^32)
    uint32_t fbytes;    // bytes of F (< 2^32)
};

// Raw buffer resource over a whole tensor: base address, no stride, the
// tensor's size in bytes as the range, 32-bit data format.  A buffer load
// then takes a per-lane byte offset (vector) plus a wave-uniform byte offset
// (scalar), so the gather needs no per-element address arithmetic.
__device__ inline __amdgpu_buffer_rsrc_t tensor_rsrc(const float* p, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), (short)0, (int)bytes, 0x00020000);
}

__device__ inline float buffer_load(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)voff, (int)soff, 0));
}

// One lane's share of a 16 x 16 output block: filters m .. m+3 of output
// position n (the v_mfma_f32_16x16x4_f32 result layout), contiguous in O;
// one 16-byte store when kn is a multiple of 4 and O is 16-byte aligned (vec).
__device__ inline void store_block(float* __restrict__ O, const Geometry& g, int m, int n, f4 v, int accumulate,
                                   int vec)
{
    if (n >= g.N || m >= g.M) return;
    float* o = O + (int64_t)n * g.M + m;
    if (vec) {
        if (accumulate) v += *reinterpret_cast<const f4*>(o);
        *reinterpret_cast<f4*>(o) = v;
    } else {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (m + q < g.M) o[q] = accumulate ? o[q] + v[q] : v[q];
    }
}

template <int MT, int NT, bool PAD, int KC>
__global__ __launch_bounds__(kThreads) void convgemm_kernel(Geometry g, const float* __restrict__ F,
                                                            const float* __restrict__ I,
                                                            float* __restrict__ O, int accumulate,
                                                            int vec, int mtiles, int ntiles)
{
    constexpr int kKC = KC;                        // contraction rows per staged chunk
    constexpr int kKP = KC + 4;                    // LDS floats per tile row (padded against bank conflicts)
    constexpr int WM = MT / 2, WN = NT / 2;        // wave tile
    constexpr int BM = WM / 16, BN = WN / 16;      // 16 x 16 blocks per wave
    constexpr int AK = MT == 192 ? kKC : MT * kKC / kThreads; // contraction rows per F^-loading thread
    constexpr int ATHREADS = MT * kKC / AK;        // threads that load F^ (whole waves)
    constexpr int RPT = kKC * NT / kThreads;       // im2col rows per thread per chunk
    static_assert(ATHREADS <= kThreads && ATHREADS % 64 == 0 && ATHREADS * AK == MT * kKC && AK % 4 == 0,
                  "F^ loader split");
    static_assert(RPT * kThreads == kKC * NT && RPT % 4 == 0 && BM >= 1 && BN >= 1 && kKC % 16 == 0,
                  "tile shape");

    __shared__ __attribute__((aligned(16))) float As[2][MT * kKP];
    __shared__ __attribute__((aligned(16))) float Bs[2][NT * kKP];

    // XCD-aware tile order: within the largest multiple of 8 of the tile
    // count, workgroup id -> XCD (id mod 8) gets the contiguous tile range
    // [xcd * T8/8, (xcd + 1) * T8/8); the remainder keeps the identity.
    const int T = mtiles * ntiles;
    const int T8 = T & ~7;
    const int bid = blockIdx.x;
    const int t = bid < T8 ? (bid & 7) * (T8 >> 3) + (bid >> 3) : bid;
    const int m0 = (t % mtiles) * MT;
    const int n0 = (t / mtiles) * NT;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wm = wave & 1, wn = wave >> 1;

    // F^ loader: filter am (clamped: rows past kn only feed outputs that are
    // never stored), contraction rows akg .. akg+AK-1 of each chunk.
    const bool a_loader = tid < ATHREADS;            // whole waves
    const int am = tid % MT;
    const int akg = (tid / MT) * AK;
    const int am_c = min(m0 + am, g.M - 1);
    const uint32_t aoff = (uint32_t)(akg * g.M + am_c) * 4u;   // bytes from row k0 of F^

    // im2col gatherer: output position bcol of the tile (clamped to the last
    // one: columns past N only feed outputs that are never stored), decoded
    // once into (oh, ow, n); contraction rows brow .. brow+RPT-1 of each chunk.
    // brow is the same for a whole wave, so the row -> (y, x, c) walk and the
    // row's offset y + hi*x + hi*wi*c live in scalar registers.
    const int bcol = tid % NT;
    const int brow = __builtin_amdgcn_readfirstlane((tid / NT) * RPT);
    const int ncol = min(n0 + bcol, g.N - 1);
    const int nb = ncol / g.hw;
    const int prem = ncol - nb * g.hw;
    const int ow = prem / g.ho;
    const int oh = prem - ow * g.ho;
    const int hbase = oh * g.s - g.p;
    const int wbase = ow * g.s - g.p;
    // without padding every tap of a valid column is inside the input: the
    // element is I[colpos + row offset], colpos < 2^30 (checked on the host)
    const uint32_t colbyte = PAD ? 0u : (uint32_t)(nb * g.sample + hbase + g.hi * wbase) * 4u;
    const float* __restrict__ Ib = I + (int64_t)nb * g.sample;
    const __amdgpu_buffer_rsrc_t irs = tensor_rsrc(I, g.ibytes);
    const __amdgpu_buffer_rsrc_t frs = tensor_rsrc(F, g.fbytes);

    float ra[AK];
    float rb[RPT];
    uint32_t amask = ~0u, bmask = ~0u;   // bit j: value j is a real entry (else stored as 0)

    auto load_chunk = [&](int chunk) {
        const int k0 = chunk * kKC;
        const bool tail = k0 + kKC > g.K;            // uniform: only the last chunk can be partial
        if (a_loader) {
            if (!tail) {
#pragma unroll
                for (int i = 0; i < AK; ++i) ra[i] = buffer_load(frs, aoff, (uint32_t)(k0 + i) * g.M * 4u);
                amask = ~0u;
            } else {
                amask = 0;
#pragma unroll
                for (int i = 0; i < AK; ++i) {
                    const int k = k0 + akg + i;
                    const bool ok = k < g.K;
                    ra[i] = F[(int64_t)(ok ? k : g.K - 1) * g.M + am_c];
                    amask |= (uint32_t)ok << i;
                }
            }
        }
        const int r0 = k0 + brow;
        int c = r0 / g.khw;
        const int rem = r0 - c * g.khw;
        int x = rem / g.kh;
        int y = rem - x * g.kh;
        bmask = 0;
#pragma unroll
        for (int j = 0; j < RPT; ++j) {
            const bool rok = r0 + j < g.K;           // uniform
            if (!PAD) {
                const int roff = rok ? y + g.hi * x + g.hiwi * c : 0;
                rb[j] = buffer_load(irs, colbyte, (uint32_t)roff * 4u);
                bmask |= (uint32_t)rok << j;
            } else {
                const int hh = hbase + y, ww = wbase + x;
                const bool ok = rok && (unsigned)hh < (unsigned)g.hi && (unsigned)ww < (unsigned)g.wi;
                const float v = Ib[ok ? hh + g.hi * ww + g.hiwi * c : 0];
                rb[j] = v;
                bmask |= (uint32_t)ok << j;
            }
            // next contraction row: y fastest, then x, then c
            ++y;
            const bool wy = y == g.kh;
            y = wy ? 0 : y;
            x += wy;
            const bool wx = x == g.kw;
            x = wx ? 0 : x;
            c += wx;
        }
    };

    // The zeroing is applied here, after the MFMAs, so that nothing waits for
    // the loads before the MFMAs are issued; full chunks without padding store
    // the loaded values as they are.
    auto store_chunk = [&](int buf, bool tail) {
        if (a_loader) {
            float* ap = &As[buf][am * kKP + akg];
#pragma unroll
            for (int i = 0; i < AK; i += 4) {
                f4 v = f4{ra[i], ra[i + 1], ra[i + 2], ra[i + 3]};
                if (tail) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) v[q] = (amask >> (i + q)) & 1 ? v[q] : 0.0f;
                }
                *reinterpret_cast<f4*>(ap + i) = v;
            }
        }
        float* bp = &Bs[buf][bcol * kKP + brow];
#pragma unroll
        for (int j = 0; j < RPT; j += 4) {
            f4 v = f4{rb[j], rb[j + 1], rb[j + 2], rb[j + 3]};
            if (PAD || tail) {
#pragma unroll
                for (int q = 0; q < 4; ++q) v[q] = (bmask >> (j + q)) & 1 ? v[q] : 0.0f;
            }
            *reinterpret_cast<f4*>(bp + j) = v;
        }
    };

    f4 acc[BM][BN];
#pragma unroll
    for (int i = 0; i < BM; ++i)
#pragma unroll
        for (int j = 0; j < BN; ++j) acc[i][j] = f4{0.0f, 0.0f, 0.0f, 0.0f};

    // Each group of 16 contraction rows: lane group q = lane/16 takes rows
    // 4q .. 4q+3 of the group, one per MFMA of the group's four.
    auto compute = [&](int buf) {
        const float* ap = &As[buf][(wm * WM + (lane & 15)) * kKP + 4 * (lane >> 4)];
        const float* bp = &Bs[buf][(wn * WN + (lane & 15)) * kKP + 4 * (lane >> 4)];
#pragma unroll
        for (int g16 = 0; g16 < kKC; g16 += 16) {
            f4 a[BM], b[BN];
#pragma unroll
            for (int i = 0; i < BM; ++i) a[i] = *reinterpret_cast<const f4*>(ap + i * 16 * kKP + g16);
#pragma unroll
            for (int j = 0; j < BN; ++j) b[j] = *reinterpret_cast<const f4*>(bp + j * 16 * kKP + g16);
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)
#pragma unroll
                for (int i = 0; i < BM; ++i)
#pragma unroll
                    for (int j = 0; j < BN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][kk], b[j][kk], acc[i][j], 0, 0, 0);
        }
    };

    const int nchunks = (g.K + kKC - 1) / kKC;
    load_chunk(0);
    store_chunk(0, kKC > g.K);
    __syncthreads();
    // The scheduling barriers keep the next chunk's loads ahead of the MFMAs
    // and their LDS stores behind them, so the loads' latency is covered.
    for (int chunk = 0; chunk + 1 < nchunks; ++chunk) {
        const int buf = chunk & 1;
        load_chunk(chunk + 1);
        __builtin_amdgcn_sched_barrier(0);
        compute(buf);
        __builtin_amdgcn_sched_barrier(0);
        store_chunk(buf ^ 1, (chunk + 2) * kKC > g.K);
        __syncthreads();
    }
    compute((nchunks - 1) & 1);

    // Epilogue: lane holds rows 4*(lane/16) .. +3 of column lane%16 of each
    // 16 x 16 block.
#pragma unroll
    for (int i = 0; i < BM; ++i)
#pragma unroll
        for (int j = 0; j < BN; ++j)
            store_block(O, g, m0 + wm * WM + i * 16 + 4 * (lane >> 4), n0 + wn * WN + j * 16 + (lane & 15),
                        acc[i][j], accumulate, vec);
}

// Register-direct CONVGEMM (no padding): every wave loads the operand values
// its own MFMAs consume straight into registers, so there is no LDS staging
// and no barrier in the contraction loop; waves run independently and the
// operands they share (F^ rows between the two waves of a tile row, input
// positions between the two of a tile column, and the im2col duplication of
// the input) are served by the L1 and L2 caches.
//
// Tile: 4 waves (2 x 2), wave tile 16BM x 16BN, workgroup tile 32BM x 32BN.
// Contraction in groups of 16 rows; lane group q = lane/16 takes rows
// 4q .. 4q+3 of a group, one per MFMA, so that:
//   * F^ value (filter m, row k0 + 4q + kk): byte (k0 + kk)*4kn [wave-uniform,
//     the scalar offset] + (4q kn + m)*4 [per lane, fixed];
//   * im2col value (row k0 + 4q + kk, position n): byte colpos(n) [per lane,
//     fixed] + rowoff(k0 + 4q + kk) [per lane group], where rowoff(r) =
//     4 (y + hi x + hi wi c) comes from a table of all rows built in LDS when
//     the workgroup starts (one ds_read_b128 gives a lane its four rows of a
//     group).  Without padding every tap of a valid position is inside the
//     input, so no element needs a check.
// Two register sets pipeline the groups: the next group's loads are issued
// before the current group's MFMAs.
// O += v with one atomic add per element: the contraction of a tile split
// over several workgroups (O cleared first unless accumulating).
__device__ inline void add_block(float* __restrict__ O, const Geometry& g, int m, int n, f4 v)
{
    if (n >= g.N || m >= g.M) return;
    float* o = O + (int64_t)n * g.M + m;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (m + q < g.M) unsafeAtomicAdd(o + q, v[q]);
}

__global__ void zero_kernel(float* __restrict__ O, int64_t count)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
        O[i] = 0.0f;
}

template <int BM, int BN, bool SPLIT>
__global__ __launch_bounds__(kThreads) void convgemm_direct_kernel(Geometry g, const float* __restrict__ F,
                                                                   const float* __restrict__ I,
                                                                   float* __restrict__ O, int accumulate,
                                                                   int vec, int mtiles, int ntiles, int kpad,
                                                                   int kparts)
{
    constexpr int WM = 16 * BM, WN = 16 * BN;
    constexpr int MT = 2 * WM, NT = 2 * WN;
    extern __shared__ int rowoff[];                // kpad entries; rows past K read offset 0
    // workgroup T * part + b takes groups [part * G / kparts, (part + 1) * G /
    // kparts) of the contraction of tile b; only its rows' offsets are formed
    const int T = mtiles * ntiles;
    const int ngroups = (g.K + 15) / 16;
    int part = 0, glo = 0, ghi = ngroups;
    if (SPLIT) {
        part = blockIdx.x / T;
        glo = part * ngroups / kparts;
        ghi = (part + 1) * ngroups / kparts;
    }
    for (int r = glo * 16 + threadIdx.x; r < ghi * 16; r += kThreads) {
        int v = 0;
        if (r < g.K) {
            const int c = r / g.khw, rem = r - c * g.khw, x = rem / g.kh, y = rem - x * g.kh;
            v = (y + g.hi * x + g.hiwi * c) * 4;
        }
        rowoff[r] = v;
    }
    __syncthreads();

    // XCD-aware tile order, as in the LDS-staged kernel
    const int T8 = T & ~7;
    const int bid = blockIdx.x - part * T;
    const int t = bid < T8 ? (bid & 7) * (T8 >> 3) + (bid >> 3) : bid;
    const int m0 = (t % mtiles) * MT;
    const int n0 = (t / mtiles) * NT;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave & 1, wn = wave >> 1;
    const int q = lane >> 4, l16 = lane & 15;
    const __amdgpu_buffer_rsrc_t irs = tensor_rsrc(I, g.ibytes);
    const __amdgpu_buffer_rsrc_t frs = tensor_rsrc(F, g.fbytes);

    // per-lane fixed offsets; filters and positions past the edge are clamped
    // (they only feed outputs that are never stored)
    int am[BM];
    uint32_t aoff[BM], coff[BN];
#pragma unroll
    for (int i = 0; i < BM; ++i) {
        am[i] = min(m0 + wm * WM + 16 * i + l16, g.M - 1);
        aoff[i] = (uint32_t)(4 * q * g.M + am[i]) * 4u;
    }
#pragma unroll
    for (int j = 0; j < BN; ++j) {
        const int n = min(n0 + wn * WN + 16 * j + l16, g.N - 1);
        const int nb = n / g.hw, rem = n - nb * g.hw, ow = rem / g.ho, oh = rem - ow * g.ho;
        coff[j] = (uint32_t)(nb * g.sample + oh * g.s + g.hi * (ow * g.s)) * 4u;
    }

    f4 acc[BM][BN];
#pragma unroll
    for (int i = 0; i < BM; ++i)
#pragma unroll
        for (int j = 0; j < BN; ++j) acc[i][j] = f4{0.0f, 0.0f, 0.0f, 0.0f};

    float a[2][BM][4], b[2][BN][4];
    auto load = [&](int grp, int set) {
        const int k0 = grp * 16;
        const int4 r4 = *reinterpret_cast<const int4*>(&rowoff[k0 + 4 * q]);
        const uint32_t rr[4] = {(uint32_t)r4.x, (uint32_t)r4.y, (uint32_t)r4.z, (uint32_t)r4.w};
        if (k0 + 16 <= g.K) {
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
#pragma unroll
                for (int i = 0; i < BM; ++i) a[set][i][kk] = buffer_load(frs, aoff[i], (uint32_t)(k0 + kk) * g.M * 4u);
#pragma unroll
                for (int j = 0; j < BN; ++j) b[set][j][kk] = buffer_load(irs, coff[j] + rr[kk], 0u);
            }
        } else {
            // last, partial group: F^ rows past K are loaded clamped and zeroed
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                const int row = k0 + 4 * q + kk;
                const bool ok = row < g.K;
                const int rc = ok ? row : g.K - 1;
#pragma unroll
                for (int i = 0; i < BM; ++i) {
                    const float v = buffer_load(frs, (uint32_t)(rc * g.M + am[i]) * 4u, 0u);
                    a[set][i][kk] = ok ? v : 0.0f;
                }
#pragma unroll
                for (int j = 0; j < BN; ++j) b[set][j][kk] = buffer_load(irs, coff[j] + rr[kk], 0u);
            }
        }
    };
    auto compute = [&](int set) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
            for (int i = 0; i < BM; ++i)
#pragma unroll
                for (int j = 0; j < BN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[set][i][kk], b[set][j][kk], acc[i][j], 0, 0, 0);
    };

    int grp = glo;
    if (grp < ghi) load(grp, 0);
    for (; grp + 2 <= ghi; grp += 2) {
        load(grp + 1, 1);
        __builtin_amdgcn_sched_barrier(0);
        compute(0);
        __builtin_amdgcn_sched_barrier(0);
        if (grp + 2 < ghi) load(grp + 2, 0);
        __builtin_amdgcn_sched_barrier(0);
        compute(1);
        __builtin_amdgcn_sched_barrier(0);
    }
    if (grp < ghi) compute(0);

    if (SPLIT) {
#pragma unroll
        for (int i = 0; i < BM; ++i)
#pragma unroll
            for (int j = 0; j < BN; ++j)
                add_block(O, g, m0 + wm * WM + 16 * i + 4 * q, n0 + wn * WN + 16 * j + l16, acc[i][j]);
        return;
    }

#pragma unroll
    for (int i = 0; i < BM; ++i)
#pragma unroll
        for (int j = 0; j < BN; ++j)
            store_block(O, g, m0 + wm * WM + 16 * i + 4 * q, n0 + wn * WN + 16 * j + l16, acc[i][j], accumulate,
                        vec);
}

// Channel-block CONVGEMM (any stride and padding).  The contraction may be
// taken in any order: here a group of 16 rows is 16 consecutive channels at one
// tap (y, x), the taps running inside a block of 16 channels.  Then within a
// group
//   * every address is a fixed per-lane part plus a wave-uniform part (the
//     buffer load's scalar offset), in both operands: no row table, no
//     per-element address arithmetic;
//   * whether a tap of a position falls into the padding is one decision per
//     position and group, not per element: the position's offset is replaced
//     by one past the buffer's range, for which the load returns zero (the
//     channels past the last one, in a partial block, likewise, in both
//     operands);
//   * the taps of a channel block re-read the same 16 input planes, a working
//     set that the L1 holds.
// As in the register-direct kernel every wave loads its own MFMA operands,
// lane group q taking channels 4q .. 4q+3 of the block, and two register sets
// pipeline the groups.  With VECA (kn a multiple of BM) a lane's BM filters are
// consecutive, one wide load per contraction row.
// The waves of a workgroup share one 16 BM x 16 BN tile and split its
// contraction; their partial sums meet in LDS and are added in wave order.
// Small tiles keep the last round of the grid short and let few positions
// (single images) fill the chip, and a 64 x 32 wave tile needs 12 loads per 32
// MFMAs where the 32 x 64 wave tile of four waves side by side needs 20.
// Measured (GEMM M x N x K): AlexNet layer 4 at b = 80 (192 x 208080
// x 1600) 1.13 -> 0.95 ms (134 TFLOP/s, 87 % of a large fp32 matrix product's
// rate), layer 8 (256 x 9680 x 3456) 0.193 -> 0.136 ms, layer 7 at b = 1 (384
// x 121 x 3456) 45 -> 15 us, 3 x 3 with padding 1 (384 x 11664 x 1728) 270 ->
// 133 us (register-direct and LDS-staged kernels before).
constexpr uint32_t kOutside = 0x80000000u;     // past any tensor these kernels take (checked on the host)

__host__ __device__ inline int tap_groups(const Geometry& g) { return (g.ci + 15) / 16 * g.khw; }
struct TapWalk {                               // the group's tap and channel block, wave-uniform
    int y, x, c0;
};
__device__ inline TapWalk tap_at(const Geometry& g, int grp)
{
    TapWalk t;
    const int cb = grp / g.khw, tap = grp - cb * g.khw;
    t.x = tap / g.kh;
    t.y = tap - t.x * g.kh;
    t.c0 = cb * 16;
    return t;
}
__device__ inline void tap_next(const Geometry& g, TapWalk& t)
{
    if (++t.y == g.kh) {
        t.y = 0;
        if (++t.x == g.kw) {
            t.x = 0;
            t.c0 += 16;
        }
    }
}

template <int BM>
__device__ inline void load_filters(float (&a)[BM][4], int kk, __amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff)
{
    if constexpr (BM == 1) {
        a[0][kk] = buffer_load(r, voff, soff);
    } else if constexpr (BM == 2) {
        typedef float f2 __attribute__((ext_vector_type(2)));
        const f2 v = __builtin_bit_cast(f2, __builtin_amdgcn_raw_buffer_load_b64(r, (int)voff, (int)soff, 0));
        a[0][kk] = v[0], a[1][kk] = v[1];
    } else {
        const f4 v = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, (int)soff, 0));
        a[0][kk] = v[0], a[1][kk] = v[1], a[2][kk] = v[2], a[3][kk] = v[3];
    }
}

// One wave's 16 BM x 16 BN tile at filters m0, positions n0, over groups
// [glo, ghi).
template <int BM, int BN, bool PAD, bool VECA>
__device__ inline void tap_tile(const Geometry& g, __amdgpu_buffer_rsrc_t frs, __amdgpu_buffer_rsrc_t irs, int m0,
                                int n0, int glo, int ghi, f4 (&acc)[BM][BN])
{
    const int lane = threadIdx.x & 63, q = lane >> 4, l16 = lane & 15;
    // per-lane fixed parts; filters and positions past the edge are clamped
    // (they only feed outputs that are never stored)
    uint32_t aoff[VECA ? 1 : BM], coff[BN];
    int hb[BN], wb[BN];
    if constexpr (VECA) {
        aoff[0] = (uint32_t)(4 * q * g.khw * g.M + min(m0 + BM * l16, g.M - BM)) * 4u;
    } else {
#pragma unroll
        for (int i = 0; i < BM; ++i) aoff[i] = (uint32_t)(4 * q * g.khw * g.M + min(m0 + BM * l16 + i, g.M - 1)) * 4u;
    }
#pragma unroll
    for (int j = 0; j < BN; ++j) {
        const int n = min(n0 + 16 * j + l16, g.N - 1);
        const int nb = n / g.hw, rem = n - nb * g.hw, ow = rem / g.ho, oh = rem - ow * g.ho;
        hb[j] = oh * g.s - g.p;
        wb[j] = ow * g.s - g.p;
        coff[j] = (uint32_t)(nb * g.sample + (int64_t)4 * q * g.hiwi + hb[j] + (int64_t)g.hi * wb[j]) * 4u;
    }
#pragma unroll
    for (int i = 0; i < BM; ++i)
#pragma unroll
        for (int j = 0; j < BN; ++j) acc[i][j] = f4{0.0f, 0.0f, 0.0f, 0.0f};

    float a[2][BM][4], b[2][BN][4];
    TapWalk tw = tap_at(g, glo);
    auto load = [&](int set) {
        const uint32_t tapoff = (uint32_t)(tw.y + g.hi * tw.x) * 4u;
        uint32_t vo[BN];
#pragma unroll
        for (int j = 0; j < BN; ++j) {
            if (PAD) {
                const bool in = (unsigned)(hb[j] + tw.y) < (unsigned)g.hi && (unsigned)(wb[j] + tw.x) < (unsigned)g.wi;
                vo[j] = in ? coff[j] + tapoff : kOutside;
            } else {
                vo[j] = coff[j];
            }
        }
        // whole: every lane's four channels exist (all but a partial block)
        auto rows = [&](bool whole) {
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                const bool in = whole || tw.c0 + 4 * q + kk < g.ci;
                const uint32_t frow = (uint32_t)(tw.y + g.kh * tw.x + (tw.c0 + kk) * g.khw) * g.M * 4u;
                const uint32_t irow = (uint32_t)(tw.c0 + kk) * g.hiwi * 4u + (PAD ? 0u : tapoff);
                if constexpr (VECA) {
                    load_filters<BM>(a[set], kk, frs, in ? aoff[0] : kOutside, frow);
                } else {
#pragma unroll
                    for (int i = 0; i < BM; ++i) a[set][i][kk] = buffer_load(frs, in ? aoff[i] : kOutside, frow);
                }
#pragma unroll
                for (int j = 0; j < BN; ++j) b[set][j][kk] = buffer_load(irs, in ? vo[j] : kOutside, irow);
            }
        };
        if (tw.c0 + 16 <= g.ci) rows(true);
        else rows(false);
        tap_next(g, tw);
    };
    auto compute = [&](int set) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
            for (int i = 0; i < BM; ++i)
#pragma unroll
                for (int j = 0; j < BN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[set][i][kk], b[set][j][kk], acc[i][j], 0, 0, 0);
    };
    int grp = glo;
    if (grp < ghi) load(0);
    for (; grp + 2 <= ghi; grp += 2) {
        load(1);
        __builtin_amdgcn_sched_barrier(0);
        compute(0);
        __builtin_amdgcn_sched_barrier(0);
        if (grp + 2 < ghi) load(0);
        __builtin_amdgcn_sched_barrier(0);
        compute(1);
        __builtin_amdgcn_sched_barrier(0);
    }
    if (grp < ghi) compute(0);
}

// The lane's outputs of one position: BM accumulators of one block column hold
// filters m .. m + 4 BM - 1, entry r of accumulator i being filter BM r + i.
template <int BM>
__device__ inline void store_column(float* __restrict__ O, const Geometry& g, int m, int n, const f4 (&v)[BM],
                                    int accumulate, int vec)
{
#pragma unroll
    for (int h = 0; h < BM; ++h) {
        f4 w;
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = v[(4 * h + e) % BM][(4 * h + e) / BM];
        store_block(O, g, m + 4 * h, n, w, accumulate, vec);
    }
}

// The waves of a workgroup side by side (2 x 2), a tile each: contractions too
// short to split.
template <int BM, int BN, bool PAD, bool VECA>
__global__ __launch_bounds__(kThreads) void convgemm_square_kernel(Geometry g, const float* __restrict__ F,
                                                                const float* __restrict__ I, float* __restrict__ O,
                                                                int accumulate, int vec, int mtiles, int ntiles)
{
    constexpr int WM = 16 * BM, WN = 16 * BN;
    // XCD-aware tile order, as in the LDS-staged kernel
    const int T = mtiles * ntiles, T8 = T & ~7, bid = blockIdx.x;
    const int t = bid < T8 ? (bid & 7) * (T8 >> 3) + (bid >> 3) : bid;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m0 = (t % mtiles) * 2 * WM + (wave & 1) * WM;
    const int n0 = (t / mtiles) * 2 * WN + (wave >> 1) * WN;
    f4 acc[BM][BN];
    tap_tile<BM, BN, PAD, VECA>(g, tensor_rsrc(F, g.fbytes), tensor_rsrc(I, g.ibytes), m0, n0, 0, tap_groups(g), acc);
    const int q = (threadIdx.x & 63) >> 4, l16 = threadIdx.x & 15;
#pragma unroll
    for (int j = 0; j < BN; ++j) {
        f4 v[BM];
#pragma unroll
        for (int i = 0; i < BM; ++i) v[i] = acc[i][j];
        store_column<BM>(O, g, m0 + 4 * BM * q, n0 + 16 * j + l16, v, accumulate, vec);
    }
}

// The waves of a workgroup share one 16 BM x 16 BN tile and split its
// contraction.
template <int BM, int BN, bool PAD, bool VECA, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void convgemm_split_kernel(Geometry g, const float* __restrict__ F,
                                                                  const float* __restrict__ I, float* __restrict__ O,
                                                                  int accumulate, int vec, int mtiles, int ntiles)
{
    __shared__ f4 part[WAVES][BN][BM][64];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int T = mtiles * ntiles, T8 = T & ~7, bid = blockIdx.x;
    const int t = bid < T8 ? (bid & 7) * (T8 >> 3) + (bid >> 3) : bid;
    const int m0 = (t % mtiles) * 16 * BM, n0 = (t / mtiles) * 16 * BN;
    const int groups = tap_groups(g);
    f4 acc[BM][BN];
    tap_tile<BM, BN, PAD, VECA>(g, tensor_rsrc(F, g.fbytes), tensor_rsrc(I, g.ibytes), m0, n0, wave * groups / WAVES,
                                (wave + 1) * groups / WAVES, acc);
#pragma unroll
    for (int j = 0; j < BN; ++j)
#pragma unroll
        for (int i = 0; i < BM; ++i) part[wave][j][i][lane] = acc[i][j];
    __syncthreads();
    if (wave < BN) {
        f4 v[BM];
#pragma unroll
        for (int i = 0; i < BM; ++i) {
            v[i] = part[0][wave][i][lane];
#pragma unroll
            for (int w = 1; w < WAVES; ++w) v[i] += part[w][wave][i][lane];
        }
        store_column<BM>(O, g, m0 + 4 * BM * (lane >> 4), n0 + 16 * wave + (lane & 15), v, accumulate, vec);
    }
}

// CONVGEMM by runs of taps (few channels, strided, no padding: first layers).
// A lane's four contraction rows of a group are four taps y .. y + 3 of one
// (x, c): contiguous in the input, so one 16-byte load replaces four (the
// LDS-staged gather loads every element by itself, and at stride 4 each such
// load spans four times the lines).  Where kh is not a multiple of four the last
// run of a column starts at kh - 4, so that no load leaves its window, and its
// first rows, which the run before it holds, are zeroed in both operands.  Lane
// group q takes run 4 grp + q; a table of the runs' offsets is built in LDS when
// the workgroup starts.  The waves of a workgroup split one 64 x 32 tile's runs,
// as in the channel-block kernels.  Measured: AlexNet's first layer (64 x 93312 x
// 363, stride 4) 59 -> 49 us, 16 x 16 patches (768 x 12544 x 768) 229 -> 129 us.
// What bounds it, on that first layer: the matrix instructions (46.6 us without
// the loads, 23 with the loads alone; 31 at the matrix rate, one product in eleven
// of them padding: 11 taps to 12, 99 runs to 100) and what does not overlap with
// them, 10.8 us of launch, partial sums and stores; table and exchange cost under
// 0.5 us each.
struct Run {
    uint32_t f, i;     // byte offsets of its first row in F and of its first tap in I
    int skip;          // rows left out at its front: 0 to 3, or 4 past the last run
    int pad;
};
template <int BM, int BN, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void convgemm_runs_kernel(Geometry g, const float* __restrict__ F,
                                                                   const float* __restrict__ I, float* __restrict__ O,
                                                                   int accumulate, int vec, int mtiles, int ntiles)
{
    static_assert(WAVES >= BN, "each column of the tile is stored by a wave of its own");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int nyq = (g.kh + 3) / 4, nruns = nyq * g.kw * g.ci, groups = (nruns + 3) / 4;
    Run* runs = reinterpret_cast<Run*>(smem);
    f4* part = reinterpret_cast<f4*>(smem + (size_t)groups * 4 * sizeof(Run));   // [WAVES][BN][BM][64]
    for (int r = threadIdx.x; r < groups * 4; r += 64 * WAVES) {
        Run v{kOutside, kOutside, 4, 0};
        if (r < nruns) {
            const int xc = r / nyq, y4 = 4 * (r - xc * nyq), y = min(y4, g.kh - 4), c = xc / g.kw, x = xc - c * g.kw;
            v.f = (uint32_t)(y + g.kh * xc) * g.M * 4u;
            v.i = (uint32_t)(y + g.hi * x + g.hiwi * c) * 4u;
            v.skip = y4 - y;
        }
        runs[r] = v;
    }
    __syncthreads();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int q = lane >> 4, l16 = lane & 15;
    const int T = mtiles * ntiles, T8 = T & ~7, bid = blockIdx.x;
    const int t = bid < T8 ? (bid & 7) * (T8 >> 3) + (bid >> 3) : bid;
    const int m0 = (t % mtiles) * 16 * BM, n0 = (t / mtiles) * 16 * BN;
    const __amdgpu_buffer_rsrc_t frs = tensor_rsrc(F, g.fbytes), irs = tensor_rsrc(I, g.ibytes);
    // the filter count is a multiple of BM (the caller's rule: wide loads);
    // filters and positions past the edge are clamped: they only feed outputs
    // that are never stored
    const uint32_t aoff = (uint32_t)min(m0 + BM * l16, g.M - BM) * 4u;
    uint32_t coff[BN];
#pragma unroll
    for (int j = 0; j < BN; ++j) {
        const int n = min(n0 + 16 * j + l16, g.N - 1);
        const int nb = n / g.hw, rem = n - nb * g.hw, ow = rem / g.ho, oh = rem - ow * g.ho;
        coff[j] = (uint32_t)(nb * g.sample + oh * g.s + (int64_t)g.hi * (ow * g.s)) * 4u;
    }
    f4 acc[BM][BN];
#pragma unroll
    for (int i = 0; i < BM; ++i)
#pragma unroll
        for (int j = 0; j < BN; ++j) acc[i][j] = f4{0.0f, 0.0f, 0.0f, 0.0f};
    float a[2][BM][4];
    f4 b[2][BN];
    int skip[2];
    auto load = [&](int grp, int set) {
        const Run r = runs[4 * grp + q];
        skip[set] = r.skip;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            const uint32_t row = r.f + (uint32_t)kk * g.M * 4u;
            load_filters<BM>(a[set], kk, frs, kk >= r.skip ? aoff + row : kOutside, 0u);
        }
#pragma unroll
        for (int j = 0; j < BN; ++j)
            b[set][j] = __builtin_bit_cast(
                f4, __builtin_amdgcn_raw_buffer_load_b128(irs, (int)(r.skip < 4 ? coff[j] + r.i : kOutside), 0, 0));
    };
    auto compute = [&](int set) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            float bv[BN];
#pragma unroll
            for (int j = 0; j < BN; ++j) bv[j] = kk >= skip[set] ? b[set][j][kk] : 0.0f;
#pragma unroll
            for (int i = 0; i < BM; ++i)
#pragma unroll
                for (int j = 0; j < BN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[set][i][kk], bv[j], acc[i][j], 0, 0, 0);
        }
    };
    int grp = wave * groups / WAVES;
    const int ghi = (wave + 1) * groups / WAVES;
    if (grp < ghi) load(grp, 0);
    for (; grp + 2 <= ghi; grp += 2) {
        load(grp + 1, 1);
        __builtin_amdgcn_sched_barrier(0);
        compute(0);
        __builtin_amdgcn_sched_barrier(0);
        if (grp + 2 < ghi) load(grp + 2, 0);
        __builtin_amdgcn_sched_barrier(0);
        compute(1);
        __builtin_amdgcn_sched_barrier(0);
    }
    if (grp < ghi) compute(0);
#pragma unroll
    for (int j = 0; j < BN; ++j)
#pragma unroll
        for (int i = 0; i < BM; ++i) part[((wave * BN + j) * BM + i) * 64 + lane] = acc[i][j];
    __syncthreads();
    if (wave < BN) {
        f4 v[BM];
#pragma unroll
        for (int i = 0; i < BM; ++i) {
            v[i] = part[(wave * BM + i) * 64 + lane];
#pragma unroll
            for (int w = 1; w < WAVES; ++w) v[i] += part[((w * BN + wave) * BM + i) * 64 + lane];
        }
        store_column<BM>(O, g, m0 + 4 * BM * q, n0 + 16 * wave + l16, v, accumulate, vec);
    }
}

int out_size(int h, int k, int s, int p)
{
    if (k < 1 || s < 1 || p < 0 || h < 1) return -1;
    const int64_t span = (int64_t)h - k + 2 * (int64_t)p;
    if (span < 0) return -1;
    return (int)(span / s + 1);
}

struct Tile {
    int mt, nt;
};

// Tile choice (measured on the AlexNet layers): 128 x 128 tiles when the
// filter count is a multiple of 128 and they still give at least four
// workgroups per compute unit; otherwise 64 x 64 tiles, whose small register
// and LDS footprint keeps four or more workgroups resident per compute unit.
Tile choose_tile(int M, int N, int cus)
{
    const int64_t t128 = (int64_t)((M + 127) / 128) * ((N + 127) / 128);
    if (M % 128 == 0 && t128 >= 4 * (int64_t)cus) return Tile{128, 128};
    return Tile{64, 64};
}

// KC: 32-row chunks when the grid is short (fewer than four tiles per compute
// unit: long contractions over few output positions, where fewer and larger
// chunks pay), else 16-row chunks (smaller LDS footprint, more resident
// workgroups).
template <int MT, int NT>
hipError_t launch(const Geometry& g, const float* F, const float* I, float* O, int accumulate, int vec,
                  int cus, hipStream_t stream)
{
    const int mtiles = (g.M + MT - 1) / MT;
    const int ntiles = (g.N + NT - 1) / NT;
    const int64_t tiles = (int64_t)mtiles * ntiles;
    if (tiles > 0x7fffffff) return hipErrorInvalidConfiguration;
    const bool long_k = tiles < 4 * (int64_t)cus;
    const dim3 grid((unsigned)tiles), block(kThreads);
    if (g.p == 0 && !long_k)
        hipLaunchKernelGGL((convgemm_kernel<MT, NT, false, 16>), grid, block, 0, stream, g, F, I, O, accumulate, vec,
                           mtiles, ntiles);
    else if (g.p == 0)
        hipLaunchKernelGGL((convgemm_kernel<MT, NT, false, 32>), grid, block, 0, stream, g, F, I, O, accumulate, vec,
                           mtiles, ntiles);
    else if (!long_k)
        hipLaunchKernelGGL((convgemm_kernel<MT, NT, true, 16>), grid, block, 0, stream, g, F, I, O, accumulate, vec,
                           mtiles, ntiles);
    else
        hipLaunchKernelGGL((convgemm_kernel<MT, NT, true, 32>), grid, block, 0, stream, g, F, I, O, accumulate, vec,
                           mtiles, ntiles);
    return hipGetLastError();
}

// kparts: workgroups sharing one tile's contraction (atomic adds into O)
template <int BM, int BN>
hipError_t launch_direct(const Geometry& g, const float* F, const float* I, float* O, int accumulate, int vec,
                         int kparts, hipStream_t stream)
{
    const int mtiles = (g.M + 32 * BM - 1) / (32 * BM);
    const int ntiles = (g.N + 32 * BN - 1) / (32 * BN);
    const int64_t tiles = (int64_t)mtiles * ntiles;
    if (tiles * kparts > 0x7fffffff) return hipErrorInvalidConfiguration;
    const int kpad = (g.K + 15) / 16 * 16;
    if (kparts > 1 && !accumulate) {
        const int64_t count = (int64_t)g.M * g.N;
        const int64_t blocks = std::min<int64_t>((count + 255) / 256, 4096);
        hipLaunchKernelGGL(zero_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, O, count);
    }
    if (kparts > 1)
        hipLaunchKernelGGL((convgemm_direct_kernel<BM, BN, true>), dim3((unsigned)(tiles * kparts)), dim3(kThreads),
                           (size_t)kpad * sizeof(int), stream, g, F, I, O, accumulate, vec, mtiles, ntiles, kpad, kparts);
    else
        hipLaunchKernelGGL((convgemm_direct_kernel<BM, BN, false>), dim3((unsigned)tiles), dim3(kThreads),
                           (size_t)kpad * sizeof(int), stream, g, F, I, O, accumulate, vec, mtiles, ntiles, kpad, 1);
    return hipGetLastError();
}

template <int BM, int BN>
hipError_t launch_square(const Geometry& g, const float* F, const float* I, float* O, int accumulate, int vec,
                      hipStream_t stream)
{
    const int mtiles = (g.M + 32 * BM - 1) / (32 * BM), ntiles = (g.N + 32 * BN - 1) / (32 * BN);
    const int64_t tiles = (int64_t)mtiles * ntiles;
    if (tiles > 0x7fffffff) return hipErrorInvalidConfiguration;
    const dim3 grid((unsigned)tiles), block(kThreads);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, block, 0, stream, g, F, I, O, accumulate, vec, mtiles, ntiles);
    };
    const bool veca = g.M % BM == 0;
    if (g.p == 0 && veca) go(convgemm_square_kernel<BM, BN, false, true>);
    else if (g.p == 0) go(convgemm_square_kernel<BM, BN, false, false>);
    else if (veca) go(convgemm_square_kernel<BM, BN, true, true>);
    else go(convgemm_square_kernel<BM, BN, true, false>);
    return hipGetLastError();
}

template <int BM, int BN, int WAVES>
hipError_t launch_split(const Geometry& g, const float* F, const float* I, float* O, int accumulate, int vec,
                      hipStream_t stream)
{
    const int mtiles = (g.M + 16 * BM - 1) / (16 * BM), ntiles = (g.N + 16 * BN - 1) / (16 * BN);
    const int64_t tiles = (int64_t)mtiles * ntiles;
    if (tiles > 0x7fffffff) return hipErrorInvalidConfiguration;
    const dim3 grid((unsigned)tiles), block(64 * WAVES);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, block, 0, stream, g, F, I, O, accumulate, vec, mtiles, ntiles);
    };
    const bool veca = g.M % BM == 0;
    if (g.p == 0 && veca) go(convgemm_split_kernel<BM, BN, false, true, WAVES>);
    else if (g.p == 0) go(convgemm_split_kernel<BM, BN, false, false, WAVES>);
    else if (veca) go(convgemm_split_kernel<BM, BN, true, true, WAVES>);
    else go(convgemm_split_kernel<BM, BN, true, false, WAVES>);
    return hipGetLastError();
}

// runs of four taps in a contraction
size_t run_count(const Geometry& g) { return (size_t)((g.kh + 3) / 4) * g.kw * g.ci; }

template <int BM, int BN, int WAVES>
hipError_t launch_runs(const Geometry& g, const float* F, const float* I, float* O, int accumulate, int vec,
                       hipStream_t stream)
{
    const int mtiles = (g.M + 16 * BM - 1) / (16 * BM), ntiles = (g.N + 16 * BN - 1) / (16 * BN);
    const int64_t tiles = (int64_t)mtiles * ntiles;
    if (tiles > 0x7fffffff) return hipErrorInvalidConfiguration;
    const size_t lds = (run_count(g) + 3) / 4 * 4 * sizeof(Run) + (size_t)WAVES * BN * BM * 64 * sizeof(f4);
    const dim3 grid((unsigned)tiles), block(64 * WAVES);
    hipLaunchKernelGGL((convgemm_runs_kernel<BM, BN, WAVES>), grid, block, lds, stream, g, F, I, O, accumulate, vec,
                       mtiles, ntiles);
    return hipGetLastError();
}

// What is launched: the kernel family (the codes of convgemm_choice), its tile,
// and how many workgroups (register-direct) or waves of a workgroup (channel
// blocks, runs) share one tile's contraction.
enum Family { kStaged = 1, kDirect = 2, kBlocks = 3, kRuns = 4 };
struct Choice {
    int family, mt, nt, share;
};

int64_t tile_count(const Geometry& g, int mt, int nt)
{
    return (int64_t)((g.M + mt - 1) / mt) * ((g.N + nt - 1) / nt);
}

// Register-direct tile, measured on the AlexNet layers: 64 x 128 while that
// still gives four tiles per CU; 128 x 64 for filter counts divisible by 128
// with at least 1.5 tiles per CU; 64 x 64 otherwise.  Grids short even with the
// smallest tile, and long contractions: the contraction of each tile is split
// over several workgroups (atomic adds into O) so that every CU holds about
// three, each part keeping at least 64 groups of 16 (608 tiles of 256 x 9680 x
// 3456: 0.227 -> 0.209 ms; 456 larger tiles were slower so).  By itself the library
// comes here with few channels and large taps.
Choice direct_choice(const Geometry& g, int cus)
{
    if (tile_count(g, 64, 128) >= 4 * (int64_t)cus) return Choice{kDirect, 64, 128, 1};
    if (g.M % 128 == 0 && 2 * tile_count(g, 128, 64) >= 3 * (int64_t)cus) return Choice{kDirect, 128, 64, 1};
    int kparts = 1;
    const int64_t tl = tile_count(g, 64, 64);
    const int ngroups = (g.K + 15) / 16;
    while (kparts < 4 && tl * kparts < 3 * (int64_t)cus && ngroups / (2 * kparts) >= 64) kparts *= 2;
    return Choice{kDirect, 64, 64, kparts};
}

Choice staged_choice(const Geometry& g, int cus)
{
    const Tile t = choose_tile(g.M, g.N, cus);
    return Choice{kStaged, t.mt, t.nt, 1};
}

// Tile and split of the channel-block kernels, by the estimated time of the
// grid: rounds of tiles over the CUs, times the tile's size, over the share of
// the matrix rate that the tile shape reached in measurements of 21 layers
// (GEMM N from 121 to 208080, K from 64 to 12544; the model's choice was within
// 7 % of the best shape on each).  Wide loads of the filters need kn to be a
// multiple of BM, which costs the 64-filter tiles most.
Choice blocks_choice(const Geometry& g, int cus)
{
    const int groups = tap_groups(g);
    auto cost = [&](int mt, int nt, double rate) {
        return (double)((tile_count(g, mt, nt) + cus - 1) / cus) * mt * nt / rate;
    };
    // eight or fewer groups: one wave's worth, four tiles side by side instead
    // (256 x 100352 x 64: 43 against 54 us) while they fill the chip
    if (groups <= 8 && tile_count(g, 64, 128) >= 4 * (int64_t)cus) return Choice{kBlocks, 64, 128, 1};
    const double wide = g.M % 4 == 0 ? 0.85 : 0.55;
    const double c42 = cost(64, 32, wide), c41 = cost(64, 16, wide - 0.10), c22 = cost(32, 32, g.M % 2 == 0 ? 0.68 : 0.62),
                 c24 = cost(32, 64, 0.72), c11 = cost(16, 16, 0.42);
    const double best = std::min({c42, c41, c22, c24, c11});
    // eight waves instead of four where that many more are needed to cover the
    // loads' latency: few tiles per CU, long contractions
    if (c42 == best)
        return Choice{kBlocks, 64, 32, groups >= 64 && tile_count(g, 64, 32) < 6 * (int64_t)cus ? 8 : 4};
    if (c41 == best) return Choice{kBlocks, 64, 16, tile_count(g, 64, 16) <= 2 * (int64_t)cus ? 8 : 4};
    if (c22 == best) return Choice{kBlocks, 32, 32, 8};
    if (c24 == best) return Choice{kBlocks, 32, 64, 8};
    return Choice{kBlocks, 16, 16, 16};
}

// Estimated time of a choice in microseconds, to compare the channel-block
// kernels with the general ones: rounds of tiles over the CUs, each a fixed part
// (`tile`) and a part per 16 rows of the contraction (`group`), slower where
// filters are loaded one by one (`narrow`), where padding is checked per element
// (`pad`) and where neighbouring positions lie apart in the input (`strided`);
// `store` is added per MB of outputs stored one by one (kn no multiple of 4); at
// least a launch's latency and the tensors' traffic (10 TB/s, caches included).
// The constants are fits to the times of every kernel on 13130 layers (kn 1 to
// 1500, K 11 to 124000, N 1 to 2.4 10^6; errors of 4 to 19 % root mean square).
struct Rate {
    int family, mt, nt, share;
    double tile, group, narrow, pad, strided, store;
};
constexpr Rate kRates[] = {
    {kBlocks, 64, 128, 1, 1.08, 0.631, 0.11, 0, 0.058, 0.53}, {kBlocks, 64, 32, 4, 0.63, 0.151, 0.69, 0, 0.039, 0.67},
    {kBlocks, 64, 32, 8, 1.39, 0.138, 0.69, 0, 0.036, 0.63},  {kBlocks, 64, 16, 4, 0.27, 0.084, 0.99, 0, 0.063, 0.85},
    {kBlocks, 64, 16, 8, 0.63, 0.080, 1.05, 0, 0.048, 0.61},  {kBlocks, 32, 32, 8, 0.61, 0.085, 0.29, 0, 0.115, 0.18},
    {kBlocks, 32, 64, 8, 1.48, 0.156, 0.13, 0, 0.096, 0.29},  {kBlocks, 16, 16, 16, 0.87, 0.037, 0, 0, 0.125, 0.28},
    {kDirect, 64, 128, 1, 1.43, 0.534, 0, 0, 0, 0.31},        {kDirect, 128, 64, 1, 1.70, 0.561, 0, 0, 0, 0.30},
    {kDirect, 64, 64, 1, 0.31, 0.369, 0, 0, 0, 0.42},         {kStaged, 128, 128, 1, 2.19, 1.217, 0, 0.17, 0, 0.30},
};
// its contraction shared with atomic adds; the LDS-staged 64 x 64 tile in chunks
// of 32 (short grids) and 16 rows
constexpr Rate kDirectShared = {kDirect, 64, 64, 0, 0.68, 0.372, 0, 0, 0, 1.56};
constexpr Rate kStagedLong = {kStaged, 64, 64, 1, 0.36, 0.463, 0, 0.31, 0, 0.34};
constexpr Rate kStagedShort = {kStaged, 64, 64, 1, 0.54, 0.373, 0, 0.26, 0, 0.24};

double estimate(const Geometry& g, const Choice& c, int cus)
{
    const int64_t tiles = tile_count(g, c.mt, c.nt) * (c.family == kDirect ? c.share : 1);
    const Rate* r = &kRates[0];
    if (c.family == kDirect && c.share > 1) r = &kDirectShared;
    else if (c.family == kStaged && c.mt == 64) r = tiles < 4 * (int64_t)cus ? &kStagedLong : &kStagedShort;
    else
        for (const Rate& x : kRates)
            if (x.family == c.family && x.mt == c.mt && x.nt == c.nt && x.share == c.share) r = &x;
    const bool blocks = c.family == kBlocks;
    const double groups = blocks ? tap_groups(g) : (double)((g.K + 15) / 16) / (c.family == kDirect ? c.share : 1);
    const int wide = c.nt == 128 ? 2 : c.mt / 16;            // filters a lane loads at once
    double slow = 1.0 + (g.p > 0 ? r->pad : 0.0);
    if (blocks && g.M % wide != 0) slow += r->narrow;
    if (g.s > 1) slow *= 1.0 + r->strided * (g.s - 1 + std::max(0.0, 16.0 / g.ho - 1.0));
    const double used = 0.85 + 0.15 * std::min(g.M, c.mt) / c.mt;   // filters past kn load the same bytes
    const double out_mb = 4e-6 * g.M * (double)g.N;
    double work = (double)((tiles + cus - 1) / cus) * (r->tile + r->group * groups * slow * used);
    if (g.M % 4 != 0) work += r->store * out_mb;
    double lat = 5.2;
    if (c.family == kStaged) lat = 3.0 + (r == &kStagedLong ? 0.54 : 1.5) * groups;
    if (blocks && c.share == 1) lat += 0.5 * groups;
    if (r == &kDirectShared) work += 1.6 * out_mb + 4.0;             // O cleared first, then atomic adds
    const double mem = 0.1 * (1e-6 * ((double)g.ibytes + (double)g.fbytes) + out_mb);
    return std::max({work, lat, mem});
}

// The automatic choice.
Choice choose(const Geometry& g, int cus)
{
    // without padding and at unit stride the register-direct kernel (the im2col
    // columns of neighbouring positions are then contiguous input runs that the
    // caches serve well); the LDS-staged gather otherwise (measured: the direct
    // kernel is slower at stride 4, where each load instruction spans four times
    // the lines) and for contractions longer than the direct kernel's row table
    const bool direct = g.p == 0 && g.s == 1 && g.K <= kDirectMaxK;
    const Choice general = direct ? direct_choice(g, cus) : staged_choice(g, cus);
    if (g.ibytes > kOutside || g.fbytes > kOutside) return general;
    // enough channels that blocks of 16 waste no more than a third of the
    // products (three channels would run at a fifth): the channel-block kernels.
    // With whole blocks, wide filter loads and more than 16 groups they are the
    // faster ones (2379 measured layers: 0.32 of the general kernel's time in the
    // mean, none slower by more than 12 %).  Elsewhere the estimates decide: a
    // contraction of a few groups leaves the waves that share a tile without work
    // (16 x 125440 x 16: 35 against 7.5 us general), partial blocks and filters
    // loaded one by one cost too much on many tiles (33 x 125440 x 64: 35 against
    // 20), and so do wide strides (298 x 4290 x 160, stride 4: 19.2 against 14.3).
    // Over 13130 measured layers the blocks alone took 0.515 of the general
    // kernels' time in the mean but were slower by more than 4 % on 1207 of them;
    // with this rule 0.501, and on 127.  With a partial block and a large unpadded
    // grid at unit stride the register-direct kernel, which wastes no products, is
    // faster (256 x 102660 x 297, 33 channels: 144 against 217 us).
    const bool large = tile_count(g, 64, 128) >= 4 * (int64_t)cus;
    if ((g.ci + 15) / 16 * 16 * 2 <= 3 * g.ci) {
        if (g.ci % 16 != 0 && direct && large) return general;
        const Choice blocks = blocks_choice(g, cus);
        if (g.ci % 16 == 0 && g.M % 4 == 0 && tap_groups(g) > 16) return blocks;
        return estimate(g, general, cus) < estimate(g, blocks, cus) ? general : blocks;
    }
    // few channels, strided and not padded, a tap height that runs of four cover
    // with at most a third of waste, filters in wide loads, and a contraction of
    // at least 64 taps whose table fits LDS: the runs kernel.  Old path against it:
    // kh = 5 (two runs for five taps, 64 x 14400 x 250) 13 against 17 us, an odd
    // filter count (33 x 61504 x 75) 16 against 21, 48 taps (384 x 63504) 39
    // against 39; stride 1 (7 x 7, 64 x 131072 x 147) 31 against 35, where the
    // register-direct kernel reads contiguous runs already.  Four waves share the
    // contraction from 16 groups on (64 x 46656 x 363: 33 us before, 31 with two
    // waves, 26 with four), two below (64 x 190096 x 147: 52, 46, 49).  The general
    // kernel's 128 x 128 tiles are faster where the runs waste more than a seventh
    // (384 x 130200 x 243, kh = 9: 258 against 316; 640 x 91250 x 288, kh = 6: 371,
    // 446), and slower with less waste (medians of 20 layers each: kh = 6, 9, 10 the
    // runs take 1.08, 1.09, 1.01 of their time, kh = 7, 11, 8 0.92, 0.94, 0.88).
    const size_t nruns = run_count(g);
    const bool wasteful = 7 * ((g.kh + 3) / 4 * 4) > 8 * g.kh;
    if (general.mt == 128 && wasteful) return general;
    if (g.p == 0 && g.s > 1 && g.M % 4 == 0 && g.kh >= 4 && g.kh != 5 && nruns >= 16 && nruns <= 2048)
        return Choice{kRuns, 64, 32, nruns > 60 ? 4 : 2};
    return general;
}

hipError_t launch_choice(const Geometry& g, const Choice& c, const float* F, const float* I, float* O, int accumulate,
                         int vec, int cus, hipStream_t stream)
{
    switch (c.family) {
    case kBlocks:
        if (c.nt == 128) return launch_square<2, 4>(g, F, I, O, accumulate, vec, stream);
        if (c.mt == 64 && c.nt == 32)
            return c.share == 8 ? launch_split<4, 2, 8>(g, F, I, O, accumulate, vec, stream)
                                : launch_split<4, 2, 4>(g, F, I, O, accumulate, vec, stream);
        if (c.mt == 64)
            return c.share == 8 ? launch_split<4, 1, 8>(g, F, I, O, accumulate, vec, stream)
                                : launch_split<4, 1, 4>(g, F, I, O, accumulate, vec, stream);
        if (c.mt == 32)
            return c.nt == 32 ? launch_split<2, 2, 8>(g, F, I, O, accumulate, vec, stream)
                              : launch_split<2, 4, 8>(g, F, I, O, accumulate, vec, stream);
        return launch_split<1, 1, 16>(g, F, I, O, accumulate, vec, stream);
    case kRuns:
        return c.share == 4 ? launch_runs<4, 2, 4>(g, F, I, O, accumulate, vec, stream)
                            : launch_runs<4, 2, 2>(g, F, I, O, accumulate, vec, stream);
    case kDirect:
        if (c.mt == 64)
            return c.nt == 64 ? launch_direct<2, 2>(g, F, I, O, accumulate, vec, c.share, stream)
                              : launch_direct<2, 4>(g, F, I, O, accumulate, vec, 1, stream);
        return c.nt == 64 ? launch_direct<4, 2>(g, F, I, O, accumulate, vec, 1, stream)
                          : launch_direct<4, 4>(g, F, I, O, accumulate, vec, 1, stream);
    default:
        if (c.mt == 64 && c.nt == 64) return launch<64, 64>(g, F, I, O, accumulate, vec, cus, stream);
        if (c.mt == 64 && c.nt == 128) return launch<64, 128>(g, F, I, O, accumulate, vec, cus, stream);
        if (c.mt == 64) return launch<64, 256>(g, F, I, O, accumulate, vec, cus, stream);
        if (c.mt == 128) return launch<128, 128>(g, F, I, O, accumulate, vec, cus, stream);
        return launch<192, 128>(g, F, I, O, accumulate, vec, cus, stream);
    }
}

int device_cus()
{
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 256;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
        return 256;
    return cus;
}

}  // namespace
}  // namespace convgemm

extern "C" int convgemm_out_size(int h, int k, int stride, int pad)
{
    return convgemm::out_size(h, k, stride, pad);
}

namespace convgemm {
namespace {

// The layer's geometry, or -i when argument i is out of range (b = 0 leaves g
// without output positions).
int make_geometry(int kn, int kh, int kw, int ci, int hi, int wi, int b, int stride, int pad, Geometry& g)
{
    if (kn < 1) return -1;
    if (kh < 1) return -2;
    if (kw < 1) return -3;
    if (ci < 1) return -4;
    if (hi < 1) return -5;
    if (wi < 1) return -6;
    if (b < 0) return -7;
    if (stride < 1) return -8;
    if (pad < 0) return -9;
    const int ho = out_size(hi, kh, stride, pad);
    const int wo = out_size(wi, kw, stride, pad);
    if (ho < 1) return -5;
    if (wo < 1) return -6;
    if ((int64_t)hi * wi * ci >= ((int64_t)1 << 31)) return -5;
    if ((int64_t)kh * kw * ci >= ((int64_t)1 << 31)) return -2;
    if ((int64_t)ho * wo * b >= ((int64_t)1 << 31)) return -7;
    if ((int64_t)hi * wi * ci * b >= ((int64_t)1 << 30)) return -7;
    if (kn >= (1 << 24) || (int64_t)kn * kh * kw * ci >= ((int64_t)1 << 30)) return -1;
    g.M = kn;
    g.K = kh * kw * ci;
    g.ci = ci;
    g.N = ho * wo * b;
    g.kh = kh;
    g.kw = kw;
    g.khw = kh * kw;
    g.hi = hi;
    g.wi = wi;
    g.hiwi = hi * wi;
    g.ho = ho;
    g.hw = ho * wo;
    g.s = stride;
    g.p = pad;
    g.sample = (int64_t)hi * wi * ci;
    g.ibytes = (uint32_t)(g.sample * b * 4);
    g.fbytes = (uint32_t)((int64_t)kn * g.K * 4);
    return CONVGEMM_OK;
}

}  // namespace
}  // namespace convgemm

extern "C" int convgemm_choice(int kn, int kh, int kw, int ci, int hi, int wi, int b, int stride, int pad, int* out)
{
    using namespace convgemm;
    Geometry g;
    const int r = make_geometry(kn, kh, kw, ci, hi, wi, b, stride, pad, g);
    if (r != CONVGEMM_OK) return r;
    if (!out) return -10;
    const Choice c = b == 0 ? Choice{0, 0, 0, 0} : choose(g, device_cus());
    out[0] = c.family;
    out[1] = c.mt;
    out[2] = c.nt;
    out[3] = c.share;
    return CONVGEMM_OK;
}

extern "C" int convgemm_f32(int kn, int kh, int kw, int ci, int hi, int wi, int b, int stride, int pad,
                            const float* F, const float* I, float* O, int accumulate, int path, int mt, int nt,
                            hipStream_t stream)
{
    using namespace convgemm;
    Geometry g;
    const int r = make_geometry(kn, kh, kw, ci, hi, wi, b, stride, pad, g);
    if (r != CONVGEMM_OK) return r;
    if (accumulate != 0 && accumulate != 1) return -13;
    // path: 0 automatic, 1 LDS-staged gather, 2 register-direct (no padding,
    // contraction up to kDirectMaxK rows: its row table lives in LDS)
    if (path < 0 || path > 2 || (path == 2 && (pad != 0 || g.K > kDirectMaxK)) || (path == 0 && (mt || nt)))
        return -14;
    const bool lds_tile = (mt == 64 && (nt == 64 || nt == 128 || nt == 256)) || (mt == 128 && nt == 128) ||
                          (mt == 192 && nt == 128);
    const bool direct_tile = (mt == 64 || mt == 128) && (nt == 64 || nt == 128);
    if (path == 1 && !(lds_tile || (mt == 0 && nt == 0))) return -15;
    if (path == 2 && !(direct_tile || (mt == 0 && nt == 0))) return -15;
    if (b == 0) return CONVGEMM_OK;
    if (!F) return -10;
    if (!I) return -11;
    if (!O) return -12;

    const int vec = (kn % 4 == 0) && ((uintptr_t)O % 16 == 0);
    const int cus = device_cus();
    const Choice c = path == 0   ? choose(g, cus)
                     : mt != 0   ? Choice{path == 1 ? kStaged : kDirect, mt, nt, 1}
                     : path == 1 ? staged_choice(g, cus)
                                 : direct_choice(g, cus);
    const hipError_t e = launch_choice(g, c, F, I, O, accumulate, vec, cus, stream);
    return e == hipSuccess ? CONVGEMM_OK : CONVGEMM_ERR_HIP_BASE - (int)e;
}

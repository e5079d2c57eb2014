// Candidate-batch scoring against latency SLOs on MI355X (gfx950).
//
// Implements the C ABI of include/orloj.h: the hot path of Orloj
// ("Predictably Serving Unpredictable DNNs", arXiv 2209.00159) as
// hand-written HIP kernels for CDNA4:
//
//   cdf_kernel     histogram rows -> 1 - CDF (exact 64-bit running sums)
//   score_kernel   one workgroup per (model, batch size): scan over queue
//                  position of the members' CDF rows into the batch CDF,
//                  E[L_B], finish probabilities and Eq. (2) priorities of
//                  every prefix candidate, all in one pass
//   turned_kernel  the same outputs in launches too small to fill the chip:
//                  a workgroup's waves split the bins, lanes hold prefix
//                  lengths
//   emax_kernel    affine mode: the sums behind E[L_B], once per prefix
//                  length instead of once per batch size
//   select_kernel  one workgroup per model: argmax over its candidates
//
// and, around the path, laws_kernel / iterate_kernel (one Algorithm 1
// iteration with the paper's own priority) and accumulate_kernel (profiler
// samples into the histograms).
//
// The work is a scan plus reductions over HBM-resident tables, not a dense
// contraction, so it runs on the vector ALUs (no MFMA): row loads
// prefetched into registers, fp64 running products, wave64 DPP scans and
// reductions, and LDS for the per-step snapshot the member lookups read.

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdarg.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <mutex>
#include <new>
#include <type_traits>
#include <utility>

#include "../../include/orloj.h"
#include "orloj_ctx.h"

namespace {

constexpr int kThreads = 256;               // 4 wave64 per workgroup
constexpr int kWaves = kThreads / 64;

// Device-side data error bits (reported by orloj_sync as ORLOJ_E_DATA).
constexpr int kErrEmptyHistogram = 1;
constexpr int kErrClassRange = 2;
constexpr int kErrDeadlineNaN = 4;
constexpr int kErrUnsorted = 8;
constexpr int kErrNowNaN = 16;
constexpr int kErrWidth = 32;
constexpr int kErrWeights = 64;
constexpr int kErrCost = 128;
constexpr int kErrAffine = 256;

// ---------------------------------------------------------------------------
// wave64 helpers
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint64_t wave_incl_scan_u64(uint64_t x, int lane) {
#pragma unroll
    for (int s = 1; s < 64; s <<= 1) {
        uint64_t t = __shfl_up(x, s, 64);
        if (lane >= s) x += t;
    }
    return x;
}

// Sum over the wave, in every lane.
__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t x, int lane) {
    const uint64_t s = wave_incl_scan_u64(x, lane);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)s, 63);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(s >> 32), 63);
    return ((uint64_t)hi << 32) | lo;
}

// ---------------------------------------------------------------------------
// cdf_kernel: one workgroup per histogram row.  Thread t owns the VPT
// consecutive bins [t*VPT, t*VPT + VPT): it loads them once, the workgroup
// scans the per-thread sums (64-bit, exact), and each thread writes the
// complementary CDF 1 - F(x_{k+1}) = (total - running sum) / total.  The
// complement keeps full relative precision where F is close to 1, which is
// where the batch CDF (a product over up to hundreds of members) is most
// sensitive.  Optionally the row's support is recorded as well: the first
// bin holding mass (every earlier entry is exactly 1) and the last bin
// holding mass (it and every later entry are exactly 0).
// ---------------------------------------------------------------------------
__device__ __forceinline__ float survival(uint64_t cum, uint64_t tot, double rtot) {
    if (cum >= tot) return 0.0f;
    return (float)((double)(tot - cum) * rtot);
}

__device__ __forceinline__ int wave_min_i32(int x) {
#pragma unroll
    for (int s = 1; s < 64; s <<= 1) x = min(x, __shfl_xor(x, s, 64));
    return x;
}

__device__ __forceinline__ int wave_max_i32(int x) {
#pragma unroll
    for (int s = 1; s < 64; s <<= 1) x = max(x, __shfl_xor(x, s, 64));
    return x;
}

template <int VPT>
__global__ __launch_bounds__(kThreads) void cdf_kernel(const uint32_t* __restrict__ counts,
                                                       float* __restrict__ out,
                                                       int32_t* __restrict__ support, int64_t n_rows,
                                                       int K, int* __restrict__ err) {
    __shared__ uint64_t s_wave[kWaves];
    __shared__ int s_sup[2][kWaves];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int base = tid * VPT;
    const bool vec = (VPT % 4 == 0) && ((K & 3) == 0);
    for (int64_t r = blockIdx.x; r < n_rows; r += gridDim.x) {
        const uint32_t* row = counts + (size_t)r * (size_t)K;
        uint32_t v[VPT];
        if (vec && base + VPT <= K) {
#pragma unroll
            for (int j = 0; j < VPT; j += 4) {
                const uint4 t = *reinterpret_cast<const uint4*>(row + base + j);
                v[j] = t.x; v[j + 1] = t.y; v[j + 2] = t.z; v[j + 3] = t.w;
            }
        } else {
#pragma unroll
            for (int j = 0; j < VPT; ++j) v[j] = (base + j < K) ? row[base + j] : 0u;
        }
        uint64_t local = 0;
#pragma unroll
        for (int j = 0; j < VPT; ++j) local += v[j];
        const uint64_t incl = wave_incl_scan_u64(local, lane);
        if (lane == 63) s_wave[wv] = incl;
        __syncthreads();
        uint64_t off = incl - local, tot = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const uint64_t t = s_wave[w];
            if (w < wv) off += t;
            tot += t;
        }
        float* orow = out + (size_t)r * (size_t)K;
        if (support) {
            // first bin with mass; last bin with mass (K when the row is empty)
            int lo = K, hi = -1;
#pragma unroll
            for (int j = 0; j < VPT; ++j) {
                if (v[j] != 0u) {
                    lo = min(lo, base + j);
                    hi = max(hi, base + j);
                }
            }
            lo = wave_min_i32(lo);
            hi = -wave_min_i32(-hi);
            if (lane == 0) { s_sup[0][wv] = lo; s_sup[1][wv] = hi; }
            __syncthreads();
            if (tid == 0) {
                for (int w = 1; w < kWaves; ++w) {
                    lo = min(lo, s_sup[0][w]);
                    hi = max(hi, s_sup[1][w]);
                }
                support[2 * r] = hi < 0 ? 0 : lo;
                support[2 * r + 1] = hi < 0 ? 0 : hi;
            }
        }
        __syncthreads();   // s_wave and s_sup are reused by the next row
        if (tot == 0) {
            if (tid == 0) atomicOr(err, kErrEmptyHistogram);
#pragma unroll
            for (int j = 0; j < VPT; ++j)
                if (base + j < K) orow[base + j] = NAN;
            continue;
        }
        const double rtot = 1.0 / (double)tot;
        float o[VPT];
        uint64_t cum = off;
#pragma unroll
        for (int j = 0; j < VPT; ++j) {
            cum += v[j];
            o[j] = survival(cum, tot, rtot);
        }
        if (vec && base + VPT <= K) {
#pragma unroll
            for (int j = 0; j < VPT; j += 4)
                *reinterpret_cast<float4*>(orow + base + j) =
                    make_float4(o[j], o[j + 1], o[j + 2], o[j + 3]);
        } else {
#pragma unroll
            for (int j = 0; j < VPT; ++j)
                if (base + j < K) orow[base + j] = o[j];
        }
    }
}

// ---------------------------------------------------------------------------
// DPP building blocks (gfx9 encodings: row_shr:s = 0x110+s, row_bcast:15 =
// 0x142, row_bcast:31 = 0x143).  Lanes without a source read 0.
// ---------------------------------------------------------------------------
template <int CTRL, int ROWMASK = 0xf>
__device__ __forceinline__ float dpp(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
                                         0, __builtin_bit_cast(int, x), CTRL, ROWMASK, 0xf, true));
}

// Inclusive wave64 scan with geometric weights: lane L ends with
// sum_{L' <= L} x_{L'} r^(L - L').  rp[i] = r^(2^i); w15 = r^((L & 15) + 1);
// w31 = r^(L - 31) for lanes >= 32.
// Each stage is x <- x' r + x with x' the DPP-moved x (0 where a lane has no
// source, and rows outside the row mask keep x): one v_fmac_f32 with the
// DPP move on its first source.  The compiler emits a separate move and
// fma per stage, so the stages are written out; a VALU write of a VGPR
// needs two wait states before a DPP read of it (s_nop 1), and the last
// stage is followed by two as well, since the compiler cannot see into the
// block when it places the next reader.
__device__ __forceinline__ float wave_wscan(float x, const float (&rp)[4], float w15, float w31) {
    asm volatile(
        "s_nop 1\n\t"
        "v_fmac_f32_dpp %0, %0, %1 row_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "s_nop 1\n\t"
        "v_fmac_f32_dpp %0, %0, %2 row_shr:2 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "s_nop 1\n\t"
        "v_fmac_f32_dpp %0, %0, %3 row_shr:4 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "s_nop 1\n\t"
        "v_fmac_f32_dpp %0, %0, %4 row_shr:8 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "s_nop 1\n\t"
        "v_fmac_f32_dpp %0, %0, %5 row_bcast:15 row_mask:0xa bank_mask:0xf bound_ctrl:1\n\t"
        "s_nop 1\n\t"
        "v_fmac_f32_dpp %0, %0, %6 row_bcast:31 row_mask:0xc bank_mask:0xf bound_ctrl:1\n\t"
        "s_nop 1"
        : "+v"(x)
        : "v"(rp[0]), "v"(rp[1]), "v"(rp[2]), "v"(rp[3]), "v"(w15), "v"(w31));
    return x;
}

// Inclusive wave64 sum scan: lane 63 ends with the total.
__device__ __forceinline__ float wave_scan_sum(float x) {
    x += dpp<0x111>(x);
    x += dpp<0x112>(x);
    x += dpp<0x114>(x);
    x += dpp<0x118>(x);
    x += dpp<0x142, 0xa>(x);
    x += dpp<0x143, 0xc>(x);
    return x;
}

template <int CTRL, int ROWMASK = 0xf>
__device__ __forceinline__ double dpp64(double x) {
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, ROWMASK, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, ROWMASK, 0xf, true);
    return __builtin_bit_cast(double, ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

// Two wave sums at once.  v_permlane32_swap exchanges the upper half of x
// with the lower half of y, so after one add lane l < 32 holds x_l + x_(l+32)
// and lane l >= 32 holds y_(l-32) + y_l; a DPP sum within each half (rows of
// 16, then row 0 into row 1 and row 2 into row 3) leaves the total of x in
// lane 31 and that of y in lane 63.  Each total comes out of one fixed tree,
// whatever the other value is.
__device__ __forceinline__ float wave_pair_sum(float x, float y) {
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, x),
                                                    __builtin_bit_cast(unsigned, y), false, false);
    float z = __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
    z += dpp<0x111>(z);
    z += dpp<0x112>(z);
    z += dpp<0x114>(z);
    z += dpp<0x118>(z);
    z += dpp<0x142, 0xa>(z);
    return z;
}

__device__ __forceinline__ double wave_pair_sum64(double x, double y) {
    const uint64_t ux = __builtin_bit_cast(uint64_t, x), uy = __builtin_bit_cast(uint64_t, y);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)ux, (unsigned)uy, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(ux >> 32), (unsigned)(uy >> 32), false, false);
    const double a = __builtin_bit_cast(double, ((uint64_t)(unsigned)hi[0] << 32) | (unsigned)lo[0]);
    const double b = __builtin_bit_cast(double, ((uint64_t)(unsigned)hi[1] << 32) | (unsigned)lo[1]);
    double z = a + b;
    z += dpp64<0x111>(z);
    z += dpp64<0x112>(z);
    z += dpp64<0x114>(z);
    z += dpp64<0x118>(z);
    z += dpp64<0x142, 0xa>(z);
    return z;
}

// 2^x by the hardware instruction; results below 2^-126 flush to 0.
__device__ __forceinline__ float exp2_hw(float x) { return __builtin_amdgcn_exp2f(x); }

// ---------------------------------------------------------------------------
// score_kernel
// ---------------------------------------------------------------------------
// Launches over many models of which only a few have a queue (a scheduling
// round scores the idle models only) list those models in their arguments
// and launch workgroups for them alone: workgroups that only find an empty
// queue and exit would still hold the dispatch slots for a memory round
// trip each.
constexpr int kMaxActive = 256;

struct ScoreArgs {
    const float* tab;          // [M][nbs][C][K] 1 - F(x_{k+1})
    const int64_t* queue_off;  // [M+1]
    const int32_t* cls;        // [N]
    const double* deadline;    // [N]
    const double* now;         // [M]
    const double* width;       // [M]
    const int64_t* cand_off;   // [M+1]
    const int64_t* prob_off;   // [M+1]
    float* P;
    double* E;
    float* EL;
    float* S;
    const int32_t* sup;        // [M][nbs][C][2] first / last bin with mass, or NULL
    const double* cost;        // [N] miss cost per request, or NULL (1)
    const double* c0;          // affine mode: [M] fixed batch overhead (ms); else NULL
    const double* c1;          // affine mode: [M] per-member slope; NULL = tabulated mode
    const float* fill;         // [2][16] zeros, ones (the context's stand-in rows)
    float* psum;               // affine mode: [M][np_e][maxcap] panel sums of 1 - G
    int np_e;                  // panels of those sums (emax_kernel's panel width)
    int* err;
    double b;
    int M, C, K, nbs, rect, maxcap;
    int Mg;                    // models the grid covers: M, or the listed ones
    int compact;               // 1: grid model i is act[i]
    int bs[ORLOJ_MAX_BATCH_SIZES];
    int act[kMaxActive];       // the models with a non-empty queue (compact)
};

__device__ __forceinline__ int grid_model(const ScoreArgs& a, unsigned i) {
    return a.compact ? a.act[i] : (int)i;
}

// Stand-in rows for lane chunks that lie wholly outside a row's support:
// there every entry of 1 - F is exactly 0 (past the last bin with mass) or
// exactly 1 (before the first), so the update G <- G - G (1 - F) gives the
// same bits whether it reads the table or these constants.  They live in a
// small buffer of the context (kFillFloats floats: 16 zeros, then 16 ones),
// stay in cache, and keep every row load a plain global load.
constexpr int kFillFloats = 32;

// Per-member lookup plan (it depends on the deadline only, not on the step).
//
// The bins are swept in panels of 64 CPL bins (one chunk of CPL
// consecutive bins per lane); a member with deadline bin k is handled in the
// pass over its home panel hp (the panel of bin k; dead requests in pass 0,
// beyond-the-grid requests in the last pass).  Deadline order makes the
// members of each panel a contiguous range.  In that pass, at step n, the
// wave has
//   W     = Z at the last bin of panel hp-1   (discounted prefix carried in)
//   gl    = G at the last bin of panel hp-1
//   A[]   = in-panel discounted scan of the lane chunk totals
//   g[], zq[]  snapshot of G (fp64) and of each chunk's quarter-end prefixes
// and assembles
//   G(x_k)     = g[o0]
//   G(x_{k+1}) = g[o1]
//   Z(k-2) = cW W + cG gl + cA f[oa] + fq f[oz] + z4
//   z4     = the in-quarter discounted prefix of g[o4 + 0 .. rq] (Horner)
//   P   = G(x_k) + theta (G(x_{k+1}) - G(x_k))          (fp64)
//   num = cg (G(x_k) - (1 - d) Z(k-2)) + psi (G(x_{k+1}) - G(x_k))
// where g is the fp64 area of the workgroup's LDS (the snapshot and three
// constant slots: 0, 1 and gl, the last written at every scoring step) and
// f its float area (zq, A and a zero).  The plan resolves every case into an
// offset: G(x_k) is gl when bin k-1 lies in the previous panel, 0 when
// k = 0; both G values are 0 when the deadline has passed and 1 when it lies
// beyond the grid; a term the member does not need has weight 0 and reads a
// finite slot.  So the lookup takes no branch.  P and the expected finish
// count are formed in fp64 from the fp64 snapshot and an fp64 theta (a
// float pair); the priority's terms are fp32.  A plan is 48 bytes, so that
// 64 of them and the fp64 snapshot of a 1024-bin panel leave room for
// twelve waves per compute unit.
constexpr int kMaxPanels = 63;   // panels per row (their first members sit in one lane each)

struct Member {
    uint8_t hp;     // home panel
    uint8_t rq;     // bin k-2's place in its quarter (kNoQuarter: no quarter term)
    uint16_t o0;    // LDS byte offsets of G(x_k),
    uint16_t o1;    //   G(x_{k+1}),
    uint16_t o4;    //   the quarter holding bin k-2,
    uint16_t oz;    //   the quarter-end prefix before that quarter,
    uint16_t oa;    //   and the in-panel scan before bin k-2's lane
    float cW;       // weight of W
    float cG;       // weight of gl
    float cA;       // weight of f[oa]
    float fq;       // weight of f[oz]
    float theta;    // position inside bin k (rounded to fp32) ...
    float thlo;     //   ... and the rest of the fp64 position
    float cg;       // gamma exp(-b theta w), or gamma exp(-b (tau - K w))
    float psi;      // (1 - exp(-b theta w)) / (b w)
    float cost;     // the request's miss cost (weights its priority)
};
static_assert(sizeof(Member) == 48, "member plan size");
constexpr int kNoQuarter = 0xff;

template <int CPL>
struct Quarters {
    static constexpr int QW = CPL < 4 ? CPL : 4;   // bins per quarter
    static constexpr int NQ = CPL / QW;            // quarters per lane chunk
};

// LDS layout of one workgroup (one wave), byte offsets:
//   GD  g[64 CPL]   snapshot of G over the current panel, fp64; pairs of
//                   bins interleaved over the lanes, bins j, j+1 of lane l
//                   at pair slot 64 (j/2) + (l ^ (j/2)): a lane writes 16
//                   consecutive bytes, each write is a permutation of 64
//                   consecutive slots, and the members that read the
//                   different pairs of one lane chunk hit different banks
//   KD  k[4]        constant slots (fp64): 0, 1, gl (G carried in), unused
//   ZQ  zq[64 NQ]   quarter-end discounted prefixes of each lane chunk (f32)
//   AA  A[64]       in-panel discounted scan of the lane chunk totals (f32)
//   FZ  4 zeros     (f32) what a weight-0 float term reads
//   MEM mem[maxcap] Member plans
template <int CPL>
struct ScoreLds {
    static constexpr int GD = 0;
    static constexpr int KD = 8 * 64 * CPL;
    static constexpr int ZQ = KD + 32;
    static constexpr int AA = ZQ + 4 * 64 * Quarters<CPL>::NQ;
    static constexpr int FZ = AA + 4 * 64;
    static constexpr int MEM = FZ + 16;
    static_assert(MEM % 16 == 0 && MEM < 65536, "LDS layout");
};
template <int CPL>
__host__ __device__ constexpr size_t score_fixed_bytes() { return (size_t)ScoreLds<CPL>::MEM; }
__host__ __device__ constexpr size_t score_bytes_per_member() { return sizeof(Member); }

// Byte offset of the snapshot's bin r (bin offset inside the panel).
template <int CPL>
__device__ __forceinline__ int snap_byte(int r) {
    if constexpr (CPL >= 2) {
        const int l = r / CPL, j = r - l * CPL, jp = j >> 1;
        return 8 * ((jp * 64 + (l ^ jp)) * 2 + (j & 1));
    } else {
        return 8 * r;
    }
}

// Branch-free load of one lane's CPL entries starting at p.  EXACT: the
// panels tile the row exactly, so the loads are whole float4s.  Otherwise
// offsets past lim (the row's last entry) are clamped to it and their
// values are masked at use.  Every load is issued unconditionally so the
// prefetch ring keeps fixed registers.
template <int CPL, bool EXACT>
__device__ __forceinline__ void load_chunk(float (&v)[CPL], const float* __restrict__ p, int lim) {
    if constexpr (EXACT && CPL % 4 == 0) {
        const float4* r4 = reinterpret_cast<const float4*>(p);
#pragma unroll
        for (int j = 0; j < CPL / 4; ++j) {
            const float4 t = r4[j];
            v[4 * j] = t.x; v[4 * j + 1] = t.y; v[4 * j + 2] = t.z; v[4 * j + 3] = t.w;
        }
    } else {
#pragma unroll
        for (int j = 0; j < CPL; ++j) v[j] = p[min(j, lim)];
    }
}

// Value of lane 63 in every lane.
__device__ __forceinline__ float lane63(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}
__device__ __forceinline__ double lane63(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, 63);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), 63);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Value of lane L (a constant) in every lane.
__device__ __forceinline__ float lane_read(float v, int L) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), L));
}
__device__ __forceinline__ double lane_read(double v, int L) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, L);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), L);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Same-wave LDS ordering point: keeps the compiler from moving LDS accesses
// across it (the hardware already executes one wave's LDS operations in
// order).
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

template <bool B>
struct BoolTag { static constexpr bool value = B; };

// Per-step state carried from one panel pass to the next, spread over the
// lanes: step n lives in lane n % 64 of register n / 64.  Reads and writes
// take a wave-uniform step index.
template <int CR>
struct LaneCarry {
    float v[CR];
    __device__ __forceinline__ void zero() {
#pragma unroll
        for (int r = 0; r < CR; ++r) v[r] = 0.0f;
    }
    __device__ __forceinline__ float get(int n) const {
        float out = 0.0f;
#pragma unroll
        for (int r = 0; r < CR; ++r) {
            const float x = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v[r]), n & 63));
            out = (n >> 6) == r ? x : out;
        }
        return out;
    }
    __device__ __forceinline__ void set(int n, float x) {
        const int l = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
#pragma unroll
        for (int r = 0; r < CR; ++r) v[r] = (l + 64 * r) == n ? x : v[r];
    }
    // step n's value += x (wave-uniform), added by the lane that holds it
    __device__ __forceinline__ void add(int n, float x) {
        const int l = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
#pragma unroll
        for (int r = 0; r < CR; ++r) v[r] = (l + 64 * r) == n ? v[r] + x : v[r];
    }
    // value of step r * 64 + lane
    __device__ __forceinline__ float mine(int r) const { return v[r]; }
};

template <int CR>
struct LaneCarry64 {
    LaneCarry<CR> lo, hi;
    __device__ __forceinline__ void zero() { lo.zero(); hi.zero(); }
    __device__ __forceinline__ double get(int n) const {
        const uint32_t l = __builtin_bit_cast(uint32_t, lo.get(n));
        const uint32_t h = __builtin_bit_cast(uint32_t, hi.get(n));
        return __builtin_bit_cast(double, ((uint64_t)h << 32) | l);
    }
    __device__ __forceinline__ void set(int n, double x) {
        const uint64_t u = __builtin_bit_cast(uint64_t, x);
        lo.set(n, __builtin_bit_cast(float, (uint32_t)u));
        hi.set(n, __builtin_bit_cast(float, (uint32_t)(u >> 32)));
    }
    __device__ __forceinline__ double mine(int r) const {
        const uint32_t l = __builtin_bit_cast(uint32_t, lo.mine(r));
        const uint32_t h = __builtin_bit_cast(uint32_t, hi.mine(r));
        return __builtin_bit_cast(double, ((uint64_t)h << 32) | l);
    }
    // step n's value += x (wave-uniform), added by the lane that holds it:
    // the same fp64 addition as get + set, without reading the lane out
    __device__ __forceinline__ void add(int n, double x) {
        const int l = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
#pragma unroll
        for (int r = 0; r < CR; ++r) {
            const double v = mine(r) + x;
            const uint64_t u = __builtin_bit_cast(uint64_t, v);
            const bool own = (l + 64 * r) == n;
            lo.v[r] = own ? __builtin_bit_cast(float, (uint32_t)u) : lo.v[r];
            hi.v[r] = own ? __builtin_bit_cast(float, (uint32_t)(u >> 32)) : hi.v[r];
        }
    }
};

// One workgroup (a single wave) scores every prefix of one model's queue at
// one batch size.  Lane l of pass p owns bins [(p*64 + l) CPL, +CPL) and
// keeps their batch CDF G_n(x_{k+1}) = prod_{i <= n} F_{c_i}(x_{k+1}) as an
// fp64 running product over the steps n (the table holds 1 - F, so a step
// is one fma per bin).  Per step: the sums of 1 - G and the discounted
// prefix over the panel (4-bin quarters keep the dependency chains short,
// a DPP scan joins the lanes), the carries into the next panel, and, if
// some member's deadline falls in this panel, a snapshot in LDS that the
// same wave then reads to score those members.  Rows are prefetched PF
// iterations ahead through a register ring.  Panels past the last member's
// deadline need only the sums of 1 - G: a second, lean loop takes them
// (tabulated mode).  Launches with too few workgroups to fill the chip go to
// turned_kernel.
#ifndef ORLOJ_SCORE_PREFETCH
#define ORLOJ_SCORE_PREFETCH 2   // iterations a row is loaded ahead of its use
#endif
#ifndef ORLOJ_EONLY_PREFETCH
#define ORLOJ_EONLY_PREFETCH 3   // iterations ahead in the E-only panels' loop
#endif
#ifndef ORLOJ_EONLY_CACHE
#define ORLOJ_EONLY_CACHE 2      // classes whose slices the E-only loop keeps in registers
#endif
#ifndef ORLOJ_EONLY_LDS_CACHE
#define ORLOJ_EONLY_LDS_CACHE 3  // further classes whose slices it keeps in LDS
#endif
template <int CPL, int PF, bool EXACT, int CR, bool AFF>
__device__ __forceinline__ void score_wave(const ScoreArgs& a, const unsigned bid) {
    using Q = Quarters<CPL>;
    constexpr int PW = 64 * CPL;                   // bins per panel
    extern __shared__ __align__(16) unsigned char smem_raw[];
    using L = ScoreLds<CPL>;
    double* s_kd = reinterpret_cast<double*>(smem_raw + L::KD);   // constant slots
    float* s_zq = reinterpret_cast<float*>(smem_raw + L::ZQ);
    float* s_A = reinterpret_cast<float*>(smem_raw + L::AA);
    float* s_fz = reinterpret_cast<float*>(smem_raw + L::FZ);
    Member* s_mem = reinterpret_cast<Member*>(smem_raw + L::MEM);   // CR > 1 only
    const int maxcap = a.maxcap;

    const int lane = threadIdx.x;

    // Largest batch sizes first: those workgroups run longest.
    const int bi = a.nbs - 1 - (int)(bid / (unsigned)a.Mg);
    const int q = grid_model(a, bid % (unsigned)a.Mg);
    const int64_t q0 = a.queue_off[q];
    const int64_t N = a.queue_off[q + 1] - q0;
    const int bsz = a.bs[bi];
    const int64_t cap64 = a.rect ? N : (N < bsz ? N : (int64_t)bsz);
    if (cap64 <= 0 || cap64 > maxcap || cap64 > 64 * CR) return;   // the host sizes both
    const int ncap = (int)cap64;
    // The longest workgroups set a saturated launch's length (their steps
    // run one after another while shorter ones share their SIMD): they
    // take issue priority over the short ones, graded by their step count.
    if (ncap >= 48) __builtin_amdgcn_s_setprio(3);
    else if (ncap >= 32) __builtin_amdgcn_s_setprio(2);
    else if (ncap >= 16) __builtin_amdgcn_s_setprio(1);

    // Affine mode (Eq. (3)): a batch of size s whose slowest member takes l
    // runs c0 + c1 s l, so its latency histogram is the base grid's with
    // bins c1 s w wide, shifted by c0.  Everything below works on that
    // grid: the bin width is c1 s w, the time left is tau - c0, and
    // E[L_B] = c0 + c1 s E[max] (Eq. (5)).  Tabulated mode: c0 = 0, width w.
    // The product over members is the same for every batch size there, so
    // E[max]'s sums come from emax_kernel, and a wave walks only the panels
    // up to its last member's home panel.
    const double wq = a.width[q];
    double c0q = 0.0;
    bool aok = true;
    double w = wq;
    if constexpr (AFF) {
        c0q = a.c0[q];
        const double c1 = a.c1[q];
        aok = c0q >= 0.0 && c0q < HUGE_VAL && c1 > 0.0 && c1 < HUGE_VAL;
        w = c1 * (double)bsz * wq;
    }
    const bool wok = wq > 0.0 && wq < HUGE_VAL && aok && w > 0.0 && w < HUGE_VAL;   // else a data error
    const double nowq = a.now[q];
    const double b = a.b;
    const double bw = b * w;
    const int K = a.K;
    const int NP = (K + PW - 1) / PW;

    const double d64 = exp(-bw);                      // discount per bin
    const float log2d = (float)(-bw * 1.4426950408889634);
    const float gamma = (float)(-expm1(-bw) / bw);   // (1 - d) / (b w)
    const float omd = (float)(-expm1(-bw));          // 1 - d

    // ---- member lookup plans (fp64 time relative to now).  `check` flags
    // the member's data errors (once per member and workgroup).
    auto make_plan = [&](int m, bool check) -> Member {
        int c = a.cls[q0 + m];
        const double D = a.deadline[q0 + m];
        double cm = a.cost ? a.cost[q0 + m] : 1.0;
        if (check) {
            int flag = 0;
            if (c < 0 || c >= a.C) flag |= kErrClassRange;
            if (isnan(D)) flag |= kErrDeadlineNaN;
            if (m > 0 && D < a.deadline[q0 + m - 1]) flag |= kErrUnsorted;
            if (m == 0 && isnan(nowq)) flag |= kErrNowNaN;
            if (m == 0 && !(wq > 0.0 && wq < HUGE_VAL)) flag |= kErrWidth;
            if (m == 0 && !aok) flag |= kErrAffine;
            if (!(cm >= 0.0 && cm < HUGE_VAL)) flag |= kErrCost;
            if (flag) atomicOr(a.err, flag);
        }
        if (c < 0 || c >= a.C) c = 0;
        if (!(cm >= 0.0 && cm < HUGE_VAL)) cm = 0.0;
        Member mb;
        mb.cost = (float)cm;
        mb.rq = (uint8_t)kNoQuarter;
        // byte offsets: KD reads 0, KD + 8 reads 1, KD + 16 reads gl; FZ
        // reads a float 0
        int hp = 0, o0 = L::KD, o1 = L::KD, o4 = 0, oz = L::FZ, oa = L::FZ;
        mb.cW = mb.cG = mb.cA = mb.fq = 0.0f;
        mb.theta = mb.thlo = mb.cg = mb.psi = 0.0f;
        const double tau = D - nowq - c0q;
        int kz = -1;   // bin whose discounted prefix Z the priority needs
        if (tau > 0.0 && wok) {
            const double u = tau / w;
            if (u >= (double)K) {                  // beyond the grid: P = 1
                o0 = o1 = L::KD + 8;
                mb.cg = gamma * (float)exp(-b * (tau - (double)K * w));
                hp = NP - 1;
                kz = K - 2;
            } else {
                const double kf = floor(u);
                const double th = u - kf;
                const int k = (int)kf;
                hp = k / PW;
                mb.theta = (float)th;
                mb.thlo = (float)(th - (double)mb.theta);
                mb.cg = gamma * (float)exp(-b * th * w);
                mb.psi = (float)(-expm1(-b * th * w) / bw);
                o1 = snap_byte<CPL>(k - hp * PW);
                if (k >= 1) o0 = k - 1 >= hp * PW ? snap_byte<CPL>(k - 1 - hp * PW) : L::KD + 16;
                kz = k - 2;
            }
        }
        if (kz >= 0) {
            const int p0 = hp * PW;                // first bin of the home panel
            if (kz >= p0) {
                const int r = kz - p0, l = r / CPL, j = r - l * CPL;
                const int qq = j / Q::QW, rq = j - qq * Q::QW;
                mb.cW = hp > 0 ? exp2f(log2d * (float)(kz - p0 + 1)) : 0.0f;
                if (l > 0) {
                    oa = L::AA + 4 * (l - 1);
                    mb.cA = exp2f(log2d * (float)(j + 1));
                }
                if (qq > 0) {
                    oz = L::ZQ + 4 * (l * Q::NQ + qq - 1);
                    mb.fq = exp2f(log2d * (float)(rq + 1));
                }
                o4 = snap_byte<CPL>(r - rq);       // first bin of the quarter
                mb.rq = (uint8_t)rq;
            } else if (kz == p0 - 1) {             // last bin of the previous panel
                mb.cW = 1.0f;
            } else {                               // kz = p0 - 2: step back one bin
                mb.cW = (float)exp(bw);
                mb.cG = -(float)exp(bw);
            }
        }
        mb.hp = (uint8_t)hp;
        mb.o0 = (uint16_t)o0; mb.o1 = (uint16_t)o1; mb.o4 = (uint16_t)o4;
        mb.oz = (uint16_t)oz; mb.oa = (uint16_t)oa;
        return mb;
    };
    // Everything from here on is compiled twice: for the waves whose members
    // all lie in panel 0 (ONE: no carries between panel passes, every step
    // scores members; at configuration 5 that is every wave) and for the
    // rest.  The branch comes before any per-lane state, so the two versions
    // share no registers' worth of live values.  The last member's plan
    // gives its home panel, as it does below.
    const int lastp = __builtin_amdgcn_readfirstlane((int)make_plan(ncap - 1, false).hp);
    auto rest = [&](auto one_tag) {
        constexpr bool ONE = decltype(one_tag)::value;
        // The prologue is a chain of memory round trips, which the launches too
        // small to fill the chip wait on: the loads that do not depend on each
        // other are issued together.  This batch size's block of candidates and
        // member slots starts after those of the batch sizes before it (one per
        // lane, summed across the wave).
        int64_t cand = a.cand_off[q], prob = a.prob_off[q];
        {
            uint64_t dc = 0, dp = 0;
            for (int j0 = 0; j0 < bi; j0 += 64) {
                const int j = j0 + lane;
                if (j < bi) {
                    const int64_t c = a.rect ? N : (N < a.bs[j] ? N : (int64_t)a.bs[j]);
                    dc += (uint64_t)c;
                    dp += (uint64_t)(c * (c + 1) / 2);
                }
            }
            cand += (int64_t)wave_sum_u64(dc, lane);
            prob += (int64_t)wave_sum_u64(dp, lane);
        }
        // rows of this (model, batch size); affine mode has one set per model
        const size_t qb = AFF ? (size_t)q : (size_t)q * (size_t)a.nbs + (size_t)bi;
        const float* tab_qb = a.tab + qb * (size_t)a.C * (size_t)K;

        // class and support of member n in lane n % 64 of register n / 64, and
        // the members' plans, in one pass
        LaneCarry<CR> cls_r, lo_r, hi_r;
        const int32_t* sup_qb = a.sup ? a.sup + qb * (size_t)a.C * 2 : nullptr;
#pragma unroll
        for (int r = 0; r < CR; ++r) {
            const int m = r * 64 + lane;
            int c = a.cls[q0 + min(m, ncap - 1)];
            if (c < 0 || c >= a.C) c = 0;                     // flagged by its plan
            cls_r.v[r] = __builtin_bit_cast(float, c);
            lo_r.v[r] = __builtin_bit_cast(float, sup_qb ? sup_qb[2 * c] : 0);
            hi_r.v[r] = __builtin_bit_cast(float, sup_qb ? sup_qb[2 * c + 1] : K);
            if (m < ncap) s_mem[m] = make_plan(m, true);
        }
        if (lane == 0) {
            s_kd[0] = 0.0;
            s_kd[1] = 1.0;
            s_kd[2] = 0.0;
            s_kd[3] = 0.0;
        }
        if (lane < 4) s_fz[lane] = 0.0f;
        wave_lds_fence();
        // Home panel of the last member (the latest deadline): past it no member
        // needs G or the discounted prefix, only E[L_B] needs the sums of 1 - G.
        // The main loop walks the panels up to LASTP; the tabulated mode then
        // sums the rest (E-only panels) in a loop of its own, the affine mode
        // takes them from emax_kernel.
        const int LASTP = ONE ? 0 : __builtin_amdgcn_readfirstlane((int)s_mem[ncap - 1].hp);
        const int NPW = LASTP + 1;
        // first member of each panel p in lane p (home panels are non-decreasing
        // in m): counted up to LASTP; every member's home panel lies before the
        // later ones, so their lanes hold ncap
        int mlo_r = ncap;
        for (int p = 0; p <= LASTP; ++p) {
            int cnt = 0;
            for (int m0 = 0; m0 < ncap; m0 += 64) {
                const int m = m0 + lane;
                const bool below = m < ncap && s_mem[m].hp < p;
                cnt += __builtin_popcountll(__ballot(below));
            }
            mlo_r = lane == p ? cnt : mlo_r;
        }

        // ---- scan constants
        float rp[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) rp[i] = exp2_hw(log2d * (float)(CPL << i));
        const float w15 = exp2_hw(log2d * (float)(CPL * ((lane & 15) + 1)));
        const float w31 = exp2_hw(log2d * (float)(CPL * (lane >= 32 ? lane - 31 : 0)));
        const float dQ = exp2_hw(log2d * (float)Q::QW);
        const float dq1 = exp2f(log2d);                   // d in fp32
        // A member's in-quarter discounted prefix up to bin k-2, the quarter's
        // r-th bin being bin k-2 (rq = r <= 3): sum over j <= rq of
        // d^(rq - j) G_j, formed as a dot product with these weights (all 0
        // when the member needs no quarter term, rq = kNoQuarter).
        const float dq2 = dq1 * dq1, dq3 = dq2 * dq1;
        auto quarter_weights = [&](int rq, float (&wv)[4]) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int e = rq - r;
                wv[r] = (e < 0 || rq > 3) ? 0.0f : e == 0 ? 1.0f : e == 1 ? dq1 : e == 2 ? dq2 : dq3;
            }
        };
        const float dPW = exp2_hw(log2d * (float)PW);

        // Load the lane chunk starting at bin c0 of member n's row; chunks wholly
        // outside the row's support, and every chunk when `none` (the row's
        // values cannot change G), read a constant row instead.
        // The member's support bounds go to lo / hi: the ring slot keeps them
        // for the step that uses the row.
        auto load_step = [&](float (&v)[CPL], int n, int c0, bool none, int& lo, int& hi) {
            const int c = __builtin_bit_cast(int, cls_r.get(n));
            lo = __builtin_bit_cast(int, lo_r.get(n));
            hi = __builtin_bit_cast(int, hi_r.get(n));
            // The affine mode's solo table (M x C rows) stays in the Infinity
            // Cache, so it reads every chunk rather than spend a per-lane test
            // and select on each load; entries outside the support are exactly
            // 1 and 0 either way.
            const bool ones = !AFF && !none && c0 + CPL <= lo, zeros = none || (!AFF && c0 >= hi);
            const float* src = tab_qb + (size_t)c * (size_t)K + c0;
            int lim = K - 1 - c0;
            if (ones || zeros) {
                src = a.fill + (ones ? 16 : 0);
                lim = CPL - 1;
            }
            load_chunk<CPL, EXACT>(v, src, lim);
        };

        LaneCarry<CR> cW, cN;
        LaneCarry64<CR> cE, cP, cGl;
        cW.zero(); cGl.zero(); cN.zero(); cE.zero(); cP.zero();

        // One flat loop over (panel p, step n), n fastest, padded at the end to
        // a multiple of PF with ghost iterations (p == NP) so that ring slot i
        // always holds iteration it0 + i.  The row of iteration it + PF is
        // loaded PF iterations ahead; (p, n) and the prefetch position advance
        // by counting.
        const int total = NPW * ncap;
        const int iters = (total + PF - 1) / PF * PF;
        const int base = lane * CPL;

        double Gacc[CPL];
        float buf[PF][CPL];
        int slo[PF], shi[PF];                                 // the slots' support bounds
        int pf_p = 0, pf_n = 0;                               // prefetch position
#pragma unroll
        for (int i = 0; i < PF; ++i) {
            load_step(buf[i], pf_n, pf_p * PW + base, false, slo[i], shi[i]);
            // keep the priming loads in ring order, as the loop issues them
            __builtin_amdgcn_sched_barrier(0);
            if (++pf_n == ncap) { pf_n = 0; pf_p = min(pf_p + 1, NPW - 1); }
        }
        int p = 0, n = 0;
        int mlo = __builtin_amdgcn_readlane(mlo_r, 0);
        int mend = __builtin_amdgcn_readlane(mlo_r, 1);
        // Trivial steps.  Where a panel lies wholly past the last bin with mass
        // of member n's row (every 1 - F there is exactly 0), or where G is
        // already exactly 0 over the whole panel (an earlier member's row had
        // no mass up to its end), step n leaves G unchanged bit for bit; if no
        // member of the panel needs scoring at that step, its panel sums are
        // those of step n-1 and the update, its loads and its reductions are
        // skipped.
        bool pass_zero = false;                  // G == 0 on every bin of this pass's panel
        Member pass_mb;                          // CR == 1: this lane's member of the pass
        double pass_th = 0.0;                    //   and its position in bin k, fp64,
        float pass_wq[4] = {0.0f, 0.0f, 0.0f, 0.0f};   // and its quarter weights
        bool pass_valid = false;
        float etot_prev = 0.0f, T_prev = 0.0f;
        double gl_prev = 0.0;

        static_assert(PF % 2 == 0, "steps are reduced in pairs");
        for (int it0 = 0; it0 < iters; it0 += PF) {
            // each scoring step's member sums (0 in lanes without a member) and
            // its index (-1: no member scored)
            double redP[PF];
            float redN[PF];
            int red_n[PF];
#pragma unroll
            for (int i = 0; i < PF; ++i) redP[i] = 0.0, redN[i] = 0.0f, red_n[i] = -1;
#pragma unroll
            for (int i = 0; i < PF; ++i) {
                if (n == 0) {
                    // a real branch (the asm keeps it from becoming selects)
                    asm volatile("" ::: "memory");
#pragma unroll
                    for (int j = 0; j < CPL; ++j) Gacc[j] = 1.0;
                    pass_zero = false;
                    if constexpr (CR == 1) {
                        // at most 64 members: lane l scores member mlo + l of this
                        // pass at every step, so its plan is read from LDS once
                        pass_valid = mlo + lane < mend;
                        pass_mb = s_mem[min(mlo + lane, ncap - 1)];
                        pass_th = (double)pass_mb.theta + (double)pass_mb.thlo;
                        quarter_weights(pass_mb.rq, pass_wq);
                    }
                }
                const int p0 = ONE ? 0 : p * PW;              // first bin of the panel
                const int pbase = p0 + base;                  // first bin of this lane chunk
                const int hi_n = shi[i];
                const int lo_n = slo[i];
                // members of this panel among the first n+1 (ONE: all of them)
                const int mhi = ONE ? n + 1 : min(mend, n + 1);
                const bool due = ONE || mlo < mhi;            // some member is scored at this step
                // G unchanged by this step (a panel past the row's support, or G
                // already 0 on it): a step after the first reuses the previous
                // step's sums
                const bool unchanged = pass_zero || p0 >= hi_n;
                const bool skip = p >= NPW || (n > 0 && unchanged && !due);
                // G <- G * F = G - G (1 - F), in fp64; per-quarter sums
                double gs[Q::QW];
                float zqv[Q::NQ];
                if (!skip) {
#pragma unroll
                    for (int qq = 0; qq < Q::NQ; ++qq) {
                        double zz = 0.0;
#pragma unroll
                        for (int r = 0; r < Q::QW; ++r) {
                            const int j = qq * Q::QW + r;
                            const float t = (EXACT || pbase + j < K) ? buf[i][j] : 0.0f;
                            Gacc[j] = fma(-Gacc[j], (double)t, Gacc[j]);
                            if constexpr (!AFF) gs[r] = qq == 0 ? Gacc[j] : gs[r] + Gacc[j];
                            zz = r == 0 ? Gacc[j] : fma(zz, d64, Gacc[j]);
                        }
                        zqv[qq] = (float)zz;
                    }
                }
                // the slot is refilled only after the update has consumed it, so
                // the ring keeps its registers (no copies, no wait on the loads
                // just issued)
#pragma unroll
                for (int j = 0; j < CPL; ++j) asm volatile("" : "+v"(Gacc[j])::"memory");
                // G == 0 over the pass from here on: later steps of it need no row
                const bool zero_after = pass_zero || min(p0 + PW, K) <= lo_n;
                load_step(buf[i], pf_n, pf_p * PW + base, zero_after && pf_p == p, slo[i], shi[i]);
                if (++pf_n == ncap) { pf_n = 0; pf_p = ONE ? 0 : min(pf_p + 1, NPW - 1); }
                if (p < NPW) {                                // else a ghost iteration
                    float etot = etot_prev, T = T_prev;
                    double glast_here = gl_prev;
                    // carries in from the previous panel pass (zero in the first)
                    float Win = 0.0f;
                    double glin64 = 0.0;
                    if (!ONE && p > 0) {
                        Win = cW.get(n);
                        glin64 = cGl.get(n);
                    }
                    const float glin = (float)glin64;
                    float A = 0.0f;
                    if (!skip) {
                        // quarter ends of the in-chunk discounted prefix, and its total
                        float zc = zqv[0];
#pragma unroll
                        for (int qq = 1; qq < Q::NQ; ++qq) {
                            zc = fmaf(zc, dQ, zqv[qq]);
                            zqv[qq] = zc;
                        }
                        A = wave_wscan(zc, rp, w15, w31);
                        if (!ONE && p < LASTP) {              // carried into the next pass
                            T = lane63(A);                    // discounted prefix at the panel end
                            T_prev = T;
                        }
                    }
                    if (!skip) {
                        if constexpr (!AFF) {
                            double gsum = gs[0];
#pragma unroll
                            for (int r = 1; r < Q::QW; ++r) gsum += gs[r];
                            // 1 - G summed over the lane's bins (padding bins hold G = 1)
                            const float e = (float)((double)CPL - gsum);
                            etot = lane63(wave_scan_sum(e));
                        }
                        if (!ONE && p < LASTP) {              // carried into the next pass
                            glast_here = lane63(Gacc[CPL - 1]);
                            gl_prev = glast_here;
                        }
                        etot_prev = etot;

                        if (due) {
                            // snapshot of G over the panel, fp64, pairs of bins
                            // interleaved over the lanes (16-byte writes)
                            if constexpr (CPL >= 2) {
#pragma unroll
                                for (int j = 0; j < CPL; j += 2) {
                                    const int pair = (j >> 1) * 64 + (lane ^ (j >> 1));
                                    *reinterpret_cast<double2*>(smem_raw + L::GD + 16 * pair) =
                                        make_double2(Gacc[j], Gacc[j + 1]);
                                }
                            } else {
                                *reinterpret_cast<double*>(smem_raw + L::GD + 8 * lane) = Gacc[0];
                            }
#pragma unroll
                            for (int qq = 0; qq < Q::NQ; ++qq) s_zq[lane * Q::NQ + qq] = zqv[qq];
                            s_A[lane] = A;
                            if (!ONE && lane == 0) s_kd[2] = glin64;   // (ONE: stays 0)
                            wave_lds_fence();
                            double pP = 0.0;
                            float pN = 0.0f;
                            const int nn = n + 1;
                            auto score_member = [&](const Member& mb, int m, double th, const float (&wq4)[4]) {
                                const unsigned char* f = smem_raw;
                                auto atf = [&](int off) { return *reinterpret_cast<const float*>(f + off); };
                                auto atd = [&](int off) { return *reinterpret_cast<const double*>(f + off); };
                                const double gk64 = atd(mb.o0);
                                const double gk164 = atd(mb.o1);
                                const float al0 = atf(mb.oa);
                                const float zq0 = atf(mb.oz);
                                // the quarter's G values (fp32 terms of the priority)
                                float g4[4];
                                if constexpr (Q::QW == 4) {
                                    const double2 t0 = *reinterpret_cast<const double2*>(f + mb.o4);
                                    // the quarter's second pair: its slot follows
                                    // the first's by 64, with the lane index's
                                    // low bit flipped (the first pair's index is even)
                                    const double2 t1 = *reinterpret_cast<const double2*>(f + ((mb.o4 + 16 * 64) ^ 16));
                                    g4[0] = (float)t0.x; g4[1] = (float)t0.y;
                                    g4[2] = (float)t1.x; g4[3] = (float)t1.y;
                                } else if constexpr (Q::QW == 2) {
                                    const double2 t0 = *reinterpret_cast<const double2*>(f + mb.o4);
                                    g4[0] = (float)t0.x; g4[1] = (float)t0.y;
                                    g4[2] = g4[3] = 0.0f;
                                } else {
                                    g4[0] = (float)atd(mb.o4);
                                    g4[1] = g4[2] = g4[3] = 0.0f;
                                }
                                // discounted prefix of the quarter up to bin k-2
                                // (weights 0 when the member needs no quarter term)
                                const float z4 = fmaf(wq4[0], g4[0], fmaf(wq4[1], g4[1], fmaf(wq4[2], g4[2], wq4[3] * g4[3])));
                                const float zin = fmaf(mb.fq, zq0, z4);
                                // (ONE: no pass before this one, so no carried
                                // terms: their weights are 0 and the rest is
                                // >= +0, so dropping them keeps the bits)
                                const float Zv = ONE ? fmaf(mb.cA, al0, zin)
                                                     : fmaf(mb.cW, Win, fmaf(mb.cG, glin, fmaf(mb.cA, al0, zin)));
                                const float gk = (float)gk64, gk1 = (float)gk164;
                                const float h = gk1 - gk;
                                // P in fp64: the expected finish count sums it
                                const double P64 = fma(th, gk164 - gk64, gk64);
                                const float num = mb.cost * fmaf(mb.cg, fmaf(-omd, Zv, gk), h * mb.psi);
                                a.P[prob + (int64_t)n * nn / 2 + m] = (float)P64;
                                // (one member per lane and pass when CR == 1:
                                // its values, not a sum with 0)
                                pP = CR == 1 ? P64 : pP + P64;
                                pN = CR == 1 ? num : pN + num;
                            };
                            if constexpr (CR == 1) {
                                // the lane's member of this pass, already in registers
                                if (pass_valid && mlo + lane < mhi) score_member(pass_mb, mlo + lane, pass_th, pass_wq);
                            } else {
                                for (int m = mlo + lane; m < mhi; m += 64) {
                                    const Member mb = s_mem[m];
                                    float wq4[4];
                                    quarter_weights(mb.rq, wq4);
                                    score_member(mb, m, (double)mb.theta + (double)mb.thlo, wq4);
                                }
                            }
                            // reduced across the lanes with the other step of
                            // its pair, after the pair
                            redP[i] = pP;
                            redN[i] = pN;
                            red_n[i] = n;
                            wave_lds_fence();
                        }
                    }
                    // carries out to the next panel pass, per-step sums
                    if (!ONE && p < LASTP) {
                        cW.set(n, fmaf(Win, dPW, T));
                        cGl.set(n, glast_here);
                    }
                    if constexpr (!AFF) cE.add(n, (double)etot);
                }
                pass_zero = zero_after;
                if (++n == ncap) {
                    n = 0;
                    ++p;
                    if (!ONE) {
                        mlo = __builtin_amdgcn_readlane(mlo_r, min(p, NP));
                        mend = __builtin_amdgcn_readlane(mlo_r, min(p + 1, NP));
                    }
                }
            }
            // Sum P (fp64) and the priority terms (fp32) over the lanes, two
            // steps at a time: each step's total comes out of the same tree
            // whichever step it is paired with.
#pragma unroll
            for (int i = 0; i < PF; i += 2) {
                if (red_n[i] >= 0 || red_n[i + 1] >= 0) {
                    const double zP = wave_pair_sum64(redP[i], redP[i + 1]);
                    const float zN = wave_pair_sum(redN[i], redN[i + 1]);
                    if (red_n[i] >= 0) {
                        cP.add(red_n[i], lane_read(zP, 31));
                        cN.add(red_n[i], lane_read(zN, 31));
                    }
                    if (red_n[i + 1] >= 0) {
                        cP.add(red_n[i + 1], lane_read(zP, 63));
                        cN.add(red_n[i + 1], lane_read(zN, 63));
                    }
                }
            }
        }

        // ---- E-only panels (tabulated mode): past LASTP no member reads G, so
        // these panels only add their sums of 1 - G to E[L_B], in a loop of its
        // own: the product and the sum, no discounted prefix, snapshot or
        // carries.  Its ring is primed afresh; the panels' sums are added in
        // panel order after those of the member panels, as before.  (AFF:
        // every panel's sums come from emax_kernel.)
        if constexpr (!AFF) {
            if (LASTP + 1 < NP) {
                constexpr int PFB = ORLOJ_EONLY_PREFETCH;   // its ring is deeper: fewer registers live here
                // Classes repeat along a deadline-ordered queue (fast classes
                // come first), and a repeat's row slice has usually left L2 by
                // the time the wave reads it again.  The RC classes with the
                // most members (at most 64 members, one per lane) keep their
                // slice of the current panel in registers for the pass: the
                // class's first member in step order loads it through the ring
                // as any step does and copies it, and its later members read the
                // copy while the ring loads the constant row for them.  Same
                // values, same bits.  (Where a step is skipped because G is 0
                // over the panel, every later step of the pass is skipped too,
                // so a copy taken then is never read.)
                // The next RL classes keep theirs in LDS, in the space of the
                // member panels' snapshot, prefixes and plans (unused from here
                // on), as far as this launch's LDS holds them: the first member
                // writes its slice there, and later members read it back into
                // their ring slot (loaded with the constant row) at their step.
                // The LDS read is issued at the step rather than with the ring's
                // loads: a ring filled from two kinds of loads would make every
                // step wait for all of the ring's memory loads.
                constexpr int RC = CR == 1 ? ORLOJ_EONLY_CACHE : 0;
                constexpr int RL = CR == 1 && CPL % 4 == 0 ? ORLOJ_EONLY_LDS_CACHE : 0;
                constexpr int NC = RC + RL;
                constexpr int RCA = RC > 0 ? RC : 1;
                constexpr int SLOT = 4 * PW;                        // bytes of one slice
                const int rl = min(RL, (int)((score_fixed_bytes<CPL>() + (size_t)maxcap * score_bytes_per_member()) / SLOT));
                // step code of member `lane`: NC (read from memory), k < NC (a
                // later member of cached class k: registers below RC, LDS from
                // RC), NC + 1 + k (the first member of class k)
                int rk_r = NC;
                if constexpr (NC > 0) {
                    const int cl = lane < ncap ? __builtin_bit_cast(int, cls_r.v[0]) : -1 - lane;
                    int cnt = 0, first = 64;        // members with this lane's class, the first of them
                    for (int m = ncap - 1; m >= 0; --m) {
                        const bool same = __builtin_amdgcn_readlane(cl, m) == cl;
                        cnt += same ? 1 : 0;
                        first = same ? m : first;
                    }
                    bool taken = lane >= ncap;
#pragma unroll
                    for (int k = 0; k < NC; ++k) {
                        // most members first, ties to the earlier member; a
                        // class with a single member gains nothing
                        const int key = (taken || cnt < 2 || k >= RC + rl) ? -1 : (cnt << 6) | (63 - lane);
                        const int best = wave_max_i32(key);
                        if (best >= 0) {
                            const int ck = __builtin_amdgcn_readlane(cl, 63 - (best & 63));
                            if (cl == ck)
                                rk_r = first == lane ? NC + 1 + k : k;
                            taken = taken || cl == ck;
                        }
                    }
                }
                auto code = [&](int n) -> int {
                    if constexpr (NC > 0) return __builtin_amdgcn_readlane(rk_r, n);
                    return NC;
                };
                // slice k of the LDS classes: float4 j of lane l at 1024 j + 16 l
                // (each access a run of 64 consecutive 16-byte words)
                auto lds_slice = [&](int k, int j) {
                    return reinterpret_cast<float4*>(smem_raw + (size_t)k * SLOT + 1024 * j + 16 * lane);
                };
                // the ring's load for step n: the constant row for a later member
                // of a cached class (and where `none`), else memory
                auto load_e = [&](float (&v)[CPL], int n, int c0, bool none, int& lo, int& hi) {
                    load_step(v, n, c0, none || code(n) < NC, lo, hi);
                };
                float creg[RCA][CPL];
#pragma unroll
                for (int k = 0; k < RCA; ++k)
#pragma unroll
                    for (int j = 0; j < CPL; ++j) creg[k][j] = 0.0f;
                float bufb[PFB][CPL];
                int blo[PFB], bhi[PFB];
                const int totalB = (NP - LASTP - 1) * ncap;
                const int itersB = (totalB + PFB - 1) / PFB * PFB;
                int qf_p = LASTP + 1, qf_n = 0;
#pragma unroll
                for (int i = 0; i < PFB; ++i) {
                    load_e(bufb[i], qf_n, qf_p * PW + base, false, blo[i], bhi[i]);
                    __builtin_amdgcn_sched_barrier(0);
                    if (++qf_n == ncap) { qf_n = 0; qf_p = min(qf_p + 1, NP - 1); }
                }
                int pb = LASTP + 1, nb = 0;
                bool zero_b = false;
                float eprev = 0.0f;
                for (int it0 = 0; it0 < itersB; it0 += PFB) {
#pragma unroll
                    for (int i = 0; i < PFB; ++i) {
                        const int p0 = pb * PW;
                        const int pbase = p0 + base;
                        if (nb == 0) {
                            asm volatile("" ::: "memory");
#pragma unroll
                            for (int j = 0; j < CPL; ++j) Gacc[j] = 1.0;
                            zero_b = false;
                        }
                        const int hi_n = bhi[i];
                        const int lo_n = blo[i];
                        const bool unchanged = zero_b || p0 >= hi_n;
                        const bool skip = pb >= NP || (nb > 0 && unchanged);
                        double gs[Q::QW];
                        // G <- G (1 - t) over the lane's bins, t from the row
                        // slice (ring slot or cache register)
                        auto update = [&](const float (&tv)[CPL]) {
#pragma unroll
                            for (int qq = 0; qq < Q::NQ; ++qq) {
#pragma unroll
                                for (int r = 0; r < Q::QW; ++r) {
                                    const int j = qq * Q::QW + r;
                                    const float t = (EXACT || pbase + j < K) ? tv[j] : 0.0f;
                                    Gacc[j] = fma(-Gacc[j], (double)t, Gacc[j]);
                                    gs[r] = qq == 0 ? Gacc[j] : gs[r] + Gacc[j];
                                }
                            }
                        };
                        const int kc = code(nb);
                        // a cached class's first member: keep its slice
#pragma unroll
                        for (int k = 0; k < RC; ++k) {
                            if (kc == NC + 1 + k) {
                                asm volatile("" ::: "memory");
#pragma unroll
                                for (int j = 0; j < CPL; ++j) creg[k][j] = bufb[i][j];
                            }
                        }
                        if constexpr (RL > 0) {
                            if (kc >= NC + 1 + RC) {
                                asm volatile("" ::: "memory");
#pragma unroll
                                for (int j = 0; j < CPL / 4; ++j)
                                    *lds_slice(kc - NC - 1 - RC, j) =
                                        make_float4(bufb[i][4 * j], bufb[i][4 * j + 1], bufb[i][4 * j + 2], bufb[i][4 * j + 3]);
                            }
                        }
                        if (!skip) {
                            bool done = false;
#pragma unroll
                            for (int k = 0; k < RC; ++k) {
                                if (!done && kc == k) {
                                    // a real branch per slot (the asm keeps it
                                    // from becoming per-bin selects)
                                    asm volatile("" ::: "memory");
                                    update(creg[k]);
                                    done = true;
                                }
                            }
                            if constexpr (RL > 0) {
                                if (!done && kc >= RC && kc < NC) {
                                    asm volatile("" ::: "memory");
#pragma unroll
                                    for (int j = 0; j < CPL / 4; ++j) {
                                        const float4 t = *lds_slice(kc - RC, j);
                                        bufb[i][4 * j] = t.x; bufb[i][4 * j + 1] = t.y;
                                        bufb[i][4 * j + 2] = t.z; bufb[i][4 * j + 3] = t.w;
                                    }
                                }
                            }
                            if (!done) update(bufb[i]);
                        }
#pragma unroll
                        for (int j = 0; j < CPL; ++j) asm volatile("" : "+v"(Gacc[j])::"memory");
                        const bool zero_after = zero_b || min(p0 + PW, K) <= lo_n;
                        load_e(bufb[i], qf_n, qf_p * PW + base, zero_after && qf_p == pb, blo[i], bhi[i]);
                        if (++qf_n == ncap) { qf_n = 0; qf_p = min(qf_p + 1, NP - 1); }
                        if (pb < NP) {
                            float etot = eprev;
                            if (!skip) {
                                double gsum = gs[0];
#pragma unroll
                                for (int r = 1; r < Q::QW; ++r) gsum += gs[r];
                                const float e = (float)((double)CPL - gsum);
                                etot = lane63(wave_scan_sum(e));
                                eprev = etot;
                            }
                            cE.add(nb, (double)etot);
                        }
                        zero_b = zero_after;
                        if (++nb == ncap) { nb = 0; ++pb; }
                    }
                }
            }
        }

        // ---- candidate outputs: lane l holds steps l, l + 64, ...
#pragma unroll
        for (int r = 0; r < CR; ++r) {
            const int n = r * 64 + lane;
            if (n < ncap) {
                double esum = cE.mine(r);
                if constexpr (AFF) {
                    // the panels' sums in panel order, as this kernel adds them
                    esum = 0.0;
                    const float* ps = a.psum + (size_t)q * (size_t)a.np_e * (size_t)maxcap + n;
                    for (int pp = 0; pp < a.np_e; ++pp) esum += (double)ps[(size_t)pp * (size_t)maxcap];
                }
                a.E[cand + n] = cP.mine(r);
                double c0e = c0q, we = w;
                if constexpr (AFF) {
                    // read again: kept through the step loop they cost spills
                    const double *pc0 = a.c0, *pc1 = a.c1, *pw = a.width;
                    asm volatile("" : "+s"(pc0), "+s"(pc1), "+s"(pw));
                    c0e = pc0[q];
                    we = pc1[q] * (double)bsz * pw[q];
                }
                const double el = c0e + we * (0.5 + esum);
                a.EL[cand + n] = (float)el;
                a.S[cand + n] = (float)((double)cN.mine(r) / el);
            }
        }
    };
    if (lastp == 0) rest(BoolTag<true>{});
    else rest(BoolTag<false>{});
}

// The affine mode's waves (at most 64 members) are held to 80 VGPRs, six
// waves per SIMD instead of the four their 100 would allow: the spills that
// costs lie outside the step loop (cfg5 affine call 0.0788 -> 0.0738 ms; at
// 72 VGPRs the loop spills and it takes 0.0856 ms).
template <int CPL, int PF, bool EXACT, int CR, bool AFF>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(AFF && CR == 1 ? 6 : 1)))
void score_kernel(const ScoreArgs a) {
    score_wave<CPL, PF, EXACT, CR, AFF>(a, blockIdx.x);
}

// ---------------------------------------------------------------------------
// emax_kernel (affine mode): the sums behind E[L_B], one wave per (model,
// panel), ahead of score_kernel.  E[L_B] = c0 + c1 s w (1/2 + sum_k
// (1 - G_n(x_{k+1}))) (Eq. (5)) needs the panel sums of 1 - G for every
// prefix length n.  Under Eq. (3) every batch size's histogram is the same
// product G_n of the members' solo CDFs on the base grid, mapped onto a wider
// grid, so they are formed once per prefix length, not once per batch size.
// A wave keeps the running product of its panel's bins over the model's
// prefixes and writes each step's panel sum to psum[(model * panels + p) *
// maxcap + n], rounded to fp32 once.
// Rows are loaded PFE steps ahead; the class and support of step n sit in
// lane n % 64, so a step's row address needs no memory round trip.
// ---------------------------------------------------------------------------
// Steps loaded ahead by an emax_kernel wave: the loads of a step wait on
// nothing but the step's class, so a wave of narrow panels (few waves per
// SIMD) keeps more rows in flight.  A power of two that divides 64.
#ifndef ORLOJ_EMAX_PREFETCH_OF
#define ORLOJ_EMAX_PREFETCH_OF(CPL) ((CPL) >= 16 ? 8 : (CPL) >= 8 ? 16 : 32)
#endif

template <int CPL, bool EXACT, int CR>
__device__ __forceinline__ void emax_wave(const ScoreArgs& a, const unsigned bid) {
    using Q = Quarters<CPL>;
    constexpr int PW = 64 * CPL;
    constexpr int PFE = ORLOJ_EMAX_PREFETCH_OF(CPL);
    static_assert(PFE > 0 && 64 % PFE == 0, "a block of 64 steps ends on a prefetch round");
    const int K = a.K;
    const int NP = (K + PW - 1) / PW;
    const unsigned pair = bid / (unsigned)NP;
    const int p = (int)(bid - pair * (unsigned)NP);
    const int q = grid_model(a, pair);
    const int bi = a.nbs - 1;                   // the longest prefix (batch sizes increase)
    const size_t qb = (size_t)q;                // the model's rows and sums
    const int64_t q0 = a.queue_off[q];
    const int64_t N = a.queue_off[q + 1] - q0;
    const int64_t cap64 = a.rect ? N : (N < a.bs[bi] ? N : (int64_t)a.bs[bi]);
    if (cap64 <= 0 || cap64 > a.maxcap || cap64 > 64 * CR) return;
    const int ncap = (int)cap64;
    const int lane = threadIdx.x;
    const int pbase = p * PW + lane * CPL;
    const float* tab_q = a.tab + qb * (size_t)a.C * (size_t)K;
    const int32_t* sup_q = a.sup ? a.sup + qb * (size_t)a.C * 2 : nullptr;
    float* out = a.psum + (qb * (size_t)NP + (size_t)p) * (size_t)a.maxcap;

    LaneCarry<CR> cls_r, lo_r, hi_r;
#pragma unroll
    for (int r = 0; r < CR; ++r) {
        const int m = min(r * 64 + lane, ncap - 1);
        int c = a.cls[q0 + m];
        if (c < 0 || c >= a.C) c = 0;                     // score_kernel flags it
        cls_r.v[r] = __builtin_bit_cast(float, c);
        lo_r.v[r] = __builtin_bit_cast(float, sup_q ? sup_q[2 * c] : 0);
        hi_r.v[r] = __builtin_bit_cast(float, sup_q ? sup_q[2 * c + 1] : K);
    }
    // the lane chunk of member n's row; chunks wholly outside the row's
    // support read the constant rows (the same bits, see score_kernel)
    auto load = [&](float (&v)[CPL], int n) {
        const int c = __builtin_bit_cast(int, cls_r.get(n));
        const int lo = __builtin_bit_cast(int, lo_r.get(n));
        const int hi = __builtin_bit_cast(int, hi_r.get(n));
        const bool ones = pbase + CPL <= lo, zeros = pbase >= hi;
        const float* src = tab_q + (size_t)c * (size_t)K + pbase;
        int lim = K - 1 - pbase;
        if (ones || zeros) {
            src = a.fill + (ones ? 16 : 0);
            lim = CPL - 1;
        }
        load_chunk<CPL, EXACT>(v, src, lim);
    };

    double G[CPL];
#pragma unroll
    for (int j = 0; j < CPL; ++j) G[j] = 1.0;
    float buf[PFE][CPL];
#pragma unroll
    for (int i = 0; i < PFE; ++i) {
        load(buf[i], min(i, ncap - 1));
        __builtin_amdgcn_sched_barrier(0);
    }
    // Each step's lane sums are parked in LDS, one row per step, and every
    // 64 steps lane r adds up row r, pairwise: no cross-lane reduction on
    // every step.
    __shared__ float s_e[64][65];
    for (int n0 = 0; n0 < ncap; n0 += PFE) {
#pragma unroll
        for (int i = 0; i < PFE; ++i) {
            const int n = n0 + i;
            if (n < ncap) {
                double gs[Q::QW];
#pragma unroll
                for (int qq = 0; qq < Q::NQ; ++qq) {
#pragma unroll
                    for (int r = 0; r < Q::QW; ++r) {
                        const int j = qq * Q::QW + r;
                        const float t = (EXACT || pbase + j < K) ? buf[i][j] : 0.0f;
                        G[j] = fma(-G[j], (double)t, G[j]);
                        gs[r] = qq == 0 ? G[j] : gs[r] + G[j];
                    }
                }
                double gsum = gs[0];
#pragma unroll
                for (int r = 1; r < Q::QW; ++r) gsum += gs[r];
                s_e[n & 63][lane] = (float)((double)CPL - gsum);   // padding bins hold G = 1
            }
            // refill the slot only after the update has read it
#pragma unroll
            for (int j = 0; j < CPL; ++j) asm volatile("" : "+v"(G[j])::"memory");
            load(buf[i], min(n + PFE, ncap - 1));
        }
        // a full block of 64 steps, or the last steps: lane r sums step
        // (block start + r)
        const int done = n0 + PFE;
        if ((done & 63) == 0 || done >= ncap) {
            wave_lds_fence();
            const int blk = (done - 1) & ~63;
            const int nr = blk + lane;
            if (nr < ncap) {
                float v[32];
#pragma unroll
                for (int k = 0; k < 32; ++k) v[k] = s_e[lane][2 * k] + s_e[lane][2 * k + 1];
#pragma unroll
                for (int w = 16; w >= 1; w >>= 1)
#pragma unroll
                    for (int k = 0; k < w; ++k) v[k] = v[2 * k] + v[2 * k + 1];
                out[nr] = v[0];
            }
            wave_lds_fence();
        }
    }
}

template <int CPL, bool EXACT, int CR>
__global__ __launch_bounds__(64) void emax_kernel(const ScoreArgs a) {
    emax_wave<CPL, EXACT, CR>(a, blockIdx.x);
}

// ---------------------------------------------------------------------------
// turned_kernel: scoring in launches too small to fill the chip.
//
// There score_kernel's waves, one per (model, batch size), run their steps
// one after another with most of the chip idle.  Here a workgroup of up to
// eight waves takes a block of 64 prefix lengths of one (model, batch size)
// and its waves split the bins:
//
//   Member segments.  The bins up to the last deadline lie in equal segments,
//   a wave each.  The wave forms G transposed, a block of 16 S bins
//   x 16 RG prefix lengths (S RG = 4) at a time: a DPP row of 16 lanes takes
//   16 members at 16 bins, their products are chained over the groups of 16
//   members and turned in LDS, so that a lane holds one prefix length over
//   16 consecutive bins.  The discounted prefix of Eq. (2) and the sums
//   behind E[L_B] are then recurrences in a register, and a member's P and
//   priority for all 64 prefix lengths take one evaluation with uniform
//   constants: nothing is reduced over the lanes, and the sums over the
//   members are the lanes' own.  S = 4 or 2 for prefixes of at most 16 or 32
//   members, which would leave lanes idle otherwise.  The rows of a block are
//   loaded while the block before it is worked on.
//
//   The discounted prefix carried into a segment is known only when the
//   segments before it are done.  Every term of a priority is affine in it,
//   so a segment runs from 0 and keeps the sum of the coefficients; the
//   segments are joined at the end, in order.
//
//   The tiles past every member's deadline only add their sums of 1 - G to
//   E[L_B] (TurnedWave::e_tile): lanes hold the bins, the steps run in order
//   and each step's lane sums are added up a few steps at a time from LDS.
//   The waves take these tiles from a shared counter.  Rows of 4096 bins and
//   short queues have most of their bins here, and what bounds them is the
//   vector memory unit: loads of 64 consecutive floats a wave (256 bytes)
//   instead of every other one, and no register copies that wait for loads in
//   flight, took score + selection of one model of 4096 bins with prefixes to
//   64 from 51 to 36 us on rows in no cache, where score_kernel in step chunks
//   took 43; with tiles of 512 bins as well, prefixes to 4 took 22 -> 15 (19).
//
// What bounds it: latency, which is why the segments cut the member region
// evenly.  Its registers (188 to 234 a lane) leave two waves per SIMD, one
// workgroup of eight waves or two of four on a compute unit: a launch of more
// workgroups than compute units takes four (512 workgroups, prefixes to 32,
// 256 bins 26.7 -> 18.3 us, 1024 bins 27.6 -> 24.3; 64 workgroups 17.3 / 17.1
// and 17.6 / 20.1).  Capped at 128 registers, so that two workgroups of eight
// fit, it spills and takes 22.4 and 30.9 us there.  Score + selection, us,
// against score_kernel in step chunks, the way taken before: 1 model of 128
// bins and prefixes to 16 15.8 -> 14.9; 1024 bins, to 64 33.2 -> 19.0; 2048
// bins, to 128 144 -> 53; 5 models, 1501 bins, every prefix to 100 152 -> 36.
//
// G is an fp64 product.  Within a group of 16 members it is chained from 1,
// then multiplied by the product of the groups before: a member whose 1 - F
// is 0 leaves every bit of it unchanged, so exact ties between prefixes stay
// ties.  The segments depend on the queue and the batch size alone, and E's
// sums over a segment or tile are rounded to multiples of 2^-40 before they
// are added (any order gives the same sum), so it does not matter which wave
// takes which tile.  The number of waves sets the segments and with them the
// last bits of E and the scores.
// ---------------------------------------------------------------------------
constexpr int kETile = 128;                     // bins of a narrow E tile: two per lane
constexpr int kWide = 4;                        // narrow tiles in a wide one
constexpr int kWideFrom = 8 * kETile;           // bins past the members from which tiles are wide
constexpr int kPanel = 256;                     // bins of one affine E sum
// most affine E sums turned_esum_kernel writes: doubles that the fixed scratch
// array holds, so that the allocation-free call takes the same kernels
constexpr int64_t kTurnedSums = ORLOJ_NOALLOC_SCRATCH_FLOATS / 2;
constexpr int kGtRow = 136;                     // bytes of a turned row: 16 fp64, padded
constexpr int kERow = 640;                      // bytes of a row of lane sums: 64 fp64, padded
constexpr int kTriBytes = 64 * 65 / 2 * 4;      // a block's P when no prefix is longer than 64

struct TurnedArgs {
    const float* tab;          // [M][nbs][C][K] 1 - F(x_{k+1}); affine mode: [M][C][K]
    const int64_t* queue_off;  // [M+1]
    const int32_t* cls;        // [N]
    const double* deadline;    // [N]
    const double* now;         // [M]
    const double* width;       // [M]
    const int64_t* cand_off;   // [M+1]
    const int64_t* prob_off;   // [M+1]
    float* P;
    double* E;
    float* EL;
    float* S;
    const int32_t* sup;        // [M][nbs][C][2] first / last bin with mass, or NULL
    const double* cost;        // [N] miss cost per request, or NULL (1)
    const double* c0;          // affine mode: [M] fixed batch overhead (ms); else NULL
    const double* c1;          // affine mode: [M] per-member slope
    double* esum;              // affine mode: [M][np_e][maxcap] sums of 1 - G over kPanel bins
    int np_e;
    int* err;
    double b;
    int C, K, nbs, rect, maxcap;
    int Mg;                    // models the grid covers: all, or the listed ones
    int compact;               // 1: grid model i is act[i]
    int nblk;                  // workgroups per (model, batch size): blocks of 64 prefix lengths
    int bs[ORLOJ_MAX_BATCH_SIZES];
    int act[kMaxActive];       // the models with a non-empty queue (compact)
};

// A kernel's only argument, read where the launch put it: by value, the
// compiler copied its arrays to every lane's scratch memory (2.2 KB a lane).
template <class T>
__device__ __forceinline__ const T& kernel_args() {
    return *(const T*)__builtin_amdgcn_kernarg_segment_ptr();
}

// LDS, byte offsets: the waves' areas (the turned block, or rows of lane
// sums, per-step totals and the list of active steps), the plans, staged P
// (up to 64 prefix lengths) and the tile counter.
struct TurnedLds {
    int wave, tot, list, plan, pst, ctrl, total;
};

__host__ __device__ constexpr TurnedLds turned_lds(int R, int W) {
    TurnedLds l{};
    l.tot = 8 * kERow;
    l.list = l.tot + 512;
    l.wave = 64 * kGtRow;
    l.plan = W * l.wave;
    l.pst = l.plan + 64 * R * 32;
    l.ctrl = l.pst + (R == 1 ? kTriBytes : 0);
    l.total = l.ctrl + 16;
    return l;
}
static_assert(8 * kERow + 512 + 256 <= 64 * kGtRow, "rows of lane sums, totals, list");
// at the end the segments' sums and the waves' E sums take the areas' place
static_assert(2560 + 512 <= turned_lds(1, 1).wave, "a segment a wave");

extern __shared__ __align__(16) unsigned char turned_smem[];

template <class T>
__device__ __forceinline__ T& lds_at(int off) {
    return *reinterpret_cast<T*>(turned_smem + off);
}

template <int... J, class F>
__device__ __forceinline__ void unroll_seq(std::integer_sequence<int, J...>, F&& f) {
    (f(std::integral_constant<int, J>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void unroll(F&& f) {
    unroll_seq(std::make_integer_sequence<int, N>{}, f);
}

// Lane J of each row of 16 lanes, in every lane of the row.
template <int J>
__device__ __forceinline__ unsigned row_bcast(unsigned x) {
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x150 + J, 0xf, 0xf, true);
}

// Sum over the wave (a scalar).
template <int CTRL, int ROWMASK = 0xf>
__device__ __forceinline__ int dpp_i32(int x) {
    return __builtin_amdgcn_update_dpp(0, x, CTRL, ROWMASK, 0xf, true);
}
__device__ __forceinline__ int wave_sum_i32(int x) {
    x += dpp_i32<0x111>(x);
    x += dpp_i32<0x112>(x);
    x += dpp_i32<0x114>(x);
    x += dpp_i32<0x118>(x);
    x += dpp_i32<0x142, 0xa>(x);
    x += dpp_i32<0x143, 0xc>(x);
    return __builtin_amdgcn_readlane(x, 63);
}

// x rounded to a multiple of 2^-40, for |x| < 2048: sums of such values
// below 2^13 are exact in any order.
__device__ __forceinline__ double round_e(double x) {
    constexpr double kM = 6144.0;
    return (x + kM) - kM;
}

__device__ __forceinline__ unsigned long long lanes_below(int lane) { return (1ull << lane) - 1ull; }

// 1 - exp(-x) for x >= 0.  Every lane's x is small where a bin is short
// against the anticipated delay (the usual case): a Taylor polynomial, whose
// remainder is below 2^-57 of the value for x <= 1/64, instead of the
// library's longer chain.
__device__ __forceinline__ double one_minus_exp(double x) {
    if (__all(x <= 0x1p-6)) {
        double p = 1.0 / 40320.0;
        p = fma(-x, p, 1.0 / 5040.0);
        p = fma(-x, p, 1.0 / 720.0);
        p = fma(-x, p, 1.0 / 120.0);
        p = fma(-x, p, 1.0 / 24.0);
        p = fma(-x, p, 1.0 / 6.0);
        p = fma(-x, p, 0.5);
        p = fma(-x, p, 1.0);
        return x * p;
    }
    return -expm1(-x);
}

// One wave's members: member m in lane m % 64 of register m / 64.
template <int R>
struct TurnedWave {
    const unsigned char* tab;  // the rows of this (model, batch size)
    int K, lane, n1, blk;      // members, and the block of prefix lengths scored
    int area;                  // this wave's LDS
    TurnedLds l;
    unsigned co[R];            // byte offset of the member's row
    int lo[R], hi[R];          // its support

    __device__ __forceinline__ float row_at(unsigned off) const {
        return *reinterpret_cast<const float*>(tab + off);
    }

    __device__ __forceinline__ void load_members(const TurnedArgs& a, int64_t q0, const int32_t* sup_qb) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            co[r] = 0;
            lo[r] = 0;
            hi[r] = K;
            if (r <= blk) {
                const int m = 64 * r + lane;
                int c = m < n1 ? a.cls[q0 + m] : 0;
                if (c < 0 || c >= a.C) c = 0;             // flagged with the member's bin
                co[r] = 4u * (unsigned)c * (unsigned)K;
                if (sup_qb) {
                    lo[r] = sup_qb[2 * (size_t)c];
                    hi[r] = sup_qb[2 * (size_t)c + 1];
                }
            }
        }
    }

    // Sum of G over the valid bins of the NS kETile bins from tile0 on, prefix
    // length 64 blk + lane + 1.  Rows whose support misses the tile are not
    // read: past a row's last bin with mass 1 - F is exactly 0 (G is
    // unchanged), before its first exactly 1 (G becomes 0), so the sums are
    // the same bits with and without the support.  The rows of the next GS
    // steps are on their way while GS are worked on, in two sets of registers
    // that take turns: a copy from one to the other would wait for the loads.
    template <int NS>
    __device__ __forceinline__ double e_tile(int tile0) {
        constexpr int GS = NS == 1 ? 8 : 4;                // steps of a group
        const int tend = min(tile0 + NS * kETile, K);
        unsigned off[2 * NS];
        double G[2 * NS];
#pragma unroll
        for (int j = 0; j < 2 * NS; ++j) {
            const int b = tile0 + 64 * j + lane;           // a load takes 256 bytes of a row
            off[j] = 4u * (unsigned)min(b, K - 1);
            G[j] = b < K ? 1.0 : 0.0;
        }
        auto lane_sum = [&] {
            double s = G[0] + G[1];
#pragma unroll
            for (int j = 2; j < 2 * NS; j += 2) s += G[j] + G[j + 1];
            return s;
        };
        int nstop = 0x7fffffff;                            // first member wholly past the tile
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (r <= blk) {
                const unsigned long long mo = __ballot(64 * r + lane < n1 && tend <= lo[r]);
                if (mo != 0ull) nstop = min(nstop, 64 * r + (int)__ffsll((long long)mo) - 1);
            }
        }
        if (nstop < 64 * blk) return 0.0;
        double before = (double)(tend - tile0);            // before the block's first active member
        double sum = 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (r <= blk) {
                // the active members of this register, in order
                const int m = 64 * r + lane;
                const bool act = m < n1 && m < nstop && hi[r] > tile0;
                const unsigned long long mk = __ballot(act);
                const int cnt = __popcll(mk), rk = __popcll(mk & lanes_below(lane));
                if (act) lds_at<unsigned>(area + l.list + 4 * rk) = co[r];
                wave_lds_fence();
                const unsigned lv = cnt > 0 ? lds_at<unsigned>(area + l.list + 4 * min(lane, cnt - 1)) : 0u;
                const bool rows = r == blk;
                float ta[GS][2 * NS], tb[GS][2 * NS];
                auto load = [&](float (&v)[GS][2 * NS], int g) {
#pragma unroll
                    for (int u = 0; u < GS; ++u) {
                        const unsigned c = (unsigned)__builtin_amdgcn_readlane((int)lv, min(g + u, 63));
#pragma unroll
                        for (int j = 0; j < 2 * NS; ++j) v[u][j] = row_at(c + off[j]);
                    }
                };
                auto steps = [&](const float (&v)[GS][2 * NS], int g) {
#pragma unroll
                    for (int u = 0; u < GS; ++u) {
                        if (g + u < cnt) {
#pragma unroll
                            for (int j = 0; j < 2 * NS; ++j) G[j] = fma(-G[j], (double)v[u][j], G[j]);
                        }
                        if (rows) lds_at<double>(area + u * kERow + 8 * lane) = lane_sum();
                    }
                    if (rows) add_rows<GS>(g);
                };
                load(ta, 0);
#pragma unroll 1
                for (int g = 0; g < cnt; g += 2 * GS) {
                    load(tb, g + GS);
                    steps(ta, g);
                    if (g + GS < cnt) {
                        load(ta, g + 2 * GS);
                        steps(tb, g + GS);
                    }
                }
                if (r + 1 == blk) {
                    // G of the block before: its sum, for the block's first prefixes
                    lds_at<double>(area + 8 * lane) = lane_sum();
                    add_rows<GS>(0);
                    before = lds_at<double>(area + l.tot);
                }
                if (rows) {
                    const int last = rk + (act ? 1 : 0) - 1;   // the last active step up to this one
                    sum = last >= 0 ? lds_at<double>(area + l.tot + 8 * last) : before;
                    if (m >= nstop) sum = 0.0;
                }
                wave_lds_fence();
            }
        }
        return sum;
    }

    // the sums over the lanes of GS rows, to the totals from t0 on
    template <int GS>
    __device__ __forceinline__ void add_rows(int t0) {
        constexpr int L = 64 / GS;                         // lanes a row
        wave_lds_fence();
        const int row = lane / L, at = lane % L;
        double s = 0.0;
#pragma unroll
        for (int j = 0; j < 32 / L; ++j) {
            const double2 v = lds_at<double2>(area + row * kERow + 16 * (L * j + at));
            s = j == 0 ? v.x + v.y : s + (v.x + v.y);
        }
        s += dpp64<0xb1>(s);       // quad_perm 1 0 3 2
        s += dpp64<0x4e>(s);       // quad_perm 2 3 0 1
        s += dpp64<0x141>(s);      // row_half_mirror
        if (L == 16) s += dpp64<0x140>(s);                 // row_mirror
        if (at == 0) lds_at<double>(area + l.tot + 8 * (t0 + row)) = s;
        wave_lds_fence();
    }
};

// A member's constants for Eq. (2), in LDS: read uniformly, one member ahead.
struct alignas(16) Plan {
    double th;      // position inside bin k
    double A;       // cost (1 - d) exp(-b theta w), or cost (1 - d) exp(-b (tau - K w))
    double Bc;      // cost (1 - exp(-b theta w))
    double cc;      // A (1 - d) d^(k - the segment's first bin); 0 in the first segment
};
static_assert(sizeof(Plan) == 32, "plan size");

template <int R, bool AFF, int W>
__device__ __forceinline__ void turned_block(const TurnedArgs& a) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int K = a.K;
    constexpr TurnedLds l = turned_lds(R, W);
    // E tiles handed out.  The barrier comes before the loads: it would wait
    // for them.
    if (tid == 0) lds_at<int>(l.ctrl) = 0;
    __syncthreads();

    const unsigned per_bs = (unsigned)a.Mg * (unsigned)a.nblk;
    const int bi = a.nbs - 1 - (int)(blockIdx.x / per_bs);
    const unsigned rem = blockIdx.x % per_bs;
    const int blk = R > 1 ? a.nblk - 1 - (int)(rem / (unsigned)a.Mg) : 0;
    const int q = a.compact ? a.act[rem % (unsigned)a.Mg] : (int)(rem % (unsigned)a.Mg);
    const int64_t q0 = a.queue_off[q];
    const int64_t N = a.queue_off[q + 1] - q0;
    const int bsz = a.bs[bi];
    int64_t cand = a.cand_off[q], prob = a.prob_off[q];
    const int64_t cap64 = a.rect ? N : (N < bsz ? N : (int64_t)bsz);
    if (cap64 <= 64 * blk || cap64 > a.maxcap || cap64 > 64 * R) return;   // the host sizes both
    const int n1 = min((int)cap64, 64 * (blk + 1));        // members of the block's longest prefix
    const int nb = n1 - 64 * blk;                          // prefix lengths of the block
    const size_t qb = AFF ? (size_t)q : (size_t)q * (size_t)a.nbs + (size_t)bi;

    TurnedWave<R> t;
    t.tab = reinterpret_cast<const unsigned char*>(a.tab + qb * (size_t)a.C * (size_t)K);
    t.K = K;
    t.lane = lane;
    t.n1 = n1;
    t.blk = blk;
    t.l = l;
    t.area = wv * l.wave;
    t.load_members(a, q0, a.sup ? a.sup + qb * (size_t)a.C * 2 : nullptr);
    double tau[R], cost[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int m = 64 * r + lane;
        const bool in = r <= blk && m < n1;
        tau[r] = in ? a.deadline[q0 + m] : 0.0;
        cost[r] = in && a.cost ? a.cost[q0 + m] : 1.0;
    }

    // Affine mode (Eq. (3)): a batch of size s whose slowest member takes l
    // runs c0 + c1 s l: the bin width is c1 s w, the time left tau - c0, and
    // E[L_B] = c0 + c1 s E[max] (Eq. (5)), whose sums come from
    // turned_esum_kernel.  Tabulated mode: c0 = 0, width w.
    const double wq = a.width[q];
    double c0q = 0.0, w = wq;
    bool aok = true;
    if constexpr (AFF) {
        c0q = a.c0[q];
        const double c1 = a.c1[q];
        aok = c0q >= 0.0 && c0q < HUGE_VAL && c1 > 0.0 && c1 < HUGE_VAL;
        w = c1 * (double)bsz * wq;
    }
    const bool wok = wq > 0.0 && wq < HUGE_VAL && aok && w > 0.0 && w < HUGE_VAL;   // else a data error
    const double nowq = a.now[q];
    const double b = a.b, bw = b * w;

    // ---- deadline bins: -1 dead, K beyond the grid
    double th[R], left[R];                                 // position in the bin; time past its left edge
    int kk[R];
    int kmax = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        kk[r] = -2;                                        // no member
        th[r] = left[r] = 0.0;
        if (r <= blk) {
            const int m = 64 * r + lane;
            if (m < n1) {
                const double D = tau[r];
                if (wv == W - 1) {
                    // the member's data errors (once per workgroup)
                    const int c = a.cls[q0 + m];
                    int flag = 0;
                    if (c < 0 || c >= a.C) flag |= kErrClassRange;
                    if (isnan(D)) flag |= kErrDeadlineNaN;
                    if (m > 0 && D < a.deadline[q0 + m - 1]) flag |= kErrUnsorted;
                    if (m == 0 && isnan(nowq)) flag |= kErrNowNaN;
                    if (m == 0 && !(wq > 0.0 && wq < HUGE_VAL)) flag |= kErrWidth;
                    if (m == 0 && !aok) flag |= kErrAffine;
                    if (!(cost[r] >= 0.0 && cost[r] < HUGE_VAL)) flag |= kErrCost;
                    if (flag) atomicOr(a.err, flag);
                }
                kk[r] = -1;
                const double ta = D - nowq - c0q;
                if (ta > 0.0 && wok) {
                    const double u = ta / w, uf = floor(u);
                    if (u >= (double)K) {
                        kk[r] = K;
                        left[r] = ta - (double)K * w;
                    } else {
                        kk[r] = (int)uf;
                        th[r] = u - uf;
                        left[r] = th[r] * w;
                    }
                }
                kmax = max(kmax, min(kk[r], K - 1));
            }
        }
        if (!(cost[r] >= 0.0 && cost[r] < HUGE_VAL)) cost[r] = 0.0;
    }
    kmax = __builtin_amdgcn_readfirstlane(wave_max_i32(kmax));

    // lane (row, i) of a segment: prefix length nidx + 1, part `part` of a block
    const int S = nb <= 16 ? 4 : nb <= 32 ? 2 : 1, RG = 4 / S;
    const int row = lane >> 4, ri = lane & 15, part = row % S, grp = row / S;
    const int nrel = 16 * grp + ri, nidx = nrel < nb ? 64 * blk + nrel : -1;
    const int row0 = 16 * grp * S + ri;                    // the lane of part 0 of this prefix length
    // the member region: blocks of 16 S bins up to the last deadline, the
    // same number of them for each segment
    const int nblocks = kmax / (16 * S) + 1, per = (nblocks + W - 1) / W;
    const int Ls = per * 16 * S, kend0 = nblocks * 16 * S, lseg = (nblocks - 1) / per;
    const double omd = one_minus_exp(bw), d = 1.0 - omd;
    double accP = 0.0, accN = 0.0, accC = 0.0, es = 0.0;   // this wave's segment: sums of P, N, C and G
    double Y = 0.0, gpc = 0.0;                             // discounted prefix and G before the block

    // The rows of a block of bins are loaded 16 members at a time per DPP row:
    // passes over the members before this block of prefix lengths, then the
    // block's own.  An item is one pass; the next item's rows are on their way
    // while one is worked on.
    const int k0 = wv * Ls, kend = min(k0 + Ls, kend0);
    const int passes = blk * S + 1;
    float tv[16], tn[16];
    auto issue = [&](int base, int p) {
        unsigned c = t.co[0];
#pragma unroll
        for (int r = 1; r < R; ++r) c = p / S == r ? t.co[r] : c;
        if (S > 1) c = (unsigned)__shfl((int)c, 16 * ((p % S) * RG + grp) + ri, 64);
        // (the last entry of a row is 0: bins past the grid hold G = 1)
        const unsigned o = 4u * (unsigned)min(base + 16 * part + ri, K - 1);
        unroll<16>([&](auto j) { tn[decltype(j)::value] = t.row_at(row_bcast<decltype(j)::value>(c) + o); });
    };
    // the block before the segment only gives G at its last bin
    int base = k0 - (wv > 0 ? 16 * S : 0), pass = 0;
    if (wv <= lseg) issue(base, 0);

    // this batch size's block of candidates and member slots starts after
    // those of the batch sizes before it (their sizes are a memory round trip)
    {
        int dc = 0, dp = 0;                                // (caps are at most ORLOJ_MAX_PREFIX)
        for (int j0 = 0; j0 < bi; j0 += 64) {
            const int j = j0 + lane;
            if (j < bi) {
                const int c = (int)(a.rect ? N : (N < a.bs[j] ? N : (int64_t)a.bs[j]));
                dc += c;
                dp += c * (c + 1) / 2;
            }
        }
        cand += wave_sum_i32(dc);
        prob += wave_sum_i32(dp);
    }
    float* const Pn = a.P + prob + (int64_t)nidx * (nidx + 1) / 2;   // this prefix length's P (R > 1)

    // ---- member segments, one per wave
    if (wv <= lseg) {
        __builtin_amdgcn_s_setprio(3);                     // the others wait for these
        int me = 0, mb = 0;                                // its members
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int k = min(max(kk[r], 0), K - 1);
            me += __popcll(__ballot(kk[r] > -2 && k < k0));
            mb += __popcll(__ballot(kk[r] > -2 && (k < k0 + Ls || wv == lseg)));
        }
        me = __builtin_amdgcn_readfirstlane(me);
        mb = __builtin_amdgcn_readfirstlane(mb);
        const double d2 = d * d, d4 = d2 * d2, d8 = d4 * d4, d16 = d8 * d8;
        // its members' constants
#pragma unroll 1
        for (int r0 = me >> 6; 64 * r0 < mb; ++r0) {
            Plan p;
            double lf = left[0], cm = cost[0];
            int k = kk[0];
            p.th = th[0];
#pragma unroll
            for (int r = 1; r < R; ++r) {
                lf = r0 == r ? left[r] : lf;
                cm = r0 == r ? cost[r] : cm;
                k = r0 == r ? kk[r] : k;
                p.th = r0 == r ? th[r] : p.th;
            }
            const double m1 = one_minus_exp(b * lf);
            double e1 = 1.0 - m1;
            if (__any(e1 < 0.5)) e1 = exp(-b * lf);        // its own digits where it is small
            p.A = k >= 0 ? cm * omd * e1 : 0.0;
            p.Bc = k >= 0 && k < K ? cm * m1 : 0.0;
            p.cc = 0.0;
            if (k0 > 0) p.cc = p.A * omd * exp(-bw * (double)(k - k0));
            const int m = 64 * r0 + lane;
            if (m >= me && m < mb) lds_at<Plan>(l.plan + 32 * m) = p;
        }
        wave_lds_fence();
        auto plan_of = [&](int m) -> const Plan& { return lds_at<Plan>(l.plan + 32 * min(m, n1 - 1)); };
        Plan cur = plan_of(me), nxt = plan_of(me + 1);
        auto bin_of = [&](int m) {
            if (m >= mb) return 0x7fffffff;
            int k = kk[0];
#pragma unroll
            for (int r = 1; r < R; ++r) k = (m >> 6) == r ? kk[r] : k;
            return (int)__builtin_amdgcn_readlane(k, m & 63);
        };
        int ck = bin_of(me), cn = bin_of(me + 1);          // the next two members' bins
        // member `me` at a bin with G = gp on its left edge, gc on its right
        // one and discounted prefix y two bins before: for the lanes of part h
        auto event = [&](double y, double gp, double gc, int h) {
            if (nidx >= me && part == h) {
                const double dg = gc - gp;
                double P = fma(cur.th, dg, gp);
                const double num = fma(cur.A, fma(-omd, y, gp), cur.Bc * dg);
                P = ck >= 0 ? P : 0.0;                     // dead: its constants are 0 as well
                accP += P;
                accN += num;
                accC += cur.cc;
                if constexpr (R == 1) lds_at<float>(l.pst + 2 * nrel * (nrel + 1) + 4 * me) = (float)P;
                else Pn[me] = (float)P;
            }
            ++me;
            ck = cn;
            cn = bin_of(me + 1);
            cur = nxt;
            nxt = plan_of(me + 1);
        };
        double Gs = 1.0;                                   // product of the members before
        while (base < kend) {
#pragma unroll
            for (int j = 0; j < 16; ++j) tv[j] = tn[j];
            const int pb = base, pp = pass;
            if (++pass == passes) {
                pass = 0;
                base += 16 * S;
            }
            if (base < kend) issue(base, pass);
            double Q[16];
#pragma unroll
            for (int j = 0; j < 16; ++j)
                Q[j] = j == 0 ? 1.0 - (double)tv[0] : fma(-Q[j - 1], (double)tv[j], Q[j - 1]);
            if (pp + 1 < passes) {
                for (int h = 0; h < RG; ++h) Gs *= __shfl(Q[15], 16 * (h * S + part) + ri, 64);
                continue;
            }
            for (int h = 0; h < RG - 1; ++h) {
                const double x = __shfl(Q[15], 16 * (h * S + part) + ri, 64);
                Gs = grp > h ? Gs * x : Gs;
            }
            // turned: lane (row, i) takes 16 bins of its prefix length
            double g[16];
            const int wr = t.area + 16 * row * kGtRow + 8 * ri, rd = t.area + lane * kGtRow;
#pragma unroll
            for (int j = 0; j < 16; ++j) lds_at<double>(wr + j * kGtRow) = Gs * Q[j];
            wave_lds_fence();
#pragma unroll
            for (int j = 0; j < 16; ++j) g[j] = lds_at<double>(rd + 8 * j);
            wave_lds_fence();
            Gs = 1.0;
            double gp0 = gpc;
            if (S > 1) {
                const double gl = __shfl(g[15], lane < 16 ? lane : lane - 16, 64);
                gp0 = part == 0 ? gpc : gl;
                gpc = __shfl(g[15], row0 + 16 * (S - 1), 64);
            } else {
                gpc = g[15];
            }
            if (pb < k0) continue;
            double Ys = Y;
            if (S > 1 || ck > pb + 15) {
                // no member here, or several parts: the discounted prefix
                // first, before each part and after the block
                double y = 0.0, gp = gp0;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    y = fma(y, d, gp);
                    gp = g[i];
                    es += gp;
                }
                if (S > 1) {
                    double Yr = Y;
                    for (int h = 0; h < S; ++h) {
                        Ys = part == h ? Yr : Ys;
                        Yr = fma(Yr, d16, __shfl(y, row0 + 16 * h, 64));
                    }
                    Y = Yr;
                } else {
                    Y = fma(Y, d16, y);
                }
                if (ck > pb + 16 * S - 1) continue;
            }
            for (int h = 0; h < S; ++h) {
                const int bh = pb + 16 * h;
                if (ck > bh + 15) continue;
                double y = Ys, gp = gp0;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    while (ck <= bh + i) event(y, gp, g[i], h);
                    y = fma(y, d, gp);
                    gp = g[i];
                    if (S == 1) es += gp;
                }
                if (S == 1) Y = y;
            }
        }
        // beyond the grid: at bin K (also whatever unsorted deadlines left over)
        while (me < mb) event(Y, gpc, gpc, 0);
        __builtin_amdgcn_s_setprio(0);
    }

    // ---- E tiles past the member region (tabulated mode); lane n: prefix
    // length 64 blk + n + 1
    double eacc = 0.0;
    if constexpr (!AFF) {
        // Wide where there are many: a tile is a chain of latencies whatever its
        // width.  The width does not depend on the launch, so neither does the
        // rounding of the sums.
        const bool wide = K - kend0 > kWideFrom;
        const int width = wide ? kWide * kETile : kETile;
        for (;;) {
            int T = 0;
            if (lane == 0) T = atomicAdd(&lds_at<int>(l.ctrl), 1);
            const int tile0 = kend0 + width * __builtin_amdgcn_readfirstlane(T);
            if (tile0 >= K) break;
            const double G = wide ? t.template e_tile<kWide>(tile0) : t.template e_tile<1>(tile0);
            eacc += round_e((double)(min(tile0 + width, K) - tile0) - G);
        }
    }

    // ---- join the segments and the waves' E sums
    double v[4] = {accP, accN, accC, es};
    if (S > 1 && wv <= lseg) {
#pragma unroll
        for (int f = 0; f < 4; ++f) {
            const double x = v[f];
            v[f] = __shfl(x, row0, 64);
            for (int h = 1; h < S; ++h) v[f] += __shfl(x, row0 + 16 * h, 64);
        }
    }
    __syncthreads();
    const int ework = 2560 * W;
    if (!AFF) lds_at<double>(ework + 512 * wv + 8 * lane) = eacc;
    if (wv <= lseg && part == 0) {
        // 1 - G over the segment (bins past the grid hold G = 1)
        v[3] = round_e((double)(min(wv * Ls + Ls, kend0) - wv * Ls) - v[3]);
        const int at = 2560 * wv + 8 * nrel;
#pragma unroll
        for (int f = 0; f < 4; ++f) lds_at<double>(at + 512 * f) = v[f];
        lds_at<double>(at + 2048) = Y;
    }
    if constexpr (R == 1) {
        for (int i = tid; i < nb * (nb + 1) / 2; i += (int)blockDim.x) a.P[prob + i] = lds_at<float>(l.pst + 4 * i);
    }
    double dL = 0.0;
    if (lseg > 0 && wv == 0) dL = exp(-bw * (double)Ls);
    __syncthreads();
    if (wv == 0 && lane < nb) {
        // A priority's terms are A (gp - omd y) + Bc (gc - gp), over b w; the
        // prefix carried into a segment adds cc / A of it to every omd y
        double Yin = 0.0, P = 0.0, Nn = 0.0, E = 0.0;
        for (int seg = 0; seg <= lseg; ++seg) {
            const int at = 2560 * seg + 8 * lane;
            P += lds_at<double>(at);
            const double n0 = lds_at<double>(at + 512);
            Nn += seg > 0 ? fma(-lds_at<double>(at + 1024), Yin, n0) : n0;
            E += lds_at<double>(at + 1536);
            Yin = fma(Yin, dL, lds_at<double>(at + 2048));
        }
        Nn = wok ? Nn / bw : 0.0;
        const int n = 64 * blk + lane;
        if constexpr (AFF) {
            const double* ep = a.esum + (size_t)q * (size_t)a.np_e * (size_t)a.maxcap + n;
            E = 0.0;
            for (int p = 0; p < a.np_e; ++p) E += ep[(size_t)p * (size_t)a.maxcap];
        } else {
            for (int u = 0; u < W; ++u) E += lds_at<double>(ework + 512 * u + 8 * lane);
        }
        const double el = c0q + w * (0.5 + E);
        a.E[cand + n] = P;
        a.EL[cand + n] = (float)el;
        a.S[cand + n] = (float)(Nn / el);
    }
}

template <int R, bool AFF, int W>
__global__ __launch_bounds__(64 * W) void turned_kernel(const TurnedArgs) {
    turned_block<R, AFF, W>(kernel_args<TurnedArgs>());
}

// The sums of 1 - G behind E[max] in the affine mode (see emax_kernel), for
// turned_kernel: one workgroup of two waves per (model, kPanel bins, block
// of prefix lengths).
template <int R>
__global__ __launch_bounds__(128) void turned_esum_kernel(const TurnedArgs) {
    const TurnedArgs& a = kernel_args<TurnedArgs>();
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned per = (unsigned)a.Mg * (unsigned)a.np_e;
    const int blk = R > 1 ? a.nblk - 1 - (int)(blockIdx.x / per) : 0;
    const unsigned rem = blockIdx.x % per;
    const int q = a.compact ? a.act[rem / (unsigned)a.np_e] : (int)(rem / (unsigned)a.np_e);
    const int p = (int)(rem % (unsigned)a.np_e);
    const int64_t q0 = a.queue_off[q];
    const int64_t N = a.queue_off[q + 1] - q0;
    const int bsz = a.bs[a.nbs - 1];                       // the longest prefix (batch sizes increase)
    const int64_t cap64 = a.rect ? N : (N < bsz ? N : (int64_t)bsz);
    if (cap64 <= 64 * blk || cap64 > a.maxcap || cap64 > 64 * R) return;
    TurnedWave<R> t;
    t.tab = reinterpret_cast<const unsigned char*>(a.tab + (size_t)q * (size_t)a.C * (size_t)a.K);
    t.K = a.K;
    t.lane = lane;
    t.n1 = min((int)cap64, 64 * (blk + 1));
    t.blk = blk;
    t.l = turned_lds(R, 2);
    t.area = wv * t.l.wave;
    t.load_members(a, q0, a.sup ? a.sup + (size_t)q * (size_t)a.C * 2 : nullptr);
    static_assert(kPanel == 2 * kETile, "a tile per wave");
    const int tile0 = p * kPanel + wv * kETile;
    double e = 0.0;
    if (tile0 < a.K) e = round_e((double)(min(tile0 + kETile, a.K) - tile0) - t.template e_tile<1>(tile0));
    __syncthreads();
    lds_at<double>(512 * wv + 8 * lane) = e;
    __syncthreads();
    const int n = 64 * blk + lane;
    if (wv == 0 && n < t.n1)
        a.esum[((size_t)q * (size_t)a.np_e + (size_t)p) * (size_t)a.maxcap + n] = e + lds_at<double>(512 + 8 * lane);
}

// ---------------------------------------------------------------------------
// select_kernel: one workgroup per model; thread i reads candidates i,
// i + kSelThreads, ... (coalesced) and finds its (batch size, n) from the
// block starts of the model's batch sizes.
// ---------------------------------------------------------------------------
struct SelectArgs {
    const int64_t* queue_off;
    const int64_t* cand_off;
    const float* S;
    // scheduling rounds (mapped host memory, or NULL): after its writes,
    // each workgroup g makes them visible to the host and writes `round`
    // to done[g], so the host can see the round finish without waiting for
    // the stream
    int32_t* done;
    int32_t round;
    int32_t* sel_n;
    int32_t* sel_bs;
    float* sel_score;
    int nbs, rect;
    int M;
    int n_act;                 // compact: workgroup g < n_act selects for act[g],
    int compact;               //   workgroup n_act clears the models with an empty queue
    int bs[ORLOJ_MAX_BATCH_SIZES];
    int act[kMaxActive];
};

struct Best {
    float s;
    int n;
    int bs;
};

__device__ __forceinline__ bool better(const Best& x, const Best& y) {
    // larger score; exact ties: larger n, then smaller batch size (n = 0:
    // no candidate).  Written without branches, and applied with selects
    // (take_if_better): the branchy form of the update lost the new n on
    // some paths when compiled for gfx950.
    const bool sgt = x.s > y.s, seq = x.s == y.s;
    const bool tie = seq && (x.n > y.n || (x.n == y.n && x.bs < y.bs));
    return x.n != 0 && (y.n == 0 || sgt || tie);
}

__device__ __forceinline__ void take_if_better(Best& best, const Best& c) {
    const bool t = better(c, best);
    best.s = t ? c.s : best.s;
    best.n = t ? c.n : best.n;
    best.bs = t ? c.bs : best.bs;
}

// 16 waves per model: the kernel is a chain of latencies (block starts,
// candidate loads, reductions), so more threads per model shorten it.
constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / 64;

__global__ __launch_bounds__(kSelThreads) void select_kernel(const SelectArgs a) {
    __shared__ int64_t s_start[ORLOJ_MAX_BATCH_SIZES + 1];
    __shared__ Best s_best[kSelWaves];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    if (a.compact && (int)blockIdx.x >= a.n_act) {
        // the workgroup after the selecting ones: no batch for the models
        // with an empty queue (not listed).  Its clears, and their fence,
        // run beside the selections.
        for (int m = tid; m < a.M; m += kSelThreads) {
            if (a.queue_off[m + 1] == a.queue_off[m]) {
                a.sel_n[m] = 0;
                a.sel_bs[m] = 0;
                a.sel_score[m] = 0.0f;
            }
        }
        if (a.done) {
            // the clears reach the host before the flag (every thread that
            // cleared fences its own writes)
            if (tid < a.M) __threadfence_system();
            __syncthreads();
            if (tid == 0) __hip_atomic_store(&a.done[blockIdx.x], a.round, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
        return;
    }
    const int q = a.compact ? a.act[blockIdx.x] : (int)blockIdx.x;
    __shared__ int64_t s_wsum[kSelWaves];
    const int64_t N = a.queue_off[q + 1] - a.queue_off[q];
    // block starts: an exclusive scan of the prefix caps over the batch
    // sizes, kSelThreads at a time (a workgroup scan of per-wave scans)
    int64_t carry = 0;
    for (int b0 = 0; b0 < a.nbs; b0 += kSelThreads) {
        const int bi = b0 + tid;
        const int bsz = bi < a.nbs ? a.bs[bi] : 0;
        const int64_t cap = bi < a.nbs ? (a.rect ? N : (N < bsz ? N : (int64_t)bsz)) : 0;
        const int64_t incl = wave_incl_scan_u64((uint64_t)cap, lane);
        if (lane == 63) s_wsum[wv] = incl;
        __syncthreads();
        int64_t before = carry;
        for (int w = 0; w < wv; ++w) before += s_wsum[w];
        if (bi < a.nbs) s_start[bi] = before + incl - cap;
        for (int w = 0; w < kSelWaves; ++w) carry += s_wsum[w];
        __syncthreads();
    }
    if (tid == 0) s_start[a.nbs] = carry;
    __syncthreads();
    const float* S = a.S + a.cand_off[q];
    Best best{0.0f, 0, 0};
    // candidates i = tid, tid + kSelThreads, ... (coalesced); a candidate's
    // (batch size, n) from the block starts.  The comparison is a total
    // order, so the pick does not depend on the order of the visits.
    const int64_t total = s_start[a.nbs];
    for (int64_t i = tid; i < total; i += kSelThreads) {
        const float sc = S[i];
        int lo = 0, hi = a.nbs - 1;          // last bi with s_start[bi] <= i
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (s_start[mid] <= i) lo = mid; else hi = mid - 1;
        }
        const int n = (int)(i - s_start[lo]) + 1;
        const int bsz = a.bs[lo];
        if (n <= bsz && sc == sc)            // NaN never wins
            take_if_better(best, Best{sc, n, bsz});
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        Best o;
        o.s = __shfl_xor(best.s, off, 64);
        o.n = __shfl_xor(best.n, off, 64);
        o.bs = __shfl_xor(best.bs, off, 64);
        take_if_better(best, o);
    }
    if (lane == 0) s_best[wv] = best;
    __syncthreads();
    if (wv == 0) {
        // the waves' picks, reduced across the first kSelWaves lanes
        best = lane < kSelWaves ? s_best[lane] : Best{0.0f, 0, 0};
#pragma unroll
        for (int off = kSelWaves / 2; off > 0; off >>= 1) {
            Best o;
            o.s = __shfl_xor(best.s, off, 64);
            o.n = __shfl_xor(best.n, off, 64);
            o.bs = __shfl_xor(best.bs, off, 64);
            take_if_better(best, o);
        }
        if (lane == 0) {
            if (best.n > 0 && best.s > 0.0f) {
                a.sel_n[q] = best.n;
                a.sel_bs[q] = best.bs;
                a.sel_score[q] = best.s;
            } else {
                a.sel_n[q] = 0;
                a.sel_bs[q] = 0;
                a.sel_score[q] = 0.0f;
            }
        }
    }
    if (a.done) {
        // the selection (written by thread 0, above) reaches the host before
        // the flag
        if (tid == 0) {
            __threadfence_system();
            __hip_atomic_store(&a.done[blockIdx.x], a.round, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}

}  // namespace

// ===========================================================================
// C ABI
// ===========================================================================
namespace {

// ---------------------------------------------------------------------------
// Scheduler iteration (§3.2 Algorithm 1) with the paper's own priority.
//
// laws_kernel: one workgroup per (model, batch size).  Thread t owns the VPT
// consecutive bins [t*VPT, t*VPT + VPT).  It forms the model's class mix
// F_mix = sum_c pi_c F_c in fp64, then for each class the CDF of a
// request's batch latency, F_c F_mix^(s-1) (the request plus s-1 members
// drawn from the mix; §4.2.1: the max of k identical variables has CDF
// F^k), and its discounted prefix Z(k) = sum_{i<=k} G(x_{i+1}) d^(k-i),
// d = e^{-b w}: an in-thread fp64 prefix, a weighted DPP scan across the
// wave and a weighted combination across the four waves.  Block 0 of each
// model also writes the model-wide E[L] of F_mix^s (§4.3).
//
// Bound by HBM: the table is read twice and two tables are written.  The next
// class's row is loaded while a class is worked on (the classes are a serial
// chain of loads and a barrier otherwise), and the rows leave in whole lines,
// turned in LDS.  Tables and laws of 32 models x 64 batch sizes x 32 classes x
// 4096 bins, us: 1425 before, 1374 with the row loaded ahead, 1248 with both.
// ---------------------------------------------------------------------------
struct LawArgs {
    const float* tab;          // [M][nbs][C][K] 1 - F(x_{k+1})
    const double* weights;     // [M][C] class mix, or NULL (uniform)
    const double* width;       // [M]
    float* law;                // [M][nbs][C][K]
    float* disc;               // [M][nbs][C][K]
    float* model_el;           // [M][nbs]
    int* err;
    double* pm;                // laws_mix_kernel: [pairs][K] F_mix^(s-1)
    int vshift;                // laws_mix_kernel: log2 of laws_kernel's bins per thread
    double b;
    int M, C, K, nbs;
    int bs[ORLOJ_MAX_BATCH_SIZES];
};

// One thread's VPT consecutive entries of a table row: F = 1 - t, and 1
// beyond the row's end.  Whole float4s when the row length is a multiple
// of 4 (rows and thread chunks are then 16-byte aligned).
template <int VPT>
__device__ __forceinline__ void load_cdf_chunk(double (&F)[VPT], const float* __restrict__ t, int base,
                                               int K) {
    if constexpr (VPT % 4 == 0) {
        if ((K & 3) == 0) {
#pragma unroll
            for (int j = 0; j < VPT; j += 4) {
                if (base + j < K) {
                    const float4 v = *reinterpret_cast<const float4*>(t + base + j);
                    F[j] = 1.0 - (double)v.x; F[j + 1] = 1.0 - (double)v.y;
                    F[j + 2] = 1.0 - (double)v.z; F[j + 3] = 1.0 - (double)v.w;
                } else {
                    F[j] = F[j + 1] = F[j + 2] = F[j + 3] = 1.0;
                }
            }
            return;
        }
    }
#pragma unroll
    for (int j = 0; j < VPT; ++j) F[j] = base + j < K ? 1.0 - (double)t[base + j] : 1.0;
}

// One thread's VPT consecutive entries of a row as they are (0 past its end:
// F = 1), with load_cdf_chunk's accesses.
template <int VPT>
__device__ __forceinline__ void load_row_chunk(float (&v)[VPT], const float* __restrict__ t, int base,
                                               int K) {
    if constexpr (VPT % 4 == 0) {
        if ((K & 3) == 0) {
#pragma unroll
            for (int j = 0; j < VPT; j += 4) {
                const bool in = base + j < K;
                const float4 x = in ? *reinterpret_cast<const float4*>(t + base + j)
                                    : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                v[j] = x.x; v[j + 1] = x.y; v[j + 2] = x.z; v[j + 3] = x.w;
            }
            return;
        }
    }
#pragma unroll
    for (int j = 0; j < VPT; ++j) v[j] = base + j < K ? t[base + j] : 0.0f;
}

// Store one thread's VPT entries (those below K) of a row.
template <int VPT>
__device__ __forceinline__ void store_chunk(float* __restrict__ o, const float (&v)[VPT], int base, int K) {
    if constexpr (VPT % 4 == 0) {
        if ((K & 3) == 0) {
#pragma unroll
            for (int j = 0; j < VPT; j += 4)
                if (base + j < K)
                    *reinterpret_cast<float4*>(o + base + j) = make_float4(v[j], v[j + 1], v[j + 2], v[j + 3]);
            return;
        }
    }
#pragma unroll
    for (int j = 0; j < VPT; ++j)
        if (base + j < K) o[base + j] = v[j];
}

// store_chunk for a wave's lanes together: with more than four entries a lane,
// the lanes' float4s lie 4 VPT bytes apart; turned in LDS, a store writes 1 KB
// of the row.  Rows of LDS are padded by a float4 against bank conflicts.
template <int VPT>
constexpr int kTurnedRow = VPT % 4 == 0 && VPT > 4 ? VPT + 4 : 0;

template <int VPT>
__device__ __forceinline__ void store_row(float* __restrict__ o, const float (&v)[VPT], int base, int K,
                                          float* turn) {
    if constexpr (kTurnedRow<VPT> != 0) {
        if ((K & 3) == 0) {
            constexpr int P = VPT / 4;
            const int lane = threadIdx.x & 63, first = base - lane * VPT;
#pragma unroll
            for (int j = 0; j < VPT; j += 4)
                *reinterpret_cast<float4*>(turn + lane * kTurnedRow<VPT> + j) =
                    make_float4(v[j], v[j + 1], v[j + 2], v[j + 3]);
            wave_lds_fence();
#pragma unroll
            for (int i = 0; i < P; ++i) {
                const int f = 64 * i + lane;
                const float4 x =
                    *reinterpret_cast<const float4*>(turn + f / P * kTurnedRow<VPT> + f % P * 4);
                if (first + 4 * f < K) *reinterpret_cast<float4*>(o + first + 4 * f) = x;
            }
            wave_lds_fence();
            return;
        }
    }
    store_chunk<VPT>(o, v, base, K);
}

template <int VPT, bool AHEAD>
__global__ __launch_bounds__(kThreads) void laws_kernel(const LawArgs a) {
    __shared__ float s_wave[2][kWaves];   // of a class, by its parity
    __shared__ __align__(16) float s_turn[kWaves][kTurnedRow<VPT> ? 64 * kTurnedRow<VPT> : 4];
    __shared__ double s_el[kWaves];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int q = (int)(blockIdx.x / (unsigned)a.nbs);
    const int bi = (int)(blockIdx.x % (unsigned)a.nbs);
    const int K = a.K, C = a.C;
    const int s = a.bs[bi];
    const double w = a.width[q];
    const double d = exp(-a.b * w);
    const int base = tid * VPT;
    const size_t row0 = ((size_t)q * (size_t)a.nbs + (size_t)bi) * (size_t)C;

    // class mix and its powers at this thread's bins (padding bins: F = 1)
    double mix[VPT];
#pragma unroll
    for (int j = 0; j < VPT; ++j) mix[j] = 0.0;
    double wsum = 0.0;
    bool wbad = false;
    for (int c = 0; c < C; ++c) {
        const double wc = a.weights ? a.weights[(size_t)q * C + c] : 1.0;
        wbad |= !(wc >= 0.0) || isinf(wc);
        wsum += wc;
    }
    if (wbad || !(wsum > 0.0)) {
        if (tid == 0) atomicOr(a.err, kErrWeights);
        wsum = 1.0;
    }
    for (int c = 0; c < C; ++c) {
        const double pc = (a.weights ? a.weights[(size_t)q * C + c] : 1.0) / wsum;
        double F[VPT];
        load_cdf_chunk<VPT>(F, a.tab + (row0 + (size_t)c) * (size_t)K, base, K);
#pragma unroll
        for (int j = 0; j < VPT; ++j) mix[j] = fma(pc, F[j], mix[j]);
    }
    double pm[VPT];
    double el = 0.0;
#pragma unroll
    for (int j = 0; j < VPT; ++j) {
        pm[j] = s > 1 ? pow(mix[j], (double)(s - 1)) : 1.0;
        if (base + j < K) el += fma(-pm[j], mix[j], 1.0);
    }
    // model-wide E[L] = w (1/2 + sum_k (1 - F_mix^s(x_{k+1})))
    for (int o = 32; o > 0; o >>= 1) el += __shfl_xor(el, o, 64);
    if (lane == 0) s_el[wv] = el;
    __syncthreads();
    if (tid == 0) {
        double tot = 0.0;
        for (int i = 0; i < kWaves; ++i) tot += s_el[i];
        a.model_el[(size_t)q * a.nbs + bi] = (float)(w * (0.5 + tot));
    }

    // scan constants: a thread chunk spans VPT bins
    const float log2d = (float)(-a.b * w * 1.4426950408889634);
    float rp[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) rp[i] = exp2_hw(log2d * (float)(VPT << i));
    const float w15 = exp2_hw(log2d * (float)(VPT * ((lane & 15) + 1)));
    const float w31 = exp2_hw(log2d * (float)(VPT * (lane >= 32 ? lane - 31 : 0)));
    const float d_wave = exp2_hw(log2d * (float)(64 * VPT));

    float t[VPT];   // AHEAD: the next class's row, loaded while a class is worked on
    if (AHEAD) load_row_chunk<VPT>(t, a.tab + row0 * (size_t)K, base, K);
    for (int c = 0; c < C; ++c) {
        const size_t r = (row0 + (size_t)c) * (size_t)K;
        double g[VPT];
        double z = 0.0;
        if (!AHEAD) load_row_chunk<VPT>(t, a.tab + r, base, K);
#pragma unroll
        for (int j = 0; j < VPT; ++j) g[j] = (1.0 - (double)t[j]) * pm[j];
        if (AHEAD && c + 1 < C) load_row_chunk<VPT>(t, a.tab + r + K, base, K);
#pragma unroll
        for (int j = 0; j < VPT; ++j) {
            z = fma(z, d, g[j]);
        }
        // in-wave weighted scan of the chunk totals, then across the waves
        const float A = wave_wscan((float)z, rp, w15, w31);
        if (lane == 63) s_wave[c & 1][wv] = A;
        __syncthreads();
        float carry = 0.0f;   // discounted sum of the earlier waves' bins, at the end of the last one
#pragma unroll
        for (int i = 0; i < kWaves; ++i)
            if (i < wv) carry = fmaf(carry, d_wave, s_wave[c & 1][i]);
        // prefix up to the end of the previous thread chunk
        const float prev = __shfl_up(A, 1, 64);
        const float before = (lane > 0 ? prev : 0.0f) + carry * exp2_hw(log2d * (float)(VPT * lane));
        double zz = (double)before;
        float lv[VPT], dv[VPT];
#pragma unroll
        for (int j = 0; j < VPT; ++j) {
            zz = fma(zz, d, g[j]);
            lv[j] = (float)g[j];
            dv[j] = (float)zz;
        }
        store_row<VPT>(a.law + r, lv, base, K, s_turn[wv]);
        store_row<VPT>(a.disc + r, dv, base, K, s_turn[wv]);
    }
}

// Short rows of few pairs load a class's row in its turn: the wait for one
// loaded ahead comes after the stores of the class before and costs more than
// it hides (64 pairs x 16 classes x 64 bins 18.0 us with the row ahead, 17.2
// without; 256 x 16 x 1000 33.9 against 36.4, 2048 x 16 x 1000 158 against 165).
template <int VPT>
void launch_laws(const LawArgs& a, unsigned pairs, hipStream_t st) {
    if constexpr (VPT <= 4) {
        if (pairs <= (VPT < 4 ? 512u : 128u)) {
            hipLaunchKernelGGL((laws_kernel<VPT, false>), dim3(pairs), dim3(kThreads), 0, st, a);
            return;
        }
    }
    hipLaunchKernelGGL((laws_kernel<VPT, true>), dim3(pairs), dim3(kThreads), 0, st, a);
}

// ---------------------------------------------------------------------------
// laws_mix_kernel and laws_row_kernel: laws_kernel's outputs when the pairs
// are few (law_split).  laws_kernel walks a pair's classes one after another
// in one workgroup; here one workgroup per pair forms the class mix and its
// power per bin (to scratch) and the model-wide E[L], and then every row has
// a workgroup of its own.  Table and laws, us: 1 model x 64 batch sizes x 32
// classes x 1024 bins 44 -> 24, 2 x 16 x 32 x 4096 106 -> 52, 3 x 48 x 21 x
// 1501 101 -> 70, 8 x 32 x 16 x 1000 35 -> 32.
// ---------------------------------------------------------------------------
constexpr int kMixThreads = 1024;

// VEC: four bins a thread (rows start on 16 bytes), else one.
template <bool VEC>
__global__ __launch_bounds__(kMixThreads) void laws_mix_kernel(const LawArgs a) {
    constexpr int V = VEC ? 4 : 1;
    // each bin's 1 - F_mix^s; an entry's gap after each of laws_kernel's chunks
    // against bank conflicts
    extern __shared__ __align__(16) double s_bin[];
    __shared__ double s_el[kWaves];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int pair = (int)blockIdx.x;
    const int q = pair / a.nbs;
    const int K = a.K, C = a.C;
    const int s = a.bs[pair % a.nbs];
    const double w = a.width[q];
    const float* rows = a.tab + (size_t)pair * (size_t)C * (size_t)K;
    double wsum = 0.0;
    bool wbad = false;
    for (int c = 0; c < C; ++c) {
        const double wc = a.weights ? a.weights[(size_t)q * C + c] : 1.0;
        wbad |= !(wc >= 0.0) || isinf(wc);
        wsum += wc;
    }
    if (wbad || !(wsum > 0.0)) {
        if (tid == 0) atomicOr(a.err, kErrWeights);
        wsum = 1.0;
    }
    for (int base = V * tid; base < K; base += V * (int)blockDim.x) {
        double mix[V];
#pragma unroll
        for (int j = 0; j < V; ++j) mix[j] = 0.0;
#pragma unroll 8
        for (int c = 0; c < C; ++c) {
            const double pc = (a.weights ? a.weights[(size_t)q * C + c] : 1.0) / wsum;
            float t[V];
            const float* src = rows + (size_t)c * (size_t)K + base;
            if constexpr (VEC) {
                const float4 x = *reinterpret_cast<const float4*>(src);
                t[0] = x.x; t[1] = x.y; t[2] = x.z; t[3] = x.w;
            } else {
                t[0] = src[0];
            }
#pragma unroll
            for (int j = 0; j < V; ++j) mix[j] = fma(pc, 1.0 - (double)t[j], mix[j]);
        }
        double pm[V];
#pragma unroll
        for (int j = 0; j < V; ++j) {
            pm[j] = s > 1 ? pow(mix[j], (double)(s - 1)) : 1.0;
            s_bin[base + j + ((base + j) >> a.vshift)] = fma(-pm[j], mix[j], 1.0);
        }
        double* o = a.pm + (size_t)pair * (size_t)K + base;
        if constexpr (VEC) {
            *reinterpret_cast<double2*>(o) = make_double2(pm[0], pm[1]);
            *reinterpret_cast<double2*>(o + 2) = make_double2(pm[2], pm[3]);
        } else {
            o[0] = pm[0];
        }
    }
    // model-wide E[L] = w (1/2 + sum_k (1 - F_mix^s(x_{k+1}))), summed in the
    // order of laws_kernel's threads and waves: the same bits
    __syncthreads();
    for (int u = wv; u < kWaves; u += (int)blockDim.x / 64) {
        const int t = 64 * u + lane, first = t << a.vshift;
        const int n = min(1 << a.vshift, K - first);
        double el = 0.0;
        for (int j = 0; j < n; ++j) el += s_bin[first + t + j];
        for (int o = 32; o > 0; o >>= 1) el += __shfl_xor(el, o, 64);
        if (lane == 0) s_el[u] = el;
    }
    __syncthreads();
    if (tid == 0) {
        double tot = 0.0;
        for (int i = 0; i < kWaves; ++i) tot += s_el[i];
        a.model_el[pair] = (float)(w * (0.5 + tot));
    }
}

template <bool VEC>
hipError_t launch_laws_mix(const LawArgs& a, unsigned pairs, int threads, hipStream_t st) {
    const int lds = (int)sizeof(double) * (a.K + (a.K >> a.vshift) + 1);
    static std::atomic<int> allowed{60 * 1024};   // per template instance; device-independent
    if (lds > allowed.load(std::memory_order_relaxed)) {
        constexpr int most = (int)sizeof(double) * (ORLOJ_MAX_BINS + kThreads + 1);
        const hipError_t e = hipFuncSetAttribute((const void*)laws_mix_kernel<VEC>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, most);
        if (e != hipSuccess) return e;
        allowed.store(most, std::memory_order_relaxed);
    }
    hipLaunchKernelGGL(laws_mix_kernel<VEC>, dim3(pairs), dim3(threads), lds, st, a);
    return hipGetLastError();
}

template <int VPT>
__global__ __launch_bounds__(kThreads) void laws_row_kernel(const LawArgs a) {
    __shared__ float s_wave[kWaves];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int pair = (int)(blockIdx.x / (unsigned)a.C), c = (int)(blockIdx.x % (unsigned)a.C);
    const int K = a.K, base = tid * VPT;
    const size_t r = ((size_t)pair * (size_t)a.C + (size_t)c) * (size_t)K;
    double g[VPT], pm[VPT];
    load_cdf_chunk<VPT>(g, a.tab + r, base, K);
    const double* pmr = a.pm + (size_t)pair * (size_t)K;
#pragma unroll
    for (int j = 0; j < VPT; ++j) pm[j] = 1.0;             // padding bins: F = 1
    if (VPT % 2 == 0 && K % 2 == 0) {
#pragma unroll
        for (int j = 0; j + 1 < VPT; j += 2)
            if (base + j < K) {
                const double2 v = *reinterpret_cast<const double2*>(pmr + base + j);
                pm[j] = v.x;
                pm[j + 1] = v.y;
            }
    } else {
#pragma unroll
        for (int j = 0; j < VPT; ++j)
            if (base + j < K) pm[j] = pmr[base + j];
    }
    const double bw = a.b * a.width[pair / a.nbs];
    const double d = exp(-bw);
    // scan constants: a thread chunk spans VPT bins
    const float log2d = (float)(-bw * 1.4426950408889634);
    float rp[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) rp[i] = exp2_hw(log2d * (float)(VPT << i));
    const float w15 = exp2_hw(log2d * (float)(VPT * ((lane & 15) + 1)));
    const float w31 = exp2_hw(log2d * (float)(VPT * (lane >= 32 ? lane - 31 : 0)));
    const float d_wave = exp2_hw(log2d * (float)(64 * VPT));

    double z = 0.0;
#pragma unroll
    for (int j = 0; j < VPT; ++j) {
        g[j] *= pm[j];
        z = fma(z, d, g[j]);
    }
    // in-wave weighted scan of the chunk totals, then across the waves
    const float A = wave_wscan((float)z, rp, w15, w31);
    if (lane == 63) s_wave[wv] = A;
    __syncthreads();
    float carry = 0.0f;   // discounted sum of the earlier waves' bins, at the end of the last one
#pragma unroll
    for (int i = 0; i < kWaves; ++i)
        if (i < wv) carry = fmaf(carry, d_wave, s_wave[i]);
    // prefix up to the end of the previous thread chunk
    const float prev = __shfl_up(A, 1, 64);
    const float before = (lane > 0 ? prev : 0.0f) + carry * exp2_hw(log2d * (float)(VPT * lane));
    double zz = (double)before;
    float lv[VPT], dv[VPT];
#pragma unroll
    for (int j = 0; j < VPT; ++j) {
        zz = fma(zz, d, g[j]);
        lv[j] = (float)g[j];
        dv[j] = (float)zz;
    }
    store_chunk<VPT>(a.law + r, lv, base, K);
    store_chunk<VPT>(a.disc + r, dv, base, K);
}

template <int VPT>
hipError_t launch_laws_rows(const LawArgs& a, unsigned rows, hipStream_t st) {
    hipLaunchKernelGGL(laws_row_kernel<VPT>, dim3(rows), dim3(kThreads), 0, st, a);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// iterate_kernel: one workgroup per model, of TH threads (256, or 1024 when
// a queue is longer than 1024 requests).  Requests are strided over the
// threads (request i on thread i mod TH).  Long queues on few models split
// the iteration in two launches: the drop phase in parts of kDropPart
// requests, one workgroup each, writing per-part counts, then the rest per
// model from those counts.  For every batch size the drop
// phase keeps a request iff its deadline lies past the left edge of its
// class's first bin with mass at that batch size (then it could finish run
// alone).  Over 32 batch sizes the model's first-bin table sits in LDS and
// each wave walks its 64 requests with the batch sizes across its lanes (one
// integer compare per pair against the request's keep edge); otherwise each
// lane takes a request and the counts and the earliest kept request come
// from wave ballots.
// Thread 0 picks the candidate batch size ((D_{Q_s}, s) descending, first
// with |Q_s| >= s).  Requests kept at the candidate size get their
// priority from the model-law tables (Eq. (2) in the scan form:
// gamma e^{-b theta w} (G_k - (1-d) Z(k-2)) + h_k psi(theta), over the
// model-wide E[L]); PopBatch takes the s largest keys (kept flag, priority,
// earlier position) in rank order: for queues up to 512 requests each key's
// rank is counted against all keys in LDS; longer queues find the s-th
// largest key by a radix select (eight 8-bit digits, an LDS histogram and a
// block suffix scan per digit) and rank the selected keys.
// ---------------------------------------------------------------------------
struct IterArgs {
    const int32_t* sup;        // [M][nbs][C][2]
    const float* law;          // [M][nbs][C][K]
    const float* disc;         // [M][nbs][C][K]
    const float* model_el;     // [M][nbs]
    const int64_t* queue_off;
    const int32_t* cls;
    const double* deadline;
    const double* now;
    const double* width;
    const double* cost;        // [N] or NULL (1)
    const int64_t* step_off;   // [N+1] or NULL (one step at the deadline)
    const double* step_dl;     // [S]
    const double* step_cost;   // [S] cumulative costs
    int32_t* timed_out;        // [N]
    float* score;              // [N]
    int32_t* cand_bs;          // [M]
    int32_t* batch;            // [M][bs_max]
    int* err;
    int32_t* part_cnt;         // [M][parts][nbs] drop-phase counts of a split launch
    int32_t* part_first;       // [M][parts][nbs] and first kept positions
    int parts;
    double b;
    int M, C, K, nbs, bs_max;
    int bs[ORLOJ_MAX_BATCH_SIZES];
};

// What one iterate_kernel launch does: the whole iteration per model, or
// the iteration split in two launches for long queues on few models: the
// drop phase over parts of kDropPart requests (one workgroup each), then
// the rest per model from the parts' counts.
constexpr int kIterWhole = 0, kIterDropPart = 1, kIterFromParts = 2;
constexpr int kDropPart = 256;

constexpr int kIterMaxBatch = 1024;      // largest batch size PopBatch orders in LDS
constexpr int kIterMaxQueue = 4096;      // longest queue one workgroup ranks
constexpr int kIterWideQueue = 1024;     // longer queues get 1024-thread workgroups
constexpr int kIterStage = 8448;         // LDS words for a model's first-bin table

// The largest k in [0, K] with (double)k * w < tau, or -1 when there is
// none (tau <= 0 or NaN); w is finite and > 0.  Products k * w rise with k,
// so for any first bin lo in [0, K]: tau > lo * w iff lo <= keep_edge.
__device__ inline int keep_edge(double tau, double w, int K) {
    if (!(tau > 0.0)) return -1;
    const double t = tau / w;
    int k = t >= (double)K ? K : (int)t;
    while (k > 0 && (double)k * w >= tau) --k;
    while (k < K && (double)(k + 1) * w < tau) ++k;
    return k;
}

template <int TH, bool STAGE, int PH>
__global__ __launch_bounds__(TH) void iterate_kernel(const IterArgs a) {
    constexpr int kW = TH / 64;                    // waves
    __shared__ int s_cnt[ORLOJ_MAX_BATCH_SIZES];
    __shared__ int s_first[ORLOJ_MAX_BATCH_SIZES];
    __shared__ int s_cand;
    __shared__ double s_cd[kW];
    __shared__ int s_cb[kW];
    __shared__ unsigned s_hist[2][256];
    __shared__ int s_wcnt[kW][ORLOJ_MAX_BATCH_SIZES];
    __shared__ int s_wfirst[kW][ORLOJ_MAX_BATCH_SIZES];
    __shared__ unsigned s_wsum[4];
    __shared__ int s_digit, s_need;
    __shared__ __align__(16) unsigned long long s_sel[kIterMaxBatch];
    __shared__ int s_nsel;
    __shared__ int s_lo[STAGE ? kIterStage + 64 : 1];   // [C][nbs + 1] first bins, 64 words of tail
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = PH == kIterDropPart ? (int)blockIdx.x / a.parts : (int)blockIdx.x;
    const int64_t q0 = a.queue_off[q];
    const int N = (int)(a.queue_off[q + 1] - q0);
    // the requests whose drop phase this workgroup runs
    int ib = 0, ie = N;
    if constexpr (PH == kIterDropPart) {
        ib = ((int)blockIdx.x - q * a.parts) * kDropPart;
        ie = min(N, ib + kDropPart);
        if (ib >= ie) return;
    }
    const int nbs = a.nbs, C = a.C, K = a.K;
    const double w = a.width[q];
    const double nowq = a.now[q];
    const bool wok = w > 0.0 && w < HUGE_VAL;
    if (tid == 0) { s_cand = -1; s_nsel = 0; }
    if (tid < 256) {
        s_hist[0][tid] = 0u;
        s_hist[1][tid] = 0u;
    }
    const int32_t* sup_q = a.sup + (size_t)q * (size_t)nbs * (size_t)C * 2;
    // first bin with mass of class c at batch size index bi, in [0, K) in
    // a support that orloj_build_cdfs wrote (the LDS copy below is clamped
    // to [0, K], which changes nothing there)
    auto first_bin = [&](int bi, int c) { return sup_q[((size_t)bi * C + c) * 2]; };
    // STAGE (more than 32 batch sizes, and C (nbs + 1) <= kIterStage): the
    // model's table is staged in LDS class-major (rows of nbs + 1 words, so
    // the transposing writes spread over the banks) and the drop phase runs
    // across the batch sizes in the lanes.  Fewer batch sizes would leave
    // most lanes idle that way, so there each lane takes a request instead.
    const int ldo = nbs + 1;
    constexpr bool staged = STAGE;
    if constexpr (staged)
        for (int j = tid; j < nbs * C; j += TH) {
            const int bi = j / C, c = j - bi * C;
            s_lo[c * ldo + bi] = min(max(sup_q[2 * j], 0), K);
        }
    __syncthreads();

    // drop phase: per wave, the count of kept requests and the first kept
    // position of batch size index 64 r + l sit in lane l of cntv[r] and
    // firstv[r] (no atomics); the waves are combined afterwards
    constexpr int kBR = ORLOJ_MAX_BATCH_SIZES / 64;
    int cntv[kBR], firstv[kBR];
    unsigned long long vmask[kBR];   // lanes that hold a batch size, per row
    const int nrows = (nbs + 63) / 64;
#pragma unroll
    for (int r = 0; r < kBR; ++r) {
        cntv[r] = 0;
        firstv[r] = 0x7fffffff;
        vmask[r] = __ballot(64 * r + lane < nbs);
    }
    for (int i0 = ib; i0 < (PH == kIterFromParts ? ib : ie); i0 += TH) {
        const int i = i0 + tid;
        const bool live = i < ie;
        int c = 0;
        double tau = 0.0;
        if (live) {
            c = a.cls[q0 + i];
            const double D = a.deadline[q0 + i];
            // the drop phase looks at the last step of a step cost function
            const double Dlast = a.step_off ? a.step_dl[a.step_off[q0 + i + 1] - 1] : D;
            int flag = 0;
            if (c < 0 || c >= C) { flag |= kErrClassRange; c = 0; }
            if (isnan(D)) flag |= kErrDeadlineNaN;
            if (i > 0 && D < a.deadline[q0 + i - 1]) flag |= kErrUnsorted;
            if (i == 0 && isnan(nowq)) flag |= kErrNowNaN;
            if (i == 0 && !wok) flag |= kErrWidth;
            if (flag) atomicOr(a.err, flag);
            tau = Dlast - nowq;
        }
        if constexpr (staged) {
            // the wave's 64 requests one at a time, its lanes over the batch
            // sizes: request j is kept at batch size 64 r + l iff that
            // batch size's first bin of its class is <= its keep edge (no
            // first bin is below 0, so a request with edge -1, dead lanes
            // included, is kept nowhere).  Eight requests' rows are read
            // before any is compared.
            const int kk = live && wok ? keep_edge(tau, w, K) : -1;
            const int base = i0 + wv * 64;
            const int nj = __builtin_amdgcn_readfirstlane(min(64, ie - base));
            unsigned long long anyb = 0ull;   // bit j: request base + j kept somewhere
            auto sweep = [&](auto rows) {
                constexpr int NR = decltype(rows)::value;
                for (int j0 = 0; j0 < nj; j0 += 8) {
                    int kj[8], lo[8][NR];
#pragma unroll
                    for (int jj = 0; jj < 8; ++jj) {
                        kj[jj] = __builtin_amdgcn_readlane(kk, j0 + jj);
                        const int* row = s_lo + __builtin_amdgcn_readlane(c, j0 + jj) * ldo + lane;
#pragma unroll
                        for (int r = 0; r < NR; ++r) lo[jj][r] = row[64 * r];
                    }
#pragma unroll
                    for (int jj = 0; jj < 8; ++jj) {
                        const int ij = base + j0 + jj;
                        unsigned long long hit = 0ull;
#pragma unroll
                        for (int r = 0; r < NR; ++r) {
                            const bool keep = lo[jj][r] <= kj[jj];
                            hit |= __ballot(keep) & vmask[r];
                            cntv[r] += keep ? 1 : 0;
                            firstv[r] = min(firstv[r], keep ? ij : 0x7fffffff);
                        }
                        if (hit) anyb |= 1ull << (j0 + jj);
                    }
                }
            };
            switch (nrows) {
                case 1: sweep(std::integral_constant<int, 1>{}); break;
                case 2: sweep(std::integral_constant<int, 2>{}); break;
                case 3: sweep(std::integral_constant<int, 3>{}); break;
                default: sweep(std::integral_constant<int, 4>{}); break;
            }
            if (live) {
                a.timed_out[q0 + i] = (anyb >> lane) & 1ull ? 0 : 1;
                a.score[q0 + i] = 0.0f;
            }
            continue;
        }
        bool any = false;
        // the support's first bins of a group of batch sizes are loaded
        // together, so their latencies overlap
        constexpr int kGroup = 8;
#pragma unroll
        for (int r = 0; r < kBR; ++r) {
            const int bend = min(nbs, 64 * r + 64);
            for (int b0 = 64 * r; b0 < bend; b0 += kGroup) {
                int lo[kGroup];
#pragma unroll
                for (int j = 0; j < kGroup; ++j)
                    lo[j] = first_bin(min(b0 + j, nbs - 1), c);
#pragma unroll
                for (int j = 0; j < kGroup; ++j) {
                    const int bi = b0 + j;
                    if (bi >= bend) break;
                    const bool keep = live && wok && tau > (double)lo[j] * w;
                    any |= keep;
                    const unsigned long long m = __ballot(keep);
                    const bool me = lane == (bi & 63);
                    cntv[r] += me ? __popcll(m) : 0;
                    if (me && m != 0ull && firstv[r] == 0x7fffffff)
                        firstv[r] = i0 + wv * 64 + __ffsll((long long)m) - 1;
                }
            }
        }
        if (live) {
            a.timed_out[q0 + i] = any ? 0 : 1;
            a.score[q0 + i] = 0.0f;
        }
    }
    if constexpr (PH != kIterFromParts) {
#pragma unroll
        for (int r = 0; r < kBR; ++r) {
            s_wcnt[wv][64 * r + lane] = cntv[r];
            s_wfirst[wv][64 * r + lane] = firstv[r];
        }
        __syncthreads();
    }
    for (int bi = tid; bi < nbs; bi += TH) {
        int cnt = 0, first = 0x7fffffff;
        if constexpr (PH == kIterFromParts) {
            const size_t p0 = (size_t)q * a.parts * nbs + bi;
            for (int p = 0; p * kDropPart < N; ++p) {
                cnt += a.part_cnt[p0 + (size_t)p * nbs];
                first = min(first, a.part_first[p0 + (size_t)p * nbs]);
            }
        } else {
#pragma unroll
            for (int v = 0; v < kW; ++v) {
                cnt += s_wcnt[v][bi];
                first = min(first, s_wfirst[v][bi]);
            }
        }
        if constexpr (PH == kIterDropPart) {
            const size_t o = ((size_t)blockIdx.x) * nbs + bi;   // (q parts + part) nbs + bi
            a.part_cnt[o] = cnt;
            a.part_first[o] = first;
        } else {
            s_cnt[bi] = cnt;
            s_first[bi] = first;
        }
    }
    if constexpr (PH == kIterDropPart) return;
    __syncthreads();
    // Candidate batch size: among batch sizes whose kept set holds at least
    // s requests, the largest earliest-kept deadline D_{Q_s}, ties to the
    // larger batch size (batch sizes increase with their index).  Thread bi
    // proposes batch size bi; a wave reduction, then one over the waves.
    {
        double dc = 0.0;
        int cb = -1;
        for (int bi = tid; bi < nbs; bi += TH) {
            if (s_cnt[bi] < a.bs[bi]) continue;
            const double D = a.deadline[q0 + s_first[bi]];
            if (cb < 0 || D > dc || (D == dc && bi > cb)) { dc = D; cb = bi; }
        }
        auto take = [&](double d2, int b2) {
            if (b2 >= 0 && (cb < 0 || d2 > dc || (d2 == dc && b2 > cb))) { dc = d2; cb = b2; }
        };
        for (int o = 32; o > 0; o >>= 1) {
            const double d2 = __shfl_xor(dc, o, 64);
            const int b2 = __shfl_xor(cb, o, 64);
            take(d2, b2);
        }
        if (lane == 0) { s_cd[wv] = dc; s_cb[wv] = cb; }
        __syncthreads();
        if (tid == 0) {
            for (int i = 0; i < kW; ++i) take(s_cd[i], s_cb[i]);
            s_cand = cb;
            a.cand_bs[q] = cb >= 0 ? a.bs[cb] : 0;
        }
        __syncthreads();
    }
    const int cand = s_cand;
    int32_t* bq = a.batch + (size_t)q * (size_t)a.bs_max;
    if (cand < 0) {
        for (int j = tid; j < a.bs_max; j += TH) bq[j] = -1;
        return;
    }
    const int s = a.bs[cand];

    // priorities at the candidate size; keys = kept | priority bits | ~index
    const double bw = a.b * w;
    const double gamma = -expm1(-bw) / bw;
    const double omd = -expm1(-bw);
    const float el = a.model_el[(size_t)q * nbs + cand];
    const size_t lrow0 = ((size_t)q * nbs + cand) * (size_t)C;
    constexpr int kPer = kIterMaxQueue / TH;         // keys per thread, in registers
    unsigned long long key[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) key[j] = 0ull;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int i = j * TH + tid;
        if (i < N) {
            int c = a.cls[q0 + i];
            c = (c < 0 || c >= C) ? 0 : c;
            const double D = a.deadline[q0 + i];
            const double Dlast = a.step_off ? a.step_dl[a.step_off[q0 + i + 1] - 1] : D;
            const int lo = first_bin(cand, c);
            if (wok && Dlast - nowq > (double)lo * w) {
                const float* G = a.law + (lrow0 + c) * (size_t)K;
                const float* Z = a.disc + (lrow0 + c) * (size_t)K;
                // Eq. (2) x E[L] for one deadline, in the scan form
                auto num_at = [&](double tau) -> double {
                    if (!(tau > 0.0)) return 0.0;
                    const double u = tau / w;
                    if (u >= (double)K) {
                        const double cg = gamma * exp(-a.b * (tau - (double)K * w));
                        const double zk = K >= 2 ? (double)Z[K - 2] : 0.0;
                        return cg * (1.0 - omd * zk);
                    }
                    const int k = (int)floor(u);
                    const double th = u - (double)k;
                    const double gk = k >= 1 ? (double)G[k - 1] : 0.0;
                    const double gk1 = (double)G[k];
                    const double zk = k >= 2 ? (double)Z[k - 2] : 0.0;
                    const double cg = gamma * exp(-a.b * th * w);
                    const double psi = -expm1(-a.b * th * w) / bw;
                    return cg * (gk - omd * zk) + (gk1 - gk) * psi;
                };
                double cr = a.cost ? a.cost[q0 + i] : 1.0;
                int flag = 0;
                if (!(cr >= 0.0 && cr < HUGE_VAL)) { flag = kErrCost; cr = 0.0; }
                double num = 0.0;
                if (a.step_off) {
                    // App. B: one single step per cost increment
                    double below = 0.0, dprev = -HUGE_VAL;
                    for (int64_t st = a.step_off[q0 + i]; st < a.step_off[q0 + i + 1]; ++st) {
                        const double dj = a.step_dl[st], cj = a.step_cost[st];
                        if (!(cj >= below && cj < HUGE_VAL) || !(dj > dprev)) {
                            flag = kErrCost;
                            num = 0.0;
                            break;
                        }
                        num += (cj - below) * num_at(dj - nowq);
                        below = cj;
                        dprev = dj;
                    }
                } else {
                    num = num_at(D - nowq);
                }
                if (flag) atomicOr(a.err, flag);
                num *= cr;
                const float p = (float)(num / (double)el);
                a.score[q0 + i] = p;
                const float pp = p > 0.0f ? p : 0.0f;
                key[j] = (1ull << 63) | ((unsigned long long)__float_as_uint(pp) << 32) |
                         (unsigned long long)(0xffffffffu - (unsigned)i);
            }
        }
    }
    // Short queues: every kept key's rank is the number of larger keys
    // (keys are unique), counted over the keys staged in LDS; the s keys of
    // rank < s are the batch, in rank order.
    constexpr int kRankQueue = 512;
    constexpr int kRankSlots = (kRankQueue + TH - 1) / TH;
    static_assert(kRankQueue <= kIterMaxBatch && kRankSlots <= kPer, "s_sel holds the keys");
    if (N <= kRankQueue) {
        // staged up to a multiple of 8 with zero keys (never larger than a
        // kept key), read 16 bytes at a time
        const int N8 = (N + 7) & ~7;
#pragma unroll
        for (int j = 0; j < kRankSlots; ++j) {
            const int i = j * TH + tid;
            if (i < N8) s_sel[i] = i < N ? key[j] : 0ull;
        }
        __syncthreads();
        const ulonglong2* sel2 = reinterpret_cast<const ulonglong2*>(s_sel);
#pragma unroll
        for (int j = 0; j < kRankSlots; ++j) {
            const int i = j * TH + tid;
            if (i < N && key[j] != 0ull) {
                const unsigned long long kj = key[j];
                int rank = 0;
                for (int t = 0; t < N8 / 2; t += 4) {
                    ulonglong2 v[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) v[u] = sel2[t + u];
#pragma unroll
                    for (int u = 0; u < 4; ++u) rank += (v[u].x > kj) + (v[u].y > kj);
                }
                if (rank < s) bq[rank] = i;
            }
        }
        for (int j = s + tid; j < a.bs_max; j += TH) bq[j] = -1;
        return;
    }
    // Longer queues: the s-th largest key (at least s are non-zero, since
    // |Q_s| >= s) by a radix select, most significant digit first.  Pass by
    // pass, the keys that agree with the digits fixed so far are counted
    // per next digit; the digit is the largest whose suffix count reaches
    // the number of keys still needed, which then drops by the count of the
    // larger digits.
    unsigned long long prefix = 0ull, pmask = 0ull;
    int need = s;
    for (int shift = 56; shift >= 0; shift -= 8) {
        unsigned* hist = s_hist[(shift >> 3) & 1];    // two buffers: the other one is cleared here
        if (tid < 256) s_hist[((shift >> 3) & 1) ^ 1][tid] = 0u;
#pragma unroll
        for (int j = 0; j < kPer; ++j)
            if (key[j] != 0ull && (key[j] & pmask) == prefix)
                atomicAdd(&hist[(unsigned)(key[j] >> shift) & 255u], 1u);
        __syncthreads();
        // suffix sums over the digits: thread t < 256 holds digit 255 - t,
        // so an inclusive prefix scan over t counts the keys with digit
        // >= 255 - t (the first four waves, whole)
        const bool hw = tid < 256;
        unsigned mine = 0u, incl = 0u;
        if (hw) {
            mine = hist[255 - tid];
            incl = mine;
            for (int o = 1; o < 64; o <<= 1) {
                const unsigned up = __shfl_up(incl, o, 64);
                if (lane >= o) incl += up;
            }
            if (lane == 63) s_wsum[wv] = incl;
        }
        __syncthreads();
        if (hw) {
            for (int i = 0; i < wv; ++i) incl += s_wsum[i];
            const unsigned excl = incl - mine;
            // exactly one thread sees the crossing: keys with larger digits
            // are fewer than `need`, with this digit included they are enough
            if (excl < (unsigned)need && incl >= (unsigned)need) {
                s_digit = 255 - tid;
                s_need = need - (int)excl;
            }
        }
        __syncthreads();
        prefix |= (unsigned long long)s_digit << shift;
        pmask |= 255ull << shift;
        need = s_need;
    }
    const unsigned long long lo_k = prefix;
    // the selected keys, then each one's rank among them
#pragma unroll
    for (int j = 0; j < kPer; ++j)
        if (key[j] >= lo_k && key[j] != 0ull) {
            const int slot = atomicAdd(&s_nsel, 1);
            if (slot < kIterMaxBatch) s_sel[slot] = key[j];
        }
    __syncthreads();
    const int nsel = min(s_nsel, min(s, kIterMaxBatch));
    for (int j = tid; j < nsel; j += TH) {
        const unsigned long long kj = s_sel[j];
        int rank = 0;
        for (int i = 0; i < nsel; ++i) rank += s_sel[i] > kj;
        bq[rank] = (int32_t)(0xffffffffu - (unsigned)(kj & 0xffffffffull));
    }
    for (int j = nsel + tid; j < a.bs_max; j += TH) bq[j] = -1;
}

// ---------------------------------------------------------------------------
// accumulate_kernel: profiler feedback.  One thread per sample (grid-stride):
// validate, bin by floor(latency / w) with the last bin catching the tail,
// and add one count with a device-scope atomic.
// ---------------------------------------------------------------------------
struct AccArgs {
    const int32_t* model;
    const int32_t* bs_index;
    const int32_t* cls;
    const double* latency;
    const double* width;
    uint32_t* counts;
    unsigned long long* n_rejected;
    int64_t n;
    int M, nbs, C, K;
};

__global__ __launch_bounds__(kThreads) void accumulate_kernel(const AccArgs a) {
    unsigned long long rejected = 0;
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < a.n;
         i += (int64_t)gridDim.x * kThreads) {
        const int q = a.model[i], b = a.bs_index[i], c = a.cls[i];
        const double lat = a.latency[i];
        if (q < 0 || q >= a.M || b < 0 || b >= a.nbs || c < 0 || c >= a.C ||
            !(lat >= 0.0 && lat < HUGE_VAL)) {
            ++rejected;
            continue;
        }
        const double w = a.width[q];
        if (!(w > 0.0)) {
            ++rejected;
            continue;
        }
        const double u = floor(lat / w);
        const int k = u >= (double)(a.K - 1) ? a.K - 1 : (int)u;
        atomicAdd(a.counts + (((size_t)q * a.nbs + b) * a.C + c) * (size_t)a.K + k, 1u);
    }
    if (a.n_rejected && rejected) atomicAdd(a.n_rejected, rejected);
}

}  // namespace

namespace {


int hip_fail(orloj_ctx* ctx, hipError_t e, const char* what) {
    return orloj_ctx_fail(ctx, ORLOJ_E_HIP, "%s: %s", what, hipGetErrorString(e));
}

int check_grid(orloj_ctx* ctx, const orloj_grid* g) {
    if (!g) return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "grid is NULL");
    if (g->n_models < 0) return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "n_models < 0");
    if (g->n_classes < 1) return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "n_classes < 1");
    if (g->n_bins < 1) return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "n_bins < 1");
    if (g->n_bins > ORLOJ_MAX_BINS)
        return orloj_ctx_fail(ctx, ORLOJ_E_UNSUPPORTED, "n_bins %d > %d", g->n_bins, ORLOJ_MAX_BINS);
    if (g->n_bs < 1) return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "n_bs < 1");
    if (g->n_bs > ORLOJ_MAX_BATCH_SIZES)
        return orloj_ctx_fail(ctx, ORLOJ_E_UNSUPPORTED, "n_bs %d > %d", g->n_bs, ORLOJ_MAX_BATCH_SIZES);
    if (!g->batch_sizes) return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "batch_sizes is NULL");
    for (int i = 0; i < g->n_bs; ++i) {
        if (g->batch_sizes[i] < 1) return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "batch size < 1");
        if (i > 0 && g->batch_sizes[i] <= g->batch_sizes[i - 1])
            return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "batch sizes not strictly increasing");
    }
    if (g->n_models > 0 && !g->d_bin_width_ms)
        return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "d_bin_width_ms is NULL");
    return ORLOJ_OK;
}

int check_queues(orloj_ctx* ctx, const orloj_grid* g, const orloj_queues* qs) {
    if (!qs) return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "queues is NULL");
    if (!qs->h_queue_off) return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "h_queue_off is NULL");
    if (qs->h_queue_off[0] != 0) return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "h_queue_off[0] != 0");
    for (int q = 0; q < g->n_models; ++q)
        if (qs->h_queue_off[q + 1] < qs->h_queue_off[q])
            return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "h_queue_off decreases at model %d", q);
    if (g->n_models > 0) {
        if (!qs->d_queue_off || !qs->d_now_ms)
            return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "d_queue_off / d_now_ms is NULL");
        if (qs->h_queue_off[g->n_models] > 0 && (!qs->d_class || !qs->d_deadline_ms))
            return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "d_class / d_deadline_ms is NULL");
    }
    return ORLOJ_OK;
}

int64_t ncap_of(int64_t N, int bsz, int rect) { return rect ? N : (N < bsz ? N : (int64_t)bsz); }

int chunk_per_lane(int K) {
    int c = 1;
    while (c * kThreads < K) c <<= 1;
    return c;
}

// Whether the laws are formed by laws_mix_kernel and laws_row_kernel: pairs up
// to the compute units, as many bins in all as keep the powers' way through
// memory short, and classes enough to pay for a second launch.  Time against
// laws_kernel's, on 256 compute units:
//   16 classes, 256 bins: 64 pairs 0.77, 256 0.94; 1024 bins: 256 0.97; 2048
//     bins: 128 0.83, 192 1.02; 4096 bins: 64 0.80, 128 1.14
//   8 classes: 256 bins 1.02 to 1.12; 512 bins: 64 0.97, 256 1.02; 1024 bins:
//     128 0.93, 256 1.08; 2048 bins: 64 0.83, 128 0.98; 4096 bins: 16 0.71,
//     64 0.94
int64_t law_split_bins(const orloj_ctx* ctx) { return 1024 * (int64_t)(ctx->n_cu > 0 ? ctx->n_cu : 256); }

bool law_split(const orloj_ctx* ctx, int64_t pairs, int C, int K) {
    const int64_t most = law_split_bins(ctx);
    return C >= (K >= 512 ? 8 : 16) && 1024 * pairs <= most && pairs * K <= (C >= 16 ? most : most / 2);
}


template <int CPL, bool EXACT, int CR, bool AFF>
hipError_t launch_score_v(const ScoreArgs& a, unsigned grid, hipStream_t st) {
    constexpr int PF = ORLOJ_SCORE_PREFETCH;
    const size_t sm = score_fixed_bytes<CPL>() + (size_t)a.maxcap * score_bytes_per_member();
    static size_t attr_bytes = 0;   // per template instance; device-independent
    if (sm > attr_bytes) {
        hipError_t e = hipFuncSetAttribute((const void*)score_kernel<CPL, PF, EXACT, CR, AFF>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)sm);
        if (e != hipSuccess) return e;
        attr_bytes = sm;
    }
    hipLaunchKernelGGL((score_kernel<CPL, PF, EXACT, CR, AFF>), dim3(grid), dim3(64), sm, st, a);
    return hipGetLastError();
}

// Bins per lane chunk: panels of 64 chunks of CPL bins, at most kMaxChunk
// bins per lane (larger rows take more panels).  Wider panels spread each
// step's cross-lane reductions over more bins; narrower ones need fewer
// registers (more waves per SIMD) and re-read a repeated class's row slice
// sooner, while it may still sit in L2.  16 bins per lane (144 VGPRs, three
// waves per SIMD) balances the two on gfx950.
constexpr int kMaxChunk = 16;

int score_chunk_of(int K) {
    int c = 1;
    while (c < kMaxChunk && 64 * c < K) c <<= 1;
    return c;
}
// The affine mode's score waves read only the bins up to their members'
// deadlines (E[L_B] comes from emax_kernel), which at large batch sizes
// are a few hundred: narrower panels there mean less work per step and
// fewer registers.
#ifndef ORLOJ_AFFINE_CHUNK
#define ORLOJ_AFFINE_CHUNK 4
#endif
constexpr int kAffineChunk = ORLOJ_AFFINE_CHUNK;

int affine_chunk(int K) {
    int c = std::min(score_chunk_of(K), kAffineChunk);
    while ((K + 64 * c - 1) / (64 * c) > kMaxPanels) c <<= 1;   // a lane per panel's first member
    return c;
}

int score_chunk(int K) { return score_chunk_of(K); }

// Step carries: one register per 64 steps (longest prefix up to 64, or up to
// the compiled limit).
template <int CPL, bool EXACT, bool AFF>
hipError_t launch_score_c(const ScoreArgs& a, unsigned grid, hipStream_t st) {
    constexpr int CRL = (ORLOJ_MAX_PREFIX + 63) / 64;
    return a.maxcap <= 64 ? launch_score_v<CPL, EXACT, 1, AFF>(a, grid, st)
                          : launch_score_v<CPL, EXACT, CRL, AFF>(a, grid, st);
}

template <int CPL, bool AFF>
hipError_t launch_score_m(const ScoreArgs& a, unsigned grid, hipStream_t st) {
    return a.K % (64 * CPL) == 0 ? launch_score_c<CPL, true, AFF>(a, grid, st)
                                 : launch_score_c<CPL, false, AFF>(a, grid, st);
}

template <int CPL>
hipError_t launch_score(const ScoreArgs& a, unsigned grid, hipStream_t st) {
    return a.c1 ? launch_score_m<CPL, true>(a, grid, st) : launch_score_m<CPL, false>(a, grid, st);
}

// emax_kernel: one wave per (model, panel).
template <int CPL>
hipError_t launch_emax(const ScoreArgs& a, hipStream_t st) {
    const unsigned g = (unsigned)a.Mg * (unsigned)a.np_e;
    const bool exact = a.K % (64 * CPL) == 0;
    constexpr int CRL = (ORLOJ_MAX_PREFIX + 63) / 64;
    if (a.maxcap <= 64) {
        if (exact) hipLaunchKernelGGL((emax_kernel<CPL, true, 1>), dim3(g), dim3(64), 0, st, a);
        else hipLaunchKernelGGL((emax_kernel<CPL, false, 1>), dim3(g), dim3(64), 0, st, a);
    } else {
        if (exact) hipLaunchKernelGGL((emax_kernel<CPL, true, CRL>), dim3(g), dim3(64), 0, st, a);
        else hipLaunchKernelGGL((emax_kernel<CPL, false, CRL>), dim3(g), dim3(64), 0, st, a);
    }
    return hipGetLastError();
}

template <int R, bool AFF, int W>
hipError_t launch_turned_w(const TurnedArgs& a, hipStream_t st) {
    if constexpr (AFF) {
        const unsigned g = (unsigned)a.Mg * (unsigned)a.np_e * (unsigned)a.nblk;
        hipLaunchKernelGGL((turned_esum_kernel<R>), dim3(g), dim3(128), turned_lds(R, 2).total, st, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    constexpr int lds = turned_lds(R, W).total;
    static std::atomic<int> allowed{64 * 1024};   // per template instance; device-independent
    if (lds > allowed.load(std::memory_order_relaxed)) {
        const hipError_t e = hipFuncSetAttribute((const void*)turned_kernel<R, AFF, W>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
        allowed.store(lds, std::memory_order_relaxed);
    }
    const unsigned g = (unsigned)a.Mg * (unsigned)a.nbs * (unsigned)a.nblk;
    hipLaunchKernelGGL((turned_kernel<R, AFF, W>), dim3(g), dim3(64 * W), lds, st, a);
    return hipGetLastError();
}

template <int R>
hipError_t launch_turned_r(const TurnedArgs& a, int waves, hipStream_t st) {
    if (waves == 8) return a.c1 ? launch_turned_w<R, true, 8>(a, st) : launch_turned_w<R, false, 8>(a, st);
    return a.c1 ? launch_turned_w<R, true, 4>(a, st) : launch_turned_w<R, false, 4>(a, st);
}

// `waves`: 8 or 4 per workgroup.
hipError_t launch_turned(const TurnedArgs& a, int waves, hipStream_t st) {
    static_assert(ORLOJ_MAX_PREFIX <= 256, "four registers of members");
    if (a.maxcap <= 64) return launch_turned_r<1>(a, waves, st);
    return a.maxcap <= 128 ? launch_turned_r<2>(a, waves, st) : launch_turned_r<4>(a, waves, st);
}

template <int VPT>
hipError_t launch_cdf(const uint32_t* c, float* o, int32_t* sup, int64_t rows, int K, int* err,
                      hipStream_t st) {
    const int64_t cap = 1 << 20;
    const unsigned grid = (unsigned)(rows < cap ? rows : cap);
    hipLaunchKernelGGL(cdf_kernel<VPT>, dim3(grid), dim3(kThreads), 0, st, c, o, sup, rows, K, err);
    return hipGetLastError();
}

}  // namespace

// Scratch of orloj_score_candidates_affine_noalloc: the per-(model, panel,
// prefix length) sums of 1 - G that emax_kernel writes and score_kernel
// reads, in a fixed device array instead of the context's grown block.  Each
// device the library runs on holds its own copy until the process ends.  In
// host code `scratch` names a host-side stand-in: kernels are given the
// device address that hipGetSymbolAddress returns for the current device.
constexpr size_t kNoAllocScratchFloats = ORLOJ_NOALLOC_SCRATCH_FLOATS;
static __device__ __align__(256) float scratch[kNoAllocScratchFloats];

namespace {

constexpr int kMaxScratchDevices = 64;
std::mutex g_scratch_mu;
bool g_scratch_done[kMaxScratchDevices];
hipError_t g_scratch_err[kMaxScratchDevices];
float* g_scratch_ptr[kMaxScratchDevices];

// Device address of `scratch` on `device`, looked up once per device with
// that device current (the caller has made it current).
float* scratch_address(int device, hipError_t* err) {
    if (device < 0 || device >= kMaxScratchDevices) {
        *err = hipErrorInvalidDevice;
        return nullptr;
    }
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_done[device]) {
        void* ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        g_scratch_err[device] = e;
        g_scratch_ptr[device] = e == hipSuccess ? static_cast<float*>(ptr) : nullptr;
        g_scratch_done[device] = true;
    }
    *err = g_scratch_err[device];
    return g_scratch_ptr[device];
}

}  // namespace

extern "C" {

int orloj_create(orloj_ctx** out, int32_t hip_device, void* hip_stream) {
    if (!out) return ORLOJ_E_INVALID;
    *out = nullptr;
    orloj_ctx* ctx = new (std::nothrow) orloj_ctx;
    if (!ctx) return ORLOJ_E_NOMEM;
    ctx->device = hip_device;
    ctx->stream = (hipStream_t)hip_stream;
    ctx->d_err = nullptr;
    ctx->d_fill = nullptr;
    ctx->work = ctx->drop = ctx->mix = orloj_block{nullptr, 0};
    ctx->noalloc_scratch = nullptr;
    ctx->noalloc_err = hipSuccess;
    ctx->msg[0] = 0;
    int n = 0;
    if (hipGetDeviceCount(&n) != hipSuccess || hip_device < 0 || hip_device >= n) {
        delete ctx;
        return ORLOJ_E_INVALID;
    }
    float fill[kFillFloats];
    for (int i = 0; i < kFillFloats; ++i) fill[i] = i < kFillFloats / 2 ? 0.0f : 1.0f;
    hipError_t e = hipSetDevice(hip_device);
    ctx->n_cu = 0;
    if (e == hipSuccess) e = hipDeviceGetAttribute(&ctx->n_cu, hipDeviceAttributeMultiprocessorCount, hip_device);
    if (e == hipSuccess) e = hipMalloc((void**)&ctx->d_err, sizeof(int));
    if (e == hipSuccess) e = hipMemset(ctx->d_err, 0, sizeof(int));
    if (e == hipSuccess) e = hipMalloc((void**)&ctx->d_fill, sizeof fill);
    if (e == hipSuccess) e = hipMemcpy(ctx->d_fill, fill, sizeof fill, hipMemcpyHostToDevice);
    // the allocation-free scorer's scratch on this device (its failure only
    // disables that entry point)
    if (e == hipSuccess) ctx->noalloc_scratch = scratch_address(hip_device, &ctx->noalloc_err);
    if (e != hipSuccess) {
        if (ctx->d_err) (void)hipFree(ctx->d_err);
        if (ctx->d_fill) (void)hipFree(ctx->d_fill);
        delete ctx;
        return e == hipErrorOutOfMemory ? ORLOJ_E_NOMEM : ORLOJ_E_HIP;
    }
    *out = ctx;
    return ORLOJ_OK;
}

void orloj_destroy(orloj_ctx* ctx) {
    if (!ctx) return;
    (void)hipSetDevice(ctx->device);
    (void)hipStreamSynchronize(ctx->stream);
    if (ctx->d_err) (void)hipFree(ctx->d_err);
    if (ctx->d_fill) (void)hipFree(ctx->d_fill);
    for (const orloj_block& b : {ctx->work, ctx->drop, ctx->mix})
        if (b.p) (void)hipFree(b.p);
    delete ctx;
}

int orloj_set_score_chunk(orloj_ctx* ctx, int32_t steps) {
    if (!ctx) return ORLOJ_E_INVALID;
    if (steps < -1) return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "score chunk %d < -1", steps);
    return ORLOJ_OK;
}

int orloj_set_stream(orloj_ctx* ctx, void* hip_stream) {
    if (!ctx) return ORLOJ_E_INVALID;
    if ((hipStream_t)hip_stream != ctx->stream && (ctx->work.p || ctx->drop.p || ctx->mix.p)) {
        // calls still queued on the old stream may use the scratch
        hipError_t e = hipSetDevice(ctx->device);
        if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
        if (e != hipSuccess) return hip_fail(ctx, e, "hipStreamSynchronize");
    }
    ctx->stream = (hipStream_t)hip_stream;
    return ORLOJ_OK;
}

const char* orloj_last_error(const orloj_ctx* ctx) { return ctx ? ctx->msg : "context is NULL"; }

int orloj_sync(orloj_ctx* ctx) {
    if (!ctx) return ORLOJ_E_INVALID;
    hipError_t e = hipSetDevice(ctx->device);
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    if (e != hipSuccess) return hip_fail(ctx, e, "hipStreamSynchronize");
    int flags = 0;
    e = hipMemcpy(&flags, ctx->d_err, sizeof(int), hipMemcpyDeviceToHost);
    if (e != hipSuccess) return hip_fail(ctx, e, "reading the device status word");
    if (flags) {
        e = hipMemset(ctx->d_err, 0, sizeof(int));
        if (e != hipSuccess) return hip_fail(ctx, e, "clearing the device status word");
        return orloj_ctx_fail(ctx, ORLOJ_E_DATA, "device data error:%s%s%s%s%s%s%s%s%s",
                    (flags & kErrEmptyHistogram) ? " histogram-with-no-samples" : "",
                    (flags & kErrClassRange) ? " class-id-out-of-range" : "",
                    (flags & kErrDeadlineNaN) ? " NaN-deadline" : "",
                    (flags & kErrUnsorted) ? " deadlines-not-sorted" : "",
                    (flags & kErrNowNaN) ? " NaN-now" : "",
                    (flags & kErrWidth) ? " bin-width-not-positive" : "",
                    (flags & kErrWeights) ? " class-weights-invalid" : "",
                    (flags & kErrCost) ? " cost-or-steps-invalid" : "",
                    (flags & kErrAffine) ? " affine-constants-invalid" : "");
    }
    return ORLOJ_OK;
}

int orloj_build_cdfs(orloj_ctx* ctx, int64_t n_rows, int32_t n_bins, const uint32_t* d_counts,
                     float* d_ccdf, int32_t* d_support) {
    if (!ctx) return ORLOJ_E_INVALID;
    if (n_rows < 0) return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "n_rows < 0");
    if (n_bins < 1) return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "n_bins < 1");
    if (n_bins > ORLOJ_MAX_BINS)
        return orloj_ctx_fail(ctx, ORLOJ_E_UNSUPPORTED, "n_bins %d > %d", n_bins, ORLOJ_MAX_BINS);
    if (n_rows == 0) return ORLOJ_OK;
    if (!d_counts || !d_ccdf) return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "NULL buffer");
    const char* cb = (const char*)d_counts;
    const char* ob = (const char*)d_ccdf;
    const size_t bytes = (size_t)n_rows * (size_t)n_bins * 4;
    if (cb < ob + bytes && ob < cb + bytes)
        return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "d_counts and d_ccdf overlap");
    if (d_support) {
        const char* sb = (const char*)d_support;
        const size_t sbytes = (size_t)n_rows * 8;
        if ((sb < ob + bytes && ob < sb + sbytes) || (sb < cb + bytes && cb < sb + sbytes))
            return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "d_support overlaps d_counts or d_ccdf");
    }
    hipError_t e = hipSetDevice(ctx->device);
    if (e != hipSuccess) return hip_fail(ctx, e, "hipSetDevice");
    const int vpt = chunk_per_lane(n_bins);
    switch (vpt) {
        case 1: e = launch_cdf<1>(d_counts, d_ccdf, d_support, n_rows, n_bins, ctx->d_err, ctx->stream); break;
        case 2: e = launch_cdf<2>(d_counts, d_ccdf, d_support, n_rows, n_bins, ctx->d_err, ctx->stream); break;
        case 4: e = launch_cdf<4>(d_counts, d_ccdf, d_support, n_rows, n_bins, ctx->d_err, ctx->stream); break;
        case 8: e = launch_cdf<8>(d_counts, d_ccdf, d_support, n_rows, n_bins, ctx->d_err, ctx->stream); break;
        case 16: e = launch_cdf<16>(d_counts, d_ccdf, d_support, n_rows, n_bins, ctx->d_err, ctx->stream); break;
        default: e = launch_cdf<32>(d_counts, d_ccdf, d_support, n_rows, n_bins, ctx->d_err, ctx->stream); break;
    }
    if (e != hipSuccess) return hip_fail(ctx, e, "cdf_kernel launch");
    return ORLOJ_OK;
}

int orloj_output_sizes(const orloj_grid* grid, const orloj_queues* queues, int32_t prefix_mode,
                       int64_t* n_cands, int64_t* n_probs, int64_t* h_cand_off,
                       int64_t* h_prob_off) {
    if (prefix_mode != ORLOJ_PREFIX_TRIANGLE && prefix_mode != ORLOJ_PREFIX_RECT)
        return ORLOJ_E_INVALID;
    int rc = check_grid(nullptr, grid);
    if (rc) return rc;
    if (!queues || !queues->h_queue_off || queues->h_queue_off[0] != 0) return ORLOJ_E_INVALID;
    int64_t nc = 0, np = 0;
    if (h_cand_off) h_cand_off[0] = 0;
    if (h_prob_off) h_prob_off[0] = 0;
    for (int q = 0; q < grid->n_models; ++q) {
        const int64_t N = queues->h_queue_off[q + 1] - queues->h_queue_off[q];
        if (N < 0) return ORLOJ_E_INVALID;
        for (int bi = 0; bi < grid->n_bs; ++bi) {
            const int64_t c = ncap_of(N, grid->batch_sizes[bi], prefix_mode);
            nc += c;
            np += c * (c + 1) / 2;
        }
        if (h_cand_off) h_cand_off[q + 1] = nc;
        if (h_prob_off) h_prob_off[q + 1] = np;
    }
    if (n_cands) *n_cands = nc;
    if (n_probs) *n_probs = np;
    return ORLOJ_OK;
}

}  // extern "C"

namespace {

// A scratch block of the context, grown to at least `bytes`.  Work already
// enqueued on the context's stream may still use the old block, so the stream
// is drained before it is freed.
int ensure_block(orloj_ctx* ctx, orloj_block* blk, size_t bytes) {
    if (bytes <= blk->bytes) return ORLOJ_OK;
    hipError_t e = hipStreamSynchronize(ctx->stream);
    if (e != hipSuccess) return hip_fail(ctx, e, "hipStreamSynchronize");
    if (blk->p) {
        e = hipFree(blk->p);
        blk->p = nullptr;
        blk->bytes = 0;
        if (e != hipSuccess) return hip_fail(ctx, e, "hipFree");
    }
    e = hipMalloc(&blk->p, bytes);
    if (e != hipSuccess) {
        blk->p = nullptr;
        if (e != hipErrorOutOfMemory) return hip_fail(ctx, e, "hipMalloc");
        (void)hipGetLastError();
        return orloj_ctx_fail(ctx, ORLOJ_E_NOMEM, "scratch of %zu bytes", bytes);
    }
    blk->bytes = bytes;
    return ORLOJ_OK;
}

// The laws' scratch, allocated at its first use; false: no memory for it.
// The thread's capture mode is relaxed meanwhile: other threads may be
// capturing streams of their own, which an allocation would end otherwise.
bool have_mix(orloj_ctx* ctx) {
    if (ctx->mix.p) return true;
    const size_t bytes = (size_t)law_split_bins(ctx) * sizeof(double);
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    if (hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    const hipError_t e = hipMalloc(&ctx->mix.p, bytes);
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    if (e == hipSuccess) {
        ctx->mix.bytes = bytes;
        return true;
    }
    ctx->mix.p = nullptr;
    (void)hipGetLastError();
    return false;
}

// Whether the context's stream is being captured (or cannot say).
bool capturing(orloj_ctx* ctx) {
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(ctx->stream, &cs) != hipSuccess) {
        (void)hipGetLastError();
        return true;
    }
    return cs != hipStreamCaptureStatusNone;
}

// Validation and launch shared by the tabulated and the affine scorer
// (d_c0 / d_c1 NULL: tabulated).
// fixed_psum (affine mode only): a caller-fixed block of fixed_floats
// floats for the panel sums instead of the context's grown one (no
// allocation; ORLOJ_E_UNSUPPORTED when the call needs more).
int score_common(orloj_ctx* ctx, const orloj_grid* grid, const float* d_ccdf,
                 const int32_t* d_support, const double* d_c0, const double* d_c1,
                 const orloj_queues* queues, double b_expo_per_ms, int32_t prefix_mode,
                 const int64_t* d_cand_off, const int64_t* d_prob_off, float* d_finish_prob,
                 double* d_expected_finish, float* d_expected_latency_ms, float* d_score,
                 float* fixed_psum = nullptr, size_t fixed_floats = 0) {
    if (!ctx) return ORLOJ_E_INVALID;
    int rc = check_grid(ctx, grid);
    if (rc) return rc;
    rc = check_queues(ctx, grid, queues);
    if (rc) return rc;
    if (prefix_mode != ORLOJ_PREFIX_TRIANGLE && prefix_mode != ORLOJ_PREFIX_RECT)
        return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "prefix_mode %d", prefix_mode);
    if (!(b_expo_per_ms > 0.0) || !isfinite(b_expo_per_ms))
        return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "b_expo_per_ms must be finite and > 0");
    const int M = grid->n_models;
    if (M == 0) return ORLOJ_OK;
    int64_t maxcap = 0, total = 0, groups = 0;             // groups: workgroups of turned_kernel
    int n_act = 0;
    int act[kMaxActive];
    for (int q = 0; q < M; ++q) {
        const int64_t N = queues->h_queue_off[q + 1] - queues->h_queue_off[q];
        if (N <= 0) continue;
        if (n_act < kMaxActive) act[n_act] = q;
        ++n_act;
        for (int bi = 0; bi < grid->n_bs; ++bi) {
            const int64_t c = ncap_of(N, grid->batch_sizes[bi], prefix_mode);
            if (c > maxcap) maxcap = c;
            total += c;
            groups += (c + 63) / 64;
        }
    }
    if (maxcap > ORLOJ_MAX_PREFIX)
        return orloj_ctx_fail(ctx, ORLOJ_E_UNSUPPORTED, "prefix of %lld members > %d",
                    (long long)maxcap, ORLOJ_MAX_PREFIX);
    if (total == 0) return ORLOJ_OK;
    if (!d_ccdf || !d_cand_off || !d_prob_off || !d_finish_prob || !d_expected_finish ||
        !d_expected_latency_ms || !d_score)
        return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "NULL device buffer");
    // bins per lane of the score kernel (the affine mode reads only its
    // members' bins, in narrower panels)
    const int cpl = d_c1 ? affine_chunk(grid->n_bins) : score_chunk(grid->n_bins);
    const int panels = (grid->n_bins + 64 * cpl - 1) / (64 * cpl);
    // only the models with a queue get workgroups, when they are few enough
    // to list
    const bool compact = n_act < M && n_act <= kMaxActive;
    const int Mg = compact ? n_act : M;
    const int64_t nblk = (int64_t)Mg * grid->n_bs;
    if (nblk > 0x7fffffff) return orloj_ctx_fail(ctx, ORLOJ_E_UNSUPPORTED, "too many (model, batch size) pairs");

    // Launches too small to fill the chip go to turned_kernel (its row offsets
    // are 32-bit).  Its time grows with its workgroups, two of which run on a
    // compute unit at once.  score_kernel's is a chain of as many steps as the
    // longest prefix has members, in rows of several panels some of them for
    // each, and grows little until the chip is full.  So the line lies at a
    // number of workgroups proportional to the longest prefix.  Score +
    // selection, us, score_kernel / turned_kernel, deadlines over most of the
    // grid (the less favourable case: members in more of the bins):
    //   256 bins: prefixes to 24, 640 workgroups 24.8 / 24.1, 768 25.2 / 25.5;
    //     to 32, 1024 29.9 / 28.5, 1280 30.1 / 33.3; to 64, 2048 46.6 / 47.1
    //   1024 bins: to 24, 640 29.4 / 29.7, 768 30.6 / 34.2; to 48, 1280 49.9 /
    //     50.4; to 63, 1536 60.5 / 54.5, 2048 63.0 / 71.7; to 64, 1280 60.2 /
    //     49.8, 1536 61.5 / 54.8; to 65, 1536 93.1 / 96.7
    //   2048 bins: to 16, 768 38.1 / 37.7; to 48, 1536 86 / 76, 2048 88 / 100
    //   4096 bins: to 8, 640 38.1 / 40.7; to 48, 2048 152 / 148
    // One round of workgroups takes about as long whatever their number: there
    // it is the faster one from about ten members on (1024 bins, 512
    // workgroups: to 8 17.4 / 19.2, to 12 20.4 / 19.9, to 16 23.4 / 20.4; 384:
    // the same within 5%).  Affine mode: score_kernel waits for a launch of
    // emax_kernel's, so the line lies higher: 1024 bins, prefixes to 8, 512
    // workgroups 39 / 23, 768 40 / 29 (24.0 / 25.0 with short deadlines); to
    // 64, 2048 54.1 / 56.3.
    const int64_t n_cu = ctx->n_cu > 0 ? ctx->n_cu : 256;
    const int64_t one_round = groups <= 2 * n_cu ? std::min(groups, 5 * n_cu / 4) : groups;
    const int64_t launched = nblk * ((maxcap + 63) / 64);   // with those that find nothing to do
    const int64_t np_t = (grid->n_bins + kPanel - 1) / kPanel;
    const bool turned = (d_c1 ? groups <= 2 * n_cu + 24 * maxcap
                              : one_round <= (20 + 11 * panels) * maxcap) &&
                        launched <= 4 * groups + n_cu &&
                        (int64_t)grid->n_classes * grid->n_bins <= 0x3fffffff &&
                        (!d_c1 || (int64_t)M * np_t * maxcap <= kTurnedSums);
    // Affine mode: the sums of 1 - G, [M][panels][maxcap], floats of
    // emax_kernel or doubles of turned_esum_kernel.  The block is sized for
    // either, from the number of sums alone, so that whichever queues were
    // filled in an earlier call of a grid, a later one finds its block there
    // (a stream under capture cannot grow it).
    float* psum = fixed_psum;
    if (d_c1) {
        if ((int64_t)M * panels > 0x7fffffff)
            return orloj_ctx_fail(ctx, ORLOJ_E_UNSUPPORTED, "too many (model, panel) pairs");
        const int64_t need = (int64_t)M * std::max<int64_t>(panels, np_t) * maxcap;
        if (fixed_psum) {
            if ((uint64_t)need > fixed_floats)
                return orloj_ctx_fail(ctx, ORLOJ_E_UNSUPPORTED,
                                      "the call needs %lld scratch floats (models x panels x longest "
                                      "prefix), the fixed scratch holds %zu",
                                      (long long)need, fixed_floats);
        } else {
            hipError_t e = hipSetDevice(ctx->device);
            if (e != hipSuccess) return hip_fail(ctx, e, "hipSetDevice");
            rc = ensure_block(ctx, &ctx->work,
                              std::max((size_t)need * sizeof(float),
                                       (size_t)std::min(need, kTurnedSums) * sizeof(double)));
            if (rc) return rc;
            psum = (float*)ctx->work.p;
        }
    }
    if (turned) {
        TurnedArgs a;
        a.tab = d_ccdf;
        a.sup = d_support;
        a.c0 = d_c0;
        a.c1 = d_c1;
        a.cost = queues->d_cost;
        a.queue_off = queues->d_queue_off;
        a.cls = queues->d_class;
        a.deadline = queues->d_deadline_ms;
        a.now = queues->d_now_ms;
        a.width = grid->d_bin_width_ms;
        a.cand_off = d_cand_off;
        a.prob_off = d_prob_off;
        a.P = d_finish_prob;
        a.E = d_expected_finish;
        a.EL = d_expected_latency_ms;
        a.S = d_score;
        a.err = ctx->d_err;
        a.b = b_expo_per_ms;
        a.C = grid->n_classes;
        a.K = grid->n_bins;
        a.nbs = grid->n_bs;
        a.rect = prefix_mode;
        a.maxcap = (int)maxcap;
        a.Mg = Mg;
        a.compact = compact ? 1 : 0;
        a.nblk = (int)((maxcap + 63) / 64);
        memset(a.bs, 0, sizeof a.bs);
        for (int i = 0; i < grid->n_bs; ++i) a.bs[i] = grid->batch_sizes[i];
        memset(a.act, 0, sizeof a.act);
        if (compact)
            for (int i = 0; i < n_act; ++i) a.act[i] = act[i];
        hipError_t e = hipSetDevice(ctx->device);
        if (e != hipSuccess) return hip_fail(ctx, e, "hipSetDevice");
        a.esum = nullptr;
        a.np_e = 0;
        if (d_c1) {
            a.esum = (double*)(void*)psum;
            a.np_e = (int)np_t;
        }
        // eight waves use a compute unit up, so more workgroups than units have
        // four each and two run on one
        e = launch_turned(a, groups <= n_cu ? 8 : 4, ctx->stream);
        if (e != hipSuccess) return hip_fail(ctx, e, "turned_kernel launch");
        return ORLOJ_OK;
    }

    ScoreArgs a;
    a.tab = d_ccdf;
    a.sup = d_support;
    a.c0 = d_c0;
    a.c1 = d_c1;
    a.cost = queues->d_cost;
    a.fill = ctx->d_fill;
    a.queue_off = queues->d_queue_off;
    a.cls = queues->d_class;
    a.deadline = queues->d_deadline_ms;
    a.now = queues->d_now_ms;
    a.width = grid->d_bin_width_ms;
    a.cand_off = d_cand_off;
    a.prob_off = d_prob_off;
    a.P = d_finish_prob;
    a.E = d_expected_finish;
    a.EL = d_expected_latency_ms;
    a.S = d_score;
    a.err = ctx->d_err;
    a.b = b_expo_per_ms;
    a.M = M;
    a.C = grid->n_classes;
    a.K = grid->n_bins;
    a.nbs = grid->n_bs;
    a.rect = prefix_mode;
    a.maxcap = (int)maxcap;
    a.Mg = Mg;
    a.compact = compact ? 1 : 0;
    memset(a.bs, 0, sizeof a.bs);
    for (int i = 0; i < grid->n_bs; ++i) a.bs[i] = grid->batch_sizes[i];
    memset(a.act, 0, sizeof a.act);
    if (compact)
        for (int i = 0; i < n_act; ++i) a.act[i] = act[i];

    hipError_t e = hipSetDevice(ctx->device);
    if (e != hipSuccess) return hip_fail(ctx, e, "hipSetDevice");
    a.psum = nullptr;
    a.np_e = 0;
    if (d_c1) {
        // emax_kernel's panel sums, formed first, on the score waves' own panels
        a.psum = psum;
        a.np_e = panels;
        switch (cpl) {
            case 1: e = launch_emax<1>(a, ctx->stream); break;
            case 2: e = launch_emax<2>(a, ctx->stream); break;
            case 4: e = launch_emax<4>(a, ctx->stream); break;
            case 8: e = launch_emax<8>(a, ctx->stream); break;
            default: e = launch_emax<16>(a, ctx->stream); break;
        }
        if (e != hipSuccess) return hip_fail(ctx, e, "emax_kernel launch");
    }
    const unsigned g = (unsigned)nblk;
    static_assert(kMaxChunk == 16, "launch table below");
    static_assert((ORLOJ_MAX_BINS + 64 * kMaxChunk - 1) / (64 * kMaxChunk) <= kMaxPanels, "panels");
    switch (cpl) {
        case 1: e = launch_score<1>(a, g, ctx->stream); break;
        case 2: e = launch_score<2>(a, g, ctx->stream); break;
        case 4: e = launch_score<4>(a, g, ctx->stream); break;
        case 8: e = launch_score<8>(a, g, ctx->stream); break;
        default: e = launch_score<16>(a, g, ctx->stream); break;
    }
    if (e != hipSuccess) return hip_fail(ctx, e, "score_kernel launch");
    return ORLOJ_OK;
}

// orloj_select_batch; a scheduling round also passes the flags its
// workgroups set (d_done).
int select_common(orloj_ctx* ctx, const orloj_grid* grid, const orloj_queues* queues,
                  int32_t prefix_mode, const int64_t* d_cand_off, const float* d_score,
                  int32_t* d_sel_n, int32_t* d_sel_bs, float* d_sel_score, int32_t* d_done = nullptr, int32_t round = 0, int* n_groups = nullptr) {
    if (!ctx) return ORLOJ_E_INVALID;
    int rc = check_grid(ctx, grid);
    if (rc) return rc;
    rc = check_queues(ctx, grid, queues);
    if (rc) return rc;
    if (prefix_mode != ORLOJ_PREFIX_TRIANGLE && prefix_mode != ORLOJ_PREFIX_RECT)
        return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "prefix_mode %d", prefix_mode);
    const int M = grid->n_models;
    if (M == 0) return ORLOJ_OK;
    if (!d_cand_off || !d_sel_n || !d_sel_bs || !d_sel_score)
        return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "NULL device buffer");
    const int64_t total = queues->h_queue_off[M];
    if (total > 0 && !d_score) return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "d_score is NULL");
    SelectArgs a;
    a.done = d_done;
    a.round = round;
    a.queue_off = queues->d_queue_off;
    a.cand_off = d_cand_off;
    a.S = d_score;
    a.sel_n = d_sel_n;
    a.sel_bs = d_sel_bs;
    a.sel_score = d_sel_score;
    a.nbs = grid->n_bs;
    a.rect = prefix_mode;
    a.M = M;
    memset(a.bs, 0, sizeof a.bs);
    for (int i = 0; i < grid->n_bs; ++i) a.bs[i] = grid->batch_sizes[i];
    // the models with a queue, when they are few enough to list: one
    // workgroup each, and one more that clears the others
    int n_act = 0;
    for (int q = 0; q < M; ++q)
        if (queues->h_queue_off[q + 1] > queues->h_queue_off[q]) {
            if (n_act < kMaxActive) a.act[n_act] = q;
            ++n_act;
        }
    a.compact = n_act < M && n_act <= kMaxActive;
    a.n_act = n_act;
    const unsigned g = a.compact ? (unsigned)(n_act + 1) : (unsigned)M;
    if (n_groups) *n_groups = (int)g;
    hipError_t e = hipSetDevice(ctx->device);
    if (e != hipSuccess) return hip_fail(ctx, e, "hipSetDevice");
    hipLaunchKernelGGL(select_kernel, dim3(g), dim3(kSelThreads), 0, ctx->stream, a);
    e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(ctx, e, "select_kernel launch");
    return ORLOJ_OK;
}

}  // namespace

extern "C" {

int orloj_score_candidates(orloj_ctx* ctx, const orloj_grid* grid, const float* d_ccdf,
                           const int32_t* d_support, const orloj_queues* queues, double b_expo_per_ms, int32_t prefix_mode,
                           const int64_t* d_cand_off, const int64_t* d_prob_off,
                           float* d_finish_prob, double* d_expected_finish,
                           float* d_expected_latency_ms, float* d_score) {
    return score_common(ctx, grid, d_ccdf, d_support, nullptr, nullptr, queues, b_expo_per_ms,
                        prefix_mode, d_cand_off, d_prob_off, d_finish_prob, d_expected_finish,
                        d_expected_latency_ms, d_score);
}

int orloj_score_candidates_affine(orloj_ctx* ctx, const orloj_grid* grid, const float* d_ccdf,
                                  const int32_t* d_support, const double* d_c0_ms,
                                  const double* d_c1, const orloj_queues* queues,
                                  double b_expo_per_ms, int32_t prefix_mode,
                                  const int64_t* d_cand_off, const int64_t* d_prob_off,
                                  float* d_finish_prob, double* d_expected_finish,
                                  float* d_expected_latency_ms, float* d_score) {
    if (!ctx) return ORLOJ_E_INVALID;
    if (grid && grid->n_models > 0 && (!d_c0_ms || !d_c1))
        return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "d_c0_ms / d_c1 is NULL");
    return score_common(ctx, grid, d_ccdf, d_support, d_c0_ms, d_c1, queues, b_expo_per_ms,
                        prefix_mode, d_cand_off, d_prob_off, d_finish_prob, d_expected_finish,
                        d_expected_latency_ms, d_score);
}

int orloj_score_candidates_affine_noalloc(orloj_ctx* ctx, const orloj_grid* grid,
                                          const float* d_ccdf, const int32_t* d_support,
                                          const double* d_c0_ms, const double* d_c1,
                                          const orloj_queues* queues, double b_expo_per_ms,
                                          int32_t prefix_mode, const int64_t* d_cand_off,
                                          const int64_t* d_prob_off, float* d_finish_prob,
                                          double* d_expected_finish,
                                          float* d_expected_latency_ms, float* d_score) {
    if (!ctx) return ORLOJ_E_INVALID;
    if (grid && grid->n_models > 0 && (!d_c0_ms || !d_c1))
        return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "d_c0_ms / d_c1 is NULL");
    if (!ctx->noalloc_scratch)
        return orloj_ctx_fail(ctx, ORLOJ_E_HIP, "fixed scratch unavailable on device %d: %s",
                              ctx->device, hipGetErrorString(ctx->noalloc_err));
    return score_common(ctx, grid, d_ccdf, d_support, d_c0_ms, d_c1, queues, b_expo_per_ms,
                        prefix_mode, d_cand_off, d_prob_off, d_finish_prob, d_expected_finish,
                        d_expected_latency_ms, d_score, ctx->noalloc_scratch,
                        kNoAllocScratchFloats);
}

int orloj_build_model_laws(orloj_ctx* ctx, const orloj_grid* grid, const float* d_ccdf,
                           const double* d_class_weights, double b_expo_per_ms, float* d_law,
                           float* d_disc, float* d_model_el) {
    if (!ctx) return ORLOJ_E_INVALID;
    int rc = check_grid(ctx, grid);
    if (rc) return rc;
    if (!(b_expo_per_ms > 0.0) || !isfinite(b_expo_per_ms))
        return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "b_expo_per_ms must be finite and > 0");
    if (grid->n_models == 0) return ORLOJ_OK;
    if (!d_ccdf || !d_law || !d_disc || !d_model_el)
        return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "NULL device buffer");
    const int64_t nblk = (int64_t)grid->n_models * grid->n_bs;
    if (nblk > 0x7fffffff) return orloj_ctx_fail(ctx, ORLOJ_E_UNSUPPORTED, "too many (model, batch size) pairs");
    LawArgs a;
    a.tab = d_ccdf;
    a.weights = d_class_weights;
    a.width = grid->d_bin_width_ms;
    a.law = d_law;
    a.disc = d_disc;
    a.model_el = d_model_el;
    a.err = ctx->d_err;
    a.b = b_expo_per_ms;
    a.M = grid->n_models;
    a.C = grid->n_classes;
    a.K = grid->n_bins;
    a.nbs = grid->n_bs;
    memset(a.bs, 0, sizeof a.bs);
    for (int i = 0; i < grid->n_bs; ++i) a.bs[i] = grid->batch_sizes[i];
    hipError_t e = hipSetDevice(ctx->device);
    if (e != hipSuccess) return hip_fail(ctx, e, "hipSetDevice");
    a.pm = nullptr;
    a.vshift = 0;
    const int vpt = chunk_per_lane(grid->n_bins);
    if (law_split(ctx, nblk, a.C, a.K) && nblk * a.C <= 0x7fffffff && !capturing(ctx) && have_mix(ctx)) {
        a.pm = (double*)ctx->mix.p;
        while ((1 << a.vshift) < vpt) ++a.vshift;
        const bool vec = a.K % 4 == 0 && ((uintptr_t)a.tab & 15) == 0;
        const int per = vec ? 4 : 1;
        const int mix_threads = std::min(kMixThreads, (a.K + 64 * per - 1) / (64 * per) * 64);
        e = vec ? launch_laws_mix<true>(a, (unsigned)nblk, mix_threads, ctx->stream)
                : launch_laws_mix<false>(a, (unsigned)nblk, mix_threads, ctx->stream);
        if (e != hipSuccess) return hip_fail(ctx, e, "laws_mix_kernel launch");
        const unsigned rows = (unsigned)(nblk * a.C);
        switch (vpt) {
            case 1: e = launch_laws_rows<1>(a, rows, ctx->stream); break;
            case 2: e = launch_laws_rows<2>(a, rows, ctx->stream); break;
            case 4: e = launch_laws_rows<4>(a, rows, ctx->stream); break;
            case 8: e = launch_laws_rows<8>(a, rows, ctx->stream); break;
            case 16: e = launch_laws_rows<16>(a, rows, ctx->stream); break;
            default: e = launch_laws_rows<32>(a, rows, ctx->stream); break;
        }
        if (e != hipSuccess) return hip_fail(ctx, e, "laws_row_kernel launch");
        return ORLOJ_OK;
    }
    const unsigned g = (unsigned)nblk;
    switch (vpt) {
        case 1: launch_laws<1>(a, g, ctx->stream); break;
        case 2: launch_laws<2>(a, g, ctx->stream); break;
        case 4: launch_laws<4>(a, g, ctx->stream); break;
        case 8: launch_laws<8>(a, g, ctx->stream); break;
        case 16: launch_laws<16>(a, g, ctx->stream); break;
        default: launch_laws<32>(a, g, ctx->stream); break;
    }
    e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(ctx, e, "laws_kernel launch");
    return ORLOJ_OK;
}

int orloj_iterate(orloj_ctx* ctx, const orloj_grid* grid, const int32_t* d_support,
                  const float* d_law, const float* d_disc, const float* d_model_el,
                  const orloj_queues* queues, const orloj_steps* steps, double b_expo_per_ms,
                  int32_t* d_timed_out, float* d_score, int32_t* d_cand_bs, int32_t* d_batch) {
    if (!ctx) return ORLOJ_E_INVALID;
    int rc = check_grid(ctx, grid);
    if (rc) return rc;
    rc = check_queues(ctx, grid, queues);
    if (rc) return rc;
    if (!(b_expo_per_ms > 0.0) || !isfinite(b_expo_per_ms))
        return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "b_expo_per_ms must be finite and > 0");
    const int M = grid->n_models;
    if (M == 0) return ORLOJ_OK;
    const int bs_max = grid->batch_sizes[grid->n_bs - 1];
    if (bs_max > kIterMaxBatch)
        return orloj_ctx_fail(ctx, ORLOJ_E_UNSUPPORTED, "batch size %d > %d", bs_max, kIterMaxBatch);
    int64_t longest = 0;
    for (int q = 0; q < M; ++q) {
        const int64_t N = queues->h_queue_off[q + 1] - queues->h_queue_off[q];
        longest = std::max(longest, N);
        if (N > kIterMaxQueue)
            return orloj_ctx_fail(ctx, ORLOJ_E_UNSUPPORTED, "queue of model %d holds %lld > %d requests", q,
                        (long long)N, kIterMaxQueue);
    }
    if (!d_support || !d_law || !d_disc || !d_model_el || !d_cand_bs || !d_batch)
        return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "NULL device buffer");
    if (queues->h_queue_off[M] > 0 && (!d_timed_out || !d_score))
        return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "NULL per-request output");
    if (steps) {
        const int64_t* so = steps->h_step_off;
        if (!so || !steps->d_step_off || !steps->d_step_deadline_ms || !steps->d_step_cost)
            return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "incomplete orloj_steps");
        if (so[0] != 0) return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "h_step_off[0] != 0");
        for (int64_t r = 0; r < queues->h_queue_off[M]; ++r)
            if (so[r + 1] <= so[r])
                return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "request %lld has no cost step", (long long)r);
    }
    IterArgs a;
    a.sup = d_support;
    a.law = d_law;
    a.disc = d_disc;
    a.model_el = d_model_el;
    a.queue_off = queues->d_queue_off;
    a.cls = queues->d_class;
    a.deadline = queues->d_deadline_ms;
    a.now = queues->d_now_ms;
    a.width = grid->d_bin_width_ms;
    a.cost = queues->d_cost;
    a.step_off = steps ? steps->d_step_off : nullptr;
    a.step_dl = steps ? steps->d_step_deadline_ms : nullptr;
    a.step_cost = steps ? steps->d_step_cost : nullptr;
    a.timed_out = d_timed_out;
    a.score = d_score;
    a.cand_bs = d_cand_bs;
    a.batch = d_batch;
    a.err = ctx->d_err;
    a.b = b_expo_per_ms;
    a.M = M;
    a.C = grid->n_classes;
    a.K = grid->n_bins;
    a.nbs = grid->n_bs;
    a.bs_max = bs_max;
    memset(a.bs, 0, sizeof a.bs);
    for (int i = 0; i < grid->n_bs; ++i) a.bs[i] = grid->batch_sizes[i];
    hipError_t e = hipSetDevice(ctx->device);
    if (e != hipSuccess) return hip_fail(ctx, e, "hipSetDevice");
    a.part_cnt = a.part_first = nullptr;
    a.parts = 0;
    const bool stage = a.nbs > 32 && (int64_t)a.C * (a.nbs + 1) <= kIterStage;
    // A long queue on few models leaves most of the chip idle while one
    // workgroup per model walks it: the drop phase then runs in parts of
    // kDropPart requests, one workgroup each, before the rest per model.
    const int n_cu = ctx->n_cu > 0 ? ctx->n_cu : 256;
    if (longest > kIterWideQueue && 4 * (int64_t)M <= n_cu) {
        const int P = (int)((longest + kDropPart - 1) / kDropPart);
        const size_t n = (size_t)M * (size_t)P * (size_t)a.nbs;
        int rc2 = ensure_block(ctx, &ctx->drop, 2 * n * sizeof(int32_t));
        if (rc2) return rc2;
        a.part_cnt = static_cast<int32_t*>(ctx->drop.p);
        a.part_first = a.part_cnt + n;
        a.parts = P;
        const dim3 g((unsigned)(M * P));
        if (stage)
            hipLaunchKernelGGL((iterate_kernel<kThreads, true, kIterDropPart>), g, dim3(kThreads), 0, ctx->stream, a);
        else
            hipLaunchKernelGGL((iterate_kernel<kThreads, false, kIterDropPart>), g, dim3(kThreads), 0, ctx->stream, a);
        e = hipGetLastError();
        if (e != hipSuccess) return hip_fail(ctx, e, "iterate_kernel launch");
        hipLaunchKernelGGL((iterate_kernel<1024, false, kIterFromParts>), dim3(M), dim3(1024), 0, ctx->stream, a);
    } else if (longest > kIterWideQueue) {
        if (stage)
            hipLaunchKernelGGL((iterate_kernel<1024, true, kIterWhole>), dim3(M), dim3(1024), 0, ctx->stream, a);
        else
            hipLaunchKernelGGL((iterate_kernel<1024, false, kIterWhole>), dim3(M), dim3(1024), 0, ctx->stream, a);
    } else if (stage) {
        hipLaunchKernelGGL((iterate_kernel<kThreads, true, kIterWhole>), dim3(M), dim3(kThreads), 0, ctx->stream, a);
    } else {
        hipLaunchKernelGGL((iterate_kernel<kThreads, false, kIterWhole>), dim3(M), dim3(kThreads), 0, ctx->stream, a);
    }
    e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(ctx, e, "iterate_kernel launch");
    return ORLOJ_OK;
}

int orloj_accumulate(orloj_ctx* ctx, const orloj_grid* grid, int64_t n_samples,
                     const int32_t* d_model, const int32_t* d_bs_index, const int32_t* d_class,
                     const double* d_latency_ms, uint32_t* d_counts,
                     unsigned long long* d_n_rejected) {
    if (!ctx) return ORLOJ_E_INVALID;
    int rc = check_grid(ctx, grid);
    if (rc) return rc;
    if (n_samples < 0) return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "n_samples < 0");
    if (n_samples == 0) return ORLOJ_OK;
    if (!d_model || !d_bs_index || !d_class || !d_latency_ms || !d_counts || !grid->d_bin_width_ms)
        return orloj_ctx_fail(ctx, ORLOJ_E_INVALID, "NULL device buffer");
    AccArgs a;
    a.model = d_model;
    a.bs_index = d_bs_index;
    a.cls = d_class;
    a.latency = d_latency_ms;
    a.width = grid->d_bin_width_ms;
    a.counts = d_counts;
    a.n_rejected = d_n_rejected;
    a.n = n_samples;
    a.M = grid->n_models;
    a.nbs = grid->n_bs;
    a.C = grid->n_classes;
    a.K = grid->n_bins;
    hipError_t e = hipSetDevice(ctx->device);
    if (e != hipSuccess) return hip_fail(ctx, e, "hipSetDevice");
    const int64_t want = (n_samples + kThreads - 1) / kThreads;
    const unsigned g = (unsigned)(want < 4096 ? want : 4096);
    hipLaunchKernelGGL(accumulate_kernel, dim3(g), dim3(kThreads), 0, ctx->stream, a);
    e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(ctx, e, "accumulate_kernel launch");
    return ORLOJ_OK;
}

int orloj_select_batch(orloj_ctx* ctx, const orloj_grid* grid, const orloj_queues* queues,
                       int32_t prefix_mode, const int64_t* d_cand_off, const float* d_score,
                       int32_t* d_sel_n, int32_t* d_sel_bs, float* d_sel_score) {
    return select_common(ctx, grid, queues, prefix_mode, d_cand_off, d_score, d_sel_n, d_sel_bs,
                         d_sel_score);
}

}  // extern "C"

int orloj_internal_score_select(orloj_ctx* ctx, const orloj_grid* grid, const float* d_ccdf,
                                const int32_t* d_support, const orloj_queues* queues,
                                double b_expo_per_ms, const int64_t* d_cand_off,
                                const int64_t* d_prob_off, float* d_finish_prob,
                                double* d_expected_finish, float* d_expected_latency_ms,
                                float* d_score, int32_t* d_sel_n, int32_t* d_sel_bs,
                                float* d_sel_score, int32_t* d_done, int32_t round, int* n_groups) {
    int rc = score_common(ctx, grid, d_ccdf, d_support, nullptr, nullptr, queues, b_expo_per_ms,
                          ORLOJ_PREFIX_TRIANGLE, d_cand_off, d_prob_off, d_finish_prob,
                          d_expected_finish, d_expected_latency_ms, d_score);
    if (rc) return rc;
    return select_common(ctx, grid, queues, ORLOJ_PREFIX_TRIANGLE, d_cand_off, d_score, d_sel_n,
                         d_sel_bs, d_sel_score, d_done, round, n_groups);
}

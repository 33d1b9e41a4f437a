// Shared device helpers of the gfx950 MoE-layer kernels: bf16 packing, MFMA fragment types,
// 64-lane wavefront reductions.  Internal to the library; the public boundary is include/moe_layer.h.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "moe_layer.h"

#define MOE_WAVE 64

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;   // one MFMA A/B fragment (8 bf16 along K)
typedef __attribute__((ext_vector_type(4))) float f32x4;     // 16x16 accumulator fragment
typedef __attribute__((ext_vector_type(16))) float f32x16;   // 32x32 accumulator fragment

// Lane layouts of the two CDNA4 bf16 MFMA shapes used here (l = lane id):
//   16x16x32: A[i][k] from lane l: i = l%16, k = 8*(l/16)+0..7; B[k][j]: j = l%16, same k;
//             D[i][j]: lane l holds i = 4*(l/16)+r (r=0..3), j = l%16.
//   32x32x16: A[i][k]: i = l%32, k = 8*(l/32)+0..7; B[k][j]: j = l%32, same k;
//             D[i][j]: lane l holds i = 8*b + 4*(l/32) + r (b=0..3, r=0..3, element 4*b+r), j = l%32.

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;   // 16 bytes = 8 bf16, as loaded
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

__device__ __forceinline__ bf16x8 as_frag(u32x4 u) { return __builtin_bit_cast(bf16x8, u); }
__device__ __forceinline__ bf16x8 as_frag(uint4 u) { return __builtin_bit_cast(bf16x8, u); }

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// float -> bf16, round to nearest even, by the hardware conversion of gfx950 (v_cvt_pk_bf16_f32: two values per
// instruction, NaN stays NaN)
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}

__device__ __forceinline__ uint32_t f32_to_bf16(float f) { return pack_bf16x2(f, 0.f) & 0xffffu; }

__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
        v += __shfl_xor(v, o, MOE_WAVE);
    return v;
}

// ---- 64-lane reductions on the DPP crossbar (VALU speed; __shfl_xor goes through LDS and is ~10x slower per step).
// Inclusive row scans by 1, 2, 4, 8 leave each 16-lane row's result in its last lane; the four row results are
// then read with v_readlane, so the value returned is wave-uniform.  The combination order is fixed.
#define MOE_DPP_SHR(ident, v, n) \
    __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(ident), __float_as_int(v), 0x110 + (n), 0xF, 0xF, false))

// six steps on the crossbar (the rows' results broadcast to the next rows) and one read of lane 63
__device__ __forceinline__ int wave_max_int_dpp(int v)
{
    const int lowest = (int)0x80000000u;
    v = max(v, __builtin_amdgcn_update_dpp(lowest, v, 0x111, 0xF, 0xF, false));
    v = max(v, __builtin_amdgcn_update_dpp(lowest, v, 0x112, 0xF, 0xF, false));
    v = max(v, __builtin_amdgcn_update_dpp(lowest, v, 0x114, 0xF, 0xF, false));
    v = max(v, __builtin_amdgcn_update_dpp(lowest, v, 0x118, 0xF, 0xF, false));
    v = max(v, __builtin_amdgcn_update_dpp(lowest, v, 0x142, 0xA, 0xF, false));      // lane 15 of rows 0 and 2 -> rows 1 and 3
    v = max(v, __builtin_amdgcn_update_dpp(lowest, v, 0x143, 0xC, 0xF, false));      // lane 31 -> rows 2 and 3
    return __builtin_amdgcn_readlane(v, 63);
}

__device__ __forceinline__ float wave_sum_dpp(float v)
{
    v += MOE_DPP_SHR(0.f, v, 1);
    v += MOE_DPP_SHR(0.f, v, 2);
    v += MOE_DPP_SHR(0.f, v, 4);
    v += MOE_DPP_SHR(0.f, v, 8);
    const int b = __float_as_int(v);
    const float r0 = __int_as_float(__builtin_amdgcn_readlane(b, 15)), r1 = __int_as_float(__builtin_amdgcn_readlane(b, 31));
    const float r2 = __int_as_float(__builtin_amdgcn_readlane(b, 47)), r3 = __int_as_float(__builtin_amdgcn_readlane(b, 63));
    return (r0 + r1) + (r2 + r3);
}

// silu(g) * u with the hardware reciprocal (1 ulp) in place of an IEEE division: the result is rounded to bf16 anyway
__device__ __forceinline__ float silu_mul(float g, float u) { return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)) * u; }

// ---- work items of the experts that have rows and are masked on, without a schedule pass --------------------
// A launch of (upper bound of working experts) x per_expert blocks: every wave derives the working set itself
// as two 64-bit ballots over counts/mask, the block id is remapped so that each of the 8 XCDs (own L2) gets one
// contiguous run of the compacted item list (expert-major), and the item's expert is found by rank among the set
// bits.  Returns false for a block beyond the list.  All 64 lanes of the wave must call it.
#define MOE_NUM_XCD 8
// rows of experts l and l + 64 in lane l, 0 where the expert does not work
struct moe_rows {
    int c0, c1;
};
// Lane l holds rows and first row of experts l and l + 64.  All reads are on their way at once: counts, then the mask where a
// count allowed it, then rows and first row of the expert found were four round trips (0.5 to 1 us each at the start of a launch).
struct moe_work {
    unsigned long long lo, hi;      // the working experts
    int c0, c1, o0, o1;
    __device__ __forceinline__ int experts() const { return __popcll(lo) + __popcll(hi); }
    __device__ __forceinline__ moe_rows rows() const
    {
        const int l = threadIdx.x & 63;
        return moe_rows{(lo >> l & 1ull) != 0 ? c0 : 0, (hi >> l & 1ull) != 0 ? c1 : 0};
    }
    __device__ __forceinline__ int rows_of(int e) const { return e < 64 ? __builtin_amdgcn_readlane(c0, e) : __builtin_amdgcn_readlane(c1, e - 64); }
    __device__ __forceinline__ int first_row_of(int e) const { return e < 64 ? __builtin_amdgcn_readlane(o0, e) : __builtin_amdgcn_readlane(o1, e - 64); }
};
__device__ __forceinline__ moe_work moe_working_experts(int N, const int32_t *__restrict__ counts, const int32_t *__restrict__ offsets,
                                                        const uint8_t *__restrict__ mask)
{
    const int l = threadIdx.x & 63, l0 = min(l, N - 1), l1 = min(l + 64, N - 1);
    moe_work w;
    w.c0 = counts[l0];
    w.c1 = counts[l1];
    w.o0 = offsets[l0];
    w.o1 = offsets[l1];
    int m0 = 1, m1 = 1;
    if (mask != nullptr) {
        m0 = mask[l0];
        m1 = mask[l1];
    }
    w.lo = __ballot(l < N && w.c0 > 0 && m0 != 0);
    w.hi = __ballot(l + 64 < N && w.c1 > 0 && m1 != 0);
    return w;
}

// place of block pid in a list of total items of which every XCD takes a contiguous run (pid < total)
__device__ __forceinline__ int moe_xcd_run(int total, int pid)
{
    const int q = total / MOE_NUM_XCD, rem = total % MOE_NUM_XCD;
    const int xcd = pid % MOE_NUM_XCD, loc = pid / MOE_NUM_XCD;
    return xcd < rem ? xcd * (q + 1) + loc : rem * (q + 1) + (xcd - rem) * q + loc;
}

// item L of (working experts) x per_expert items: its expert and its place there
__device__ __forceinline__ void moe_item_at(const moe_work &w, int per_expert, int L, int &e, int &local)
{
    const int l = threadIdx.x & 63;
    const int n_lo = __popcll(w.lo);
    int a = L / per_expert;
    local = L - a * per_expert;
    unsigned long long m = w.lo;
    int base = 0;
    if (a >= n_lo) {
        a -= n_lo;
        m = w.hi;
        base = 64;
    }
    const unsigned long long below = l == 0 ? 0ull : (m << (64 - l));     // the bits of m under position l
    const bool mine = ((m >> l) & 1ull) != 0 && __popcll(below) == a;
    e = base + __ffsll((unsigned long long)__ballot(mine)) - 1;
}

// the item of block pid, or false beyond the list
__device__ __forceinline__ bool moe_item_of(const moe_work &w, int per_expert, int pid, int &e, int &local)
{
    const int total = w.experts() * per_expert;
    if (pid >= total) return false;
    moe_item_at(w, per_expert, moe_xcd_run(total, pid), e, local);
    return true;
}

// ---- token tiles of the experts that have rows and are masked on, derived by every wave ---------------------
// Lane l holds the rows of experts l and l + 64 (0: masked off), the tiles they make at the launch's tile height and their
// places in the expert-major tile list (a prefix sum on the DPP crossbar).  A table written by a kernel ahead of the
// launch cost that kernel (4.7-6.5 us per FFN call, T > 128) and two dependent reads per block; this costs a block one read
// and about 60 instructions.  All 64 lanes must call these.
struct moe_tiles {
    int n0, n1, first0, first1, total;
};

__device__ __forceinline__ moe_rows moe_masked_rows(int N, const int32_t *__restrict__ counts, const uint8_t *__restrict__ mask)
{
    // all reads on their way at once: with the count read only where the mask allows it, up to four reads followed one another
    const int l = threadIdx.x & 63, l0 = min(l, N - 1), l1 = min(l + 64, N - 1);
    const int c0 = counts[l0], c1 = counts[l1];
    int m0 = 1, m1 = 1;
    if (mask != nullptr) {
        m0 = mask[l0];
        m1 = mask[l1];
    }
    return moe_rows{l < N && m0 != 0 ? max(c0, 0) : 0, l + 64 < N && m1 != 0 ? max(c1, 0) : 0};
}

// sum over the wave of v, uniform, and the sum over lanes 0 .. l (inclusive) in v
__device__ __forceinline__ int wave_scan_int_dpp(int &v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);      // lanes 1, 2, 4, 8 below, within rows of 16
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
    const int r0 = __builtin_amdgcn_readlane(v, 15), r1 = r0 + __builtin_amdgcn_readlane(v, 31);
    const int r2 = r1 + __builtin_amdgcn_readlane(v, 47), r3 = r2 + __builtin_amdgcn_readlane(v, 63);
    const int row = (threadIdx.x & 63) >> 4;
    v += row == 0 ? 0 : row == 1 ? r0 : row == 2 ? r1 : r2;
    return r3;
}
__device__ __forceinline__ int wave_sum_int_dpp(int v) { return wave_scan_int_dpp(v); }

// n0, n1: tiles of this lane's experts
__device__ __forceinline__ moe_tiles moe_rank_tiles(int n0, int n1)
{
    moe_tiles t = {n0, n1, n0, n1, 0};
    const int lo = wave_scan_int_dpp(t.first0);
    t.total = lo + wave_scan_int_dpp(t.first1);
    t.first0 -= n0;
    t.first1 += lo - n1;
    return t;
}

// tile i of the list (i < total): expert, its first tile, its tiles (all uniform)
__device__ __forceinline__ void moe_find_tile(const moe_tiles &t, int i, int &e, int &first, int &n)
{
    const unsigned long long in_lo = __ballot(i >= t.first0 && i < t.first0 + t.n0);
    const unsigned long long in_hi = __ballot(i >= t.first1 && i < t.first1 + t.n1);
    const int l = __ffsll((unsigned long long)(in_lo != 0ull ? in_lo : in_hi)) - 1;
    e = in_lo != 0ull ? l : l + 64;
    first = in_lo != 0ull ? __builtin_amdgcn_readlane(t.first0, l) : __builtin_amdgcn_readlane(t.first1, l);
    n = in_lo != 0ull ? __builtin_amdgcn_readlane(t.n0, l) : __builtin_amdgcn_readlane(t.n1, l);
}

// K splits of the tiled down projection, decided on the device from the number of tile items that have work.  The
// cost of a launch is taken as (rounds of 256 compute units) x (item time, 1/nsp of an unsplit item); starting from no
// split, the next power of two up to nsp_max is taken whenever it lowers that cost by 15 % or more.  224 items stay
// whole (448 halves would need two rounds), 160 items run as 1280 eighths in 5 rounds (0.63 of a round of whole items).
__host__ __device__ __forceinline__ int moe_dev_splits(int items, int nsp_max)
{
    if (items <= 0) return 1;
    int nsp = 1, cost = ((items + 255) / 256) * 64;            // 64 = an unsplit item
    for (int finer = 2; finer <= nsp_max; finer *= 2) {
        const int c = ((items * finer + 255) / 256) * (64 / finer);
        if (c * 100 <= cost * 85) {
            cost = c;
            nsp = finer;
        }
    }
    return nsp;
}

#define MOE_CHECK_LAUNCH()                       \
    do {                                         \
        if (hipGetLastError() != hipSuccess)     \
            return MOE_ELAUNCH;                  \
    } while (0)

static inline size_t moe_align256(size_t x) { return (x + 255) & ~(size_t)255; }

// ---- workspace layout (one per shape; every entry point carves what it needs from offset 0) ----
// The expert FFN uses act, partial and choice, a gate product `route` (routing and prediction different parts of it): calls of different
// kinds may run side by side on one workspace.
struct moe_ws_layout {
    size_t act;        // [T*k, I] bf16 inner activations
    size_t partial;    // [nsplit, T*k, d] fp32 split-K partial sums of the down projection (skinny path, or the tiled path's K splits);
                       // in a joint launch (ffn_joint.h), which splits no K, its tickets and the counters of its token tiles
    size_t choice;     // whether the long-K kernel takes the down projection (one word)
    size_t route;      // routing scratch: sigmoid gates of the shared experts [T <= 16], idx [T*k], w [T*k] (prediction), 2 x logits [max(T,16), N] (gate product and selection in separate launches)
    size_t total;
};

#define MOE_SKINNY_MAX_T 16
#define MOE_SKINNY_WAVES 4          // waves per block on the skinny path
#define MOE_SKINNY_MAX_STEPS 32     // 32-wide K steps a wave may hold in registers (K <= 1024 per wave)
#define MOE_TILE_M 128              // token rows per tile on the tiled path (the down projection may choose 112 or 96 on the device)
#define MOE_TILE_M_MIN 96
// down projection over a long inner size (ffn_wide.h)
#define WIDE_TM 256                 // activation rows per item
#define WIDE_TN 256                 // output columns per item
#define WIDE_MAX_SPLIT 16           // most pieces of one item
#define WIDE_MAX_PIECES 256         // most pieces of items of a launch: one round of compute units (64 MB of fp32 partial sums)
#define MOE_SKINNY_DOWN_MIN_I 2048  // decode-sized down projections with I up to this run on the tiled kernel where it has enough items

static inline int moe_skinny_nsplit(int K)
{
    int per_block = MOE_SKINNY_WAVES * MOE_SKINNY_MAX_STEPS * 32;
    return (K + per_block - 1) / per_block;
}

// Tiled down projection: the most K splits a launch may use (1 = never split).  Every split keeps at least 32 k32 steps, a
// multiple of 8; the fp32 partial sums [nsp, T*k, d] must fit 64 MB.  Whether a launch splits at all is decided on
// the device (moe_dev_splits): only when the experts that have rows and are masked on leave compute units without a tile.
static inline int moe_tiled_down_max_splits(const moe_shape *s)
{
    if (s->T <= MOE_SKINNY_MAX_T) return 1;
    const int steps = s->I / 32;
    int nsp = 1;
    while (nsp < 8 && steps % (2 * nsp * 8) == 0 && steps / (2 * nsp) >= 32 &&
           (size_t)(2 * nsp) * s->T * s->k * s->d * 4 <= ((size_t)64 << 20))
        nsp *= 2;
    return nsp;
}

// Whether the kernel for long inner sizes (ffn_wide.h) is launched beside the tiled down projection; which of the two then
// works is decided on the device from the rows of the experts at work (wide_faster).  The launches that only return cost 8 us
// where this kernel works and 3 to 7 where the tiled one does, so both are launched only where the projection takes 100 us
// and more: 2^36 multiplications, 48 MB of activations, and too many rows for the tiled kernel to split K
// (moe_tiled_down_max_splits), which up to there fills the chip by itself (Mixtral shape, up to 1024 tokens).  Shorter inner
// sizes have items too short to be worth cutting (I = 5632: 97 us on the tiled kernel, 101 on this one).
static inline bool moe_wide_down(const moe_shape *s)
{
    const size_t a = (size_t)s->T * s->k * s->I;
    return s->T > 128 && s->I >= 8192 && a * 2 >= ((size_t)48 << 20) && a >= ((size_t)1 << 36) / s->d &&
           moe_tiled_down_max_splits(s) == 1 && (size_t)s->d * s->I * 2 < ((size_t)1 << 32);
}

// Most items of that kernel, and most pieces a launch of it can cut: its partial sums.
static inline size_t moe_wide_max_items(const moe_shape *s)
{
    const size_t R = (size_t)s->T * s->k, N = (size_t)s->N;
    return (R / WIDE_TM + (N < R ? N : R)) * (size_t)((s->d + WIDE_TN - 1) / WIDE_TN);
}
static inline size_t moe_wide_max_pieces(const moe_shape *s)
{
    const size_t n = WIDE_MAX_SPLIT * moe_wide_max_items(s);
    return n < WIDE_MAX_PIECES ? n : WIDE_MAX_PIECES;
}

// Joint launch: the tickets of sixteen queues, a line each, then a counter for every token tile.
#define MOE_JOINT_TICKET_STRIDE 32
#define MOE_JOINT_TICKETS (2 * MOE_NUM_XCD * MOE_JOINT_TICKET_STRIDE)
#define MOE_JOINT_MAX_POLLS (1 << 21)
static inline size_t moe_joint_max_tiles(const moe_shape *s)
{
    const size_t R = (size_t)s->T * s->k, N = (size_t)s->N;
    return R / MOE_TILE_M + (N < R ? N : R);
}
static inline size_t moe_joint_scratch_bytes(const moe_shape *s) { return (MOE_JOINT_TICKETS + moe_joint_max_tiles(s)) * 4; }

// one [max(T, 16), N] fp32 block of gate logits (the gate product and the selection are separate launches when the
// gate matrix has many rows)
static inline size_t moe_logits_scratch_bytes(const moe_shape *s)
{
    return moe_align256((size_t)(s->T > 16 ? s->T : 16) * (size_t)s->N * 4);
}

static inline moe_ws_layout moe_ws(const moe_shape *s)
{
    moe_ws_layout L;
    size_t R = (size_t)s->T * s->k;
    size_t off = 0;
    L.act = off;
    off += moe_align256(R * (size_t)s->I * 2);
    L.partial = off;
    size_t Rs = R < (size_t)MOE_SKINNY_MAX_T * MOE_MAX_TOPK ? R : (size_t)MOE_SKINNY_MAX_T * MOE_MAX_TOPK;
    size_t part = (size_t)moe_skinny_nsplit(s->I) * Rs * s->d * 4;
    const int nsp = moe_tiled_down_max_splits(s);
    if (nsp > 1 && (size_t)nsp * R * s->d * 4 > part) part = (size_t)nsp * R * s->d * 4;
    const size_t pieces = moe_wide_down(s) ? moe_wide_max_pieces(s) * WIDE_TM * WIDE_TN * 4 : 0;
    if (pieces > part) part = pieces;
    // 17 and more rows of d sums hold it but for millions of rows of a narrow layer
    if (s->T > MOE_SKINNY_MAX_T && moe_joint_scratch_bytes(s) > part) part = moe_joint_scratch_bytes(s);
    off += moe_align256(part);
    L.choice = off;
    off += 256;
    L.route = off;
    off += moe_align256(MOE_MAX_EXPERTS * 4) + 2 * moe_align256(R * 4) + 2 * moe_logits_scratch_bytes(s);
    L.total = off;
    return L;
}

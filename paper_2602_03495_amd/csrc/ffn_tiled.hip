// Grouped SwiGLU expert FFN for prefill-sized batches on gfx950.
//
// Two grouped GEMMs over the rows of the masked-on, non-empty experts:
//   up:    act[p, i] = silu(x_p . W1_e[i,:]) * (x_p . W3_e[i,:])      x_p = h[perm[p]/k, :] gathered in the tile load
//   down:  y[p, f]   = act[p,:] . W2_e[f,:]
//
// Design (what the counters said while this was built): with 128-row token tiles the kernel is bound by L2
// request throughput, not by MFMA issue, so the data path is shaped to ask L2 for as little as possible, in
// full 128-byte lines:
//   * Weights are consumed in the packed layout of moe_pack_weights: one MFMA 16x16x32 A fragment (16 weight
//     rows x 32 k) is 1 KB of contiguous memory in lane order.  Every wave owns a private set of weight rows,
//     so weights never pass through LDS: global_load_dwordx4 -> VGPR -> MFMA, prefetched 3 k32-steps ahead in
//     4 rotating register sets (the compiler's own vmcnt tracking keeps ~12 loads per wave in flight).
//   * The token tile (128 rows, shared by all 8 waves) is staged through LDS in k64 stages (16 KB each,
//     double buffered, 128-byte global requests), loaded two stages ahead so that waiting for it never
//     drains the weight prefetch queue (vmcnt retires in order).
//   * 8 waves per block (2 per SIMD, 128 fp32 accumulator registers each): one wave's barrier or load wait is
//     covered by the other's MFMAs, and the accumulators stay in place (no AGPR shuffling).
//   * The MFMA takes weight rows as A and token rows as B, so a lane ends up with 4 consecutive output columns
//     of one token: SwiGLU is applied in registers; the result leaves through LDS in whole runs of a row.
// A work item is (expert, 128-row token tile, weight tile); every wave derives the item list from counts and mask
// (moe_rank_tiles; up to 128 tokens an expert has at most one token tile and two ballots do), so empty and masked-off
// experts cost nothing, there is no host round trip and no schedule pass ahead of the launch.  Block ids are remapped so that every XCD (own
// L2) works on a contiguous run of items ordered expert-major, weight tile, token tile: the token tiles that
// share a weight tile run side by side on one XCD (measured: the same items spread round-robin over the XCDs
// run up to 40 % slower, even with one token tile per expert).
// Tiles are rarely full: the launch bounds the 16-row subtiles by T and every block runs the body sized for its own
// row count (16, 32, 64, 96, 112 or 128 rows).
// What only the device knows (counts and mask) also shapes the launch there: the last items of a launch run at half width where
// they would fill half a round of compute units or less, in some launches of the up projection all of them (up_runs_halves); with
// few items the down projection splits the K range of its tiles over several (fp32 partial sums, summed in split order by
// tiled_finish_kernel); with many, the blocks pick the token-tile height of the down projection so that its items fill whole rounds
// of compute units.
// The two projections of a whole layer run as one launch of this file's items in ffn_joint.h.
// Each item walks K as a ring starting at an expert-dependent offset, so that the token tiles that share a weight tile
// stay in step (started at different points they run 18 % slower); the summation order is a function of the expert
// and of the number of K splits only, so results are reproducible for given inputs.
#include "moe_common.h"

#include <cstdlib>

// Diagnostics: when a record buffer has been set (moe_debug_set_trace), thread 0 of every block of a tiled launch
// writes its begin / end time (constant 100 MHz clock), where it ran and what it worked on: the timeline of a launch.
// Costs one clock read per block and one scalar load of the pointer when unset.
#define MOE_TRACE_MAX_BLOCKS 65536
__device__ unsigned long long *g_moe_trace = nullptr;
extern "C" int moe_debug_set_trace(unsigned long long *records)
{
    return hipMemcpyToSymbol(HIP_SYMBOL(g_moe_trace), &records, sizeof(records)) == hipSuccess ? MOE_OK : MOE_ELAUNCH;
}
#define MOE_TRACE_BEGIN() const unsigned long long trace_t0_ = wall_clock64()
#define MOE_TRACE_END(mode_, e_, nrows_, nt_)                                                                   \
    do {                                                                                                        \
        unsigned long long *tr_ = g_moe_trace;                                                                  \
        if (tr_ != nullptr && threadIdx.x == 0 && blockIdx.x < MOE_TRACE_MAX_BLOCKS) {                          \
            unsigned hw_, xcc_;                                                                                 \
            asm volatile("s_getreg_b32 %0, hwreg(HW_REG_HW_ID)" : "=s"(hw_));                                   \
            asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc_));                                 \
            unsigned long long *r_ = tr_ + 8ull * (blockIdx.x + (mode_) * (unsigned long long)MOE_TRACE_MAX_BLOCKS); \
            r_[0] = trace_t0_; r_[1] = wall_clock64(); r_[2] = hw_; r_[3] = xcc_;                               \
            r_[4] = (e_); r_[5] = (nrows_); r_[6] = (nt_); r_[7] = 1;                                           \
        }                                                                                                       \
    } while (0)

#define TM MOE_TILE_M     // token rows per tile
#define TILED_THREADS 512

// The up projection uses 128-row tiles.  The down projection has few
// items (8 column tiles of 512 per token tile at d = 4096), so the number of rounds the launch needs on 256 compute
// units moves its duration in steps: 27 token tiles are 216 items, one round with 40 units idle, and 30 tiles of 112
// rows are 240 items, still one round of shorter items.  The tile height of the down projection is therefore chosen
// here, on the device, from the workloads: 128, 112 or 96 rows, whichever gives the smallest (rounds x item time),
// with an item's time taken as proportional to (height + 64): its weight loads do not shrink with the tile.  (A last round of
// items that run as halves, cut_item_of, counts as a whole one here and in moe_dev_splits.)
__device__ __forceinline__ int sched_cost(int tiles, int n_ntc, int tm)
{
    const int items = tiles * n_ntc;
    const int rounds2 = items <= 512 ? 2 * ((items + 255) / 256) : (2 * items + 255) / 256 + 1;   // twice the rounds; beyond two rounds the last one fills unevenly anyway
    return rounds2 * (tm + 64);
}

__device__ __forceinline__ moe_tiles tiles_128(const moe_rows &c) { return moe_rank_tiles((c.c0 + 127) / 128, (c.c1 + 127) / 128); }

// the token tiles of the down projection and their height tm
__device__ __forceinline__ moe_tiles down_tiles(const moe_rows &c, int n_ntc, int &tm)
{
    const moe_tiles t128 = tiles_128(c);
    tm = 128;
    if (t128.total * n_ntc < 256) return t128;              // the K range is split instead
    const int a112 = (c.c0 + 111) / 112, b112 = (c.c1 + 111) / 112, a96 = (c.c0 + 95) / 96, b96 = (c.c1 + 95) / 96;
    int best = sched_cost(t128.total, n_ntc, 128);
    const int c112 = sched_cost(wave_sum_int_dpp(a112 + b112), n_ntc, 112), c96 = sched_cost(wave_sum_int_dpp(a96 + b96), n_ntc, 96);
    if (c112 < best) { best = c112; tm = 112; }
    if (c96 < best) { best = c96; tm = 96; }
    return tm == 128 ? t128 : tm == 112 ? moe_rank_tiles(a112, b112) : moe_rank_tiles(a96, b96);
}

#include "ffn_wide.h"

// MODE 0: up (W1|W3 + SwiGLU -> act); a wave owns NF/2 fragments of W1 and the same NF/2 of W3.
// MODE 1: down (W2 -> y); a wave owns NF consecutive fragments of W2.
// Weight tile of a block: 8 waves x NF fragments x 16 rows.  NTT = 16-row token subtiles computed (rows past
// nrows are clamped copies whose results are dropped).
// ahead_of_stores: called by every wave between its last product and its epilogue.
struct nothing_ahead {
    __device__ __forceinline__ void operator()() const {}
};
template <int MODE, int NF, int NTT, int NSETS, bool FENCED, int WAVES, bool THROUGH = false, class Ahead = nothing_ahead>
__device__ __forceinline__ void tile_body(uint16_t *Xs, char *ys, int d, int I, int k, const uint16_t *__restrict__ xsrc,
                                          const int32_t *__restrict__ perm, const uint16_t *__restrict__ wa,
                                          const uint16_t *__restrict__ wb, uint16_t *__restrict__ out, int e, int nt,
                                          int row0, int nrows, int sp, int nsp, float *__restrict__ part, int R, const int tid, Ahead ahead_of_stores = {})
{
    constexpr int HF = MODE == 0 ? NF / 2 : NF;           // fragments per matrix per wave
    constexpr int WAVE_COLS = HF * 16;                     // output columns a wave produces
    constexpr int NT_COLS = WAVES * WAVE_COLS;             // output columns per block
    constexpr int RPP = WAVES * 8;                         // token rows one pass of the loader covers (8 threads per row)
    constexpr int HALF = (NTT > 8 ? 2 * TM : TM) * 32;     // elements of a k32 half of a stage in LDS; a stage is two, there are two stages
    const int K = MODE == 0 ? d : I;
    const int NOUT = MODE == 0 ? I : d;
    const int n0 = nt * NT_COLS;

    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: lets the weight addresses live in SGPRs
    const int li = lane & 15, lg = lane >> 4;
    const int kb_n = K / 32;                               // k32 blocks per weight row block
    const size_t rb_stride = (size_t)kb_n * 512;           // elements between consecutive 16-row blocks

    // ---- this wave's weight fragments: consecutive row blocks, so one pointer per matrix + a uniform stride
    // (wave-uniform byte base + a 32-bit lane offset: the loads take the scalar-base addressing form)
    const char *wp0, *wp1;
    const uint32_t wlane = lane * 16;
    {
        int col = n0 + wave * WAVE_COLS;
        if (col >= NOUT) col = NOUT - WAVE_COLS;           // a wave past the ragged edge recomputes the last columns
        // + the first k32 step of this item's share of K (MODE 1 with the K range split over nsp items)
        const size_t mat = (size_t)e * d * I + (size_t)(col >> 4) * rb_stride + (size_t)sp * (kb_n / nsp) * 512;
        wp0 = reinterpret_cast<const char *>(wa + mat);
        wp1 = MODE == 0 ? reinterpret_cast<const char *>(wb + mat) : wp0;
    }
    // ---- token tile loader: thread -> rows tid/8 + RPP j (j < XJ), 16-byte chunk tid%8 of the 128-byte k64 segment
    const int xc = tid & 7;
    constexpr int XJ = (NTT * 16 + RPP - 1) / RPP;         // loader passes over the token rows that are in use
    uint32_t xo[XJ];
#pragma unroll
    for (int j = 0; j < XJ; ++j) {
        int r = (tid >> 3) + RPP * j;
        if (r >= nrows) r = nrows - 1;
        if (MODE == 0)                                      // byte offsets: T*d < 2^31 elements keeps them in 32 bits
            xo[j] = ((uint32_t)(perm[row0 + r] / k) * (uint32_t)d + xc * 8) * 2u;
        else
            xo[j] = ((uint32_t)r * (uint32_t)I + xc * 8) * 2u;
    }
    const char *xbase = reinterpret_cast<const char *>(MODE == 0 ? xsrc : xsrc + (size_t)row0 * I + (size_t)sp * (kb_n / nsp) * 32);
    // LDS holds every 16-row x k32 subtile in MFMA fragment order with a swizzle: the 16 bytes of (row i, k chunk g) of
    // k32 half hf sit in slot 16 g + (i ^ g ^ 8 hf).  A fragment read is then one KB per wave, and the LDS serves a
    // 16-byte-per-lane read in four passes of 16 lanes -- lanes {0-3, 12-15, 20-23, 24-27} and so on, measured -- which
    // must hit 16 different 16-byte bank groups: i ^ g keeps that (4 clocks per read instead of 8 for plain rows), while
    // the 8 chunks of one row, which one store instruction of the loader carries in 8 adjacent lanes, land in 8
    // different bank groups (16 clocks per store instead of 64 for the unswizzled fragment order).
    uint16_t *xw = Xs + (xc >> 2) * HALF + (tid >> 7) * 512 + ((xc & 3) * 16 + (((tid >> 3) & 15) ^ (xc & 3) ^ (xc >> 2) * 8)) * 8;   // + stage * 2 * HALF + j * RPP rows
    const uint16_t *xrd0 = Xs + (lg * 16 + (li ^ lg)) * 8;       // + stage * 2 * HALF + t * 16 rows
    const uint16_t *xrd1 = Xs + HALF + (lg * 16 + (li ^ lg ^ 8)) * 8;

    f32x4 acc[NF][NTT];
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int t = 0; t < NTT; ++t) acc[f][t] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int nk = kb_n / nsp;    // k32 steps of this item (a multiple of NSETS: the launch checks K)
    const int nst = nk / 2;       // k64 stages
    const int st0 = (int)(((unsigned)e * 5u) % (unsigned)nst);   // where this item's K ring starts (per expert: tiles that share rows or weights stay in step)
    static_assert(NSETS == 4 || NSETS == 8, "an even number of stages per unrolled round");
    u32x4 wr[NSETS][NF];          // W(step) lives in set step % NSETS, loaded NSETS - 1 steps ahead
    u32x4 xg[2][XJ];              // X(stage) lives in set stage % 2: loaded 2 stages ahead, stored to LDS 1 stage ahead
    bf16x8 xf[NTT];

    // Weight steps and token stages are loaded strictly in ring order, so one running position each replaces a
    // modulo per load: kw = k32 step of the next weight load, kx = k64 stage of the next token load.
    int kw = 2 * st0, kx = st0;
#ifdef MOE_NT_WEIGHTS
#define MOE_WLD(p) __builtin_nontemporal_load(p)
#else
#define MOE_WLD(p) (*(p))
#endif
#define WLOAD(set, s)                                                                            \
    do {                                                                                         \
        const size_t ko_ = (size_t)kw * 1024;                                                    \
        kw = kw + 1 == nk ? 0 : kw + 1;                                                          \
        _Pragma("unroll") for (int f = 0; f < HF; ++f) {                                         \
            wr[set][f] = MOE_WLD(reinterpret_cast<const u32x4 *>(wp0 + (f * rb_stride * 2 + ko_) + wlane)); \
            if (MODE == 0) wr[set][f + HF] = MOE_WLD(reinterpret_cast<const u32x4 *>(wp1 + (f * rb_stride * 2 + ko_) + wlane)); \
        }                                                                                        \
    } while (0)
#define XLOAD(set, st)                                                                           \
    do {                                                                                         \
        const size_t ko_ = (size_t)kx * 128;                                                     \
        kx = kx + 1 == nst ? 0 : kx + 1;                                                         \
        _Pragma("unroll") for (int j = 0; j < XJ; ++j)                                           \
            xg[set][j] = *reinterpret_cast<const u32x4 *>(xbase + ko_ + xo[j]);                  \
    } while (0)
#define XSTORE(buf)                                                                              \
    do {                                                                                         \
        _Pragma("unroll") for (int j = 0; j < XJ; ++j)                                           \
            *reinterpret_cast<u32x4 *>(xw + (buf) * (2 * HALF) + j * (RPP * 32)) = xg[buf][j]; \
    } while (0)
#define XREAD(buf, half)                                                                         \
    do {                                                                                         \
        _Pragma("unroll") for (int t = 0; t < NTT; ++t)                                          \
            xf[t] = as_frag(*reinterpret_cast<const u32x4 *>(((half) ? xrd1 : xrd0) + (buf) * (2 * HALF) + t * (16 * 32))); \
    } while (0)
    /* token subtile outermost: the first NF MFMAs need only the first LDS read, so the later reads land behind them */ \
#define MFMAS(set)                                                                               \
    do {                                                                                         \
        _Pragma("unroll") for (int t = 0; t < NTT; ++t)                                          \
            _Pragma("unroll") for (int f = 0; f < NF; ++f)                                       \
                acc[f][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_frag(wr[set][f]), xf[t], acc[f][t], 0, 0, 0); \
    } while (0)
    // FENCED: the compiler may not move the loads and LDS reads of a stage across its MFMA groups (measured: the wide
    // down-projection tile over a long K runs 4-6 % faster that way, short-K launches 4-8 % slower)
#define FENCE()                                                                                  \
    do {                                                                                         \
        if (FENCED) __builtin_amdgcn_sched_barrier(0);                                           \
    } while (0)
    // ... and the widest up-projection tile 3-6 % faster with the one fence between the first MFMA group of a stage and
    // the loads that follow it (compared inside one run on four layer shapes)
#define FENCE_MID()                                                                              \
    do {                                                                                         \
        if (FENCED || (MODE == 0 && NF == 4)) __builtin_amdgcn_sched_barrier(0);                 \
    } while (0)
    // Issue order asked of the scheduler for the full-size up-projection body (8 LDS fragment reads, 32 MFMAs and 6 or 4
    // global loads per half stage): two fragment reads ahead, then one read and one load after every 4 MFMAs.  Measured
    // inside one run: 5 % faster at 8192 tokens, where most tiles are full, the same at 2048.
#define SGB(mask, n) __builtin_amdgcn_sched_group_barrier(mask, n, 0)     /* 0x008 MFMA, 0x020 global load, 0x100 LDS read */
#define PIPE_HALF(n_loads)                                                                       \
    do {                                                                                         \
        if (MODE == 0 && NF == 4 && NTT == 8) {                                                  \
            SGB(0x100, 2);                                                                       \
            _Pragma("unroll") for (int i_ = 0; i_ < 6; ++i_) {                                   \
                SGB(0x008, 4);                                                                   \
                SGB(0x100, 1);                                                                   \
                if (i_ < (n_loads)) SGB(0x020, 1);                                               \
            }                                                                                    \
            SGB(0x008, 8);                                                                       \
        }                                                                                        \
    } while (0)
#define PIPE_FIRST() PIPE_HALF(6)       /* token loads of the stage + the weights of one step */
#define PIPE_SECOND() PIPE_HALF(4)
    // one stage: k32 steps in weight sets ws_ and ws_ + 1; its token rows are in LDS buffer buf
#define STAGE(buf, ws_)                                                                          \
    do {                                                                                         \
        __builtin_amdgcn_s_waitcnt(0xC07F);      /* lgkmcnt(0): this thread's LDS writes of the stage have landed */ \
        __builtin_amdgcn_s_barrier();                                                            \
        FENCE();                                                                                 \
        XLOAD(buf, 0);                            /* two stages ahead; its register set is in LDS now */          \
        WLOAD(((ws_) + NSETS - 1) % NSETS, 0);                                                   \
        XREAD(buf, 0);                                                                           \
        FENCE();                                                                                 \
        MFMAS(ws_);                                                                              \
        PIPE_FIRST();                                                                            \
        FENCE_MID();                                                                             \
        WLOAD(ws_, 0);                            /* = set (ws_ + NSETS) % NSETS */              \
        XREAD(buf, 1);                                                                           \
        FENCE();                                                                                 \
        MFMAS(((ws_) + 1) % NSETS);                                                              \
        PIPE_SECOND();                                                                           \
        XSTORE((buf) ^ 1);                        /* the next stage -> the other LDS buffer */   \
    } while (0)

    XLOAD(0, 0);
    XLOAD(1, 1);
#pragma unroll
    for (int u = 0; u < NSETS - 1; ++u) WLOAD(u, u);
    XSTORE(0);
    // a round of NSETS steps (NSETS / 2 stages, an even number, so the LDS buffer of a stage is a constant too)
    for (int s = 0; s < nk; s += NSETS) {
#pragma unroll
        for (int u = 0; u < NSETS; u += 2) STAGE((u >> 1) & 1, u);
    }
#undef STAGE
#undef PIPE_SECOND
#undef PIPE_FIRST
#undef PIPE_HALF
#undef SGB
#undef FENCE_MID
#undef FENCE
#undef MFMAS
#undef XREAD
#undef XSTORE
#undef XLOAD
#undef WLOAD
#undef MOE_WLD

    ahead_of_stores();
    // ---- epilogue: in every 16x16 tile a lane holds weight rows 4*lg + 0..3 (= output columns) of token li
    const int colw = n0 + wave * WAVE_COLS;
    if (colw >= NOUT) return;                               // wave past the ragged edge: its columns were recomputed only
    if (MODE == 1 && nsp > 1) {
        // one of nsp partial sums over K: fp32, summed in split order by the finishing pass; four lanes to the 64 bytes of a row, as
        // below, chunk c of row i in slot c ^ (i >> 2 & 3)
        const int pr = lane >> 2, pc = lane & 3;
#pragma unroll
        for (int t = 0; t < NTT; ++t) {
#pragma unroll
            for (int f = 0; f < HF; ++f) {
                char *b = ys + (f & 1) * 1024;
                *reinterpret_cast<f32x4 *>(b + li * 64 + (lg ^ (li >> 2 & 3)) * 16) = acc[f][t];
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                const f32x4 v = *reinterpret_cast<const f32x4 *>(b + pr * 64 + (pc ^ (pr >> 2 & 3)) * 16);
                if (t * 16 + pr < nrows) *reinterpret_cast<f32x4 *>(part + ((size_t)sp * R + row0 + t * 16 + pr) * NOUT + colw + f * 16 + pc * 4) = v;
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            }
        }
        return;
    }
    // The results leave through LDS (up to 2 KB of the wave's own), so that the lanes of a store cover whole runs of a row: stored from the
    // accumulators, neighbouring lanes in different rows, each of the 64 lanes is an access of its own, and the next block waits
    // for all of them (12089 rows of 64 experts, d = 2048, I = 768: up 119 us level, down 87 -> 77; 12047 rows of 32, I = 1408:
    // down 95 -> 92; the whole layer's pass 6 and 4.5 % faster).  Chunk c (16 bytes) of row i sits in slot c ^ (i & (C - 1)).
    constexpr int C = WAVE_COLS / 8;                       // 16-byte chunks of a row
    constexpr int TS = NTT < 8 / C ? NTT : C == 2 ? 2 : 1; // subtiles per store: all 64 lanes, where there are that many rows
    const int yr = lane / C, yc = lane % C;
#pragma unroll
    for (int t0 = 0; t0 < NTT; t0 += TS) {
#pragma unroll
        for (int t = t0; t < t0 + TS && t < NTT; ++t) {
#pragma unroll
            for (int f = 0; f < HF; ++f) {
                u32x2 o;
                if (MODE == 0) {
                    o.x = pack_bf16x2(silu_mul(acc[f][t][0], acc[f + HF][t][0]), silu_mul(acc[f][t][1], acc[f + HF][t][1]));
                    o.y = pack_bf16x2(silu_mul(acc[f][t][2], acc[f + HF][t][2]), silu_mul(acc[f][t][3], acc[f + HF][t][3]));
                } else {
                    o.x = pack_bf16x2(acc[f][t][0], acc[f][t][1]);
                    o.y = pack_bf16x2(acc[f][t][2], acc[f][t][3]);
                }
                *reinterpret_cast<u32x2 *>(ys + ((t - t0) * 16 + li) * (C * 16) + (((f * 2 + (lg >> 1)) ^ (li & (C - 1))) * 16) + (lg & 1) * 8) = o;
            }
        }
        // the lanes of a wave exchange data: LDS serves a wave's accesses in order, the compiler keeps theirs
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int q = 0; q < TS * 16; q += 64 / C) {
            const int i = q + yr;                          // row of the TS subtiles
            if (i < TS * 16) {
                const u32x4 v = *reinterpret_cast<const u32x4 *>(ys + i * (C * 16) + ((yc ^ (i & (C - 1))) * 16));
                if (t0 * 16 + i < nrows) {
                    u32x4 *const q = reinterpret_cast<u32x4 *>(out + (size_t)(row0 + t0 * 16 + i) * NOUT + colw + yc * 8);
                    if (THROUGH)      // sc1: past the caches of this XCD
                        __builtin_amdgcn_raw_buffer_store_b128(v, __builtin_amdgcn_make_buffer_rsrc(out + (size_t)row0 * NOUT, 0, nrows * NOUT * 2, 0x00027000),
                                                               ((t0 * 16 + i) * NOUT + colw + yc * 8) * 2, 0, 0x10);
                    else
                        *q = v;
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
}

// Item of a block of a launch that can cut.  Every XCD takes a contiguous run of the item list on its 32 compute units.  Where the
// last round of the launch would occupy half of the units or less, its items run as two of half the width each (0.5 to 0.6 of
// the time, measured): the round ends after as much of an item instead of a whole one; with more the halves would not fit one round.
// Up, d = 2048, I = 768, whole / cut: 522 items of 256 inner columns 195 / 176 us, 636 198 / 185, 783 237 / 220, 1035 298 / 282.
// Down, same layer: 40 items of 512 columns 28 / 21 us, 124 32 / 28, 260 69 / 62, 376 73 / 72, 528 86 / 79, 800 118 / 111, launches that
// are not cut 0 to 1 % slower.  An exact half of a round, up, I = 2048: 640 items 230 / 226 us with one row to a tile, 270 / 259 with 128;
// down, 384 items, all of them as halves / the last ones: 17 rows 62 / 62, 128 rows 83 / 80.
// Returns the item, or -1 for a block without one; half is 0 or 1, or -1 for a whole item.
#define XCD_CUS 32
// Not cut: the narrowest tiles, and tiles of 512 columns over a K of 8192 and more (FENCED).
constexpr bool tiled_can_cut(int mode, int nf, bool fenced, int waves) { return waves == 8 && nf > 1 && (mode == 0 || !fenced); }
__device__ __forceinline__ int cut_item_of(int total, int pid, int &half)
{
    const int q = total / MOE_NUM_XCD, rem = total % MOE_NUM_XCD;
    const int xcd = pid % MOE_NUM_XCD, loc = pid / MOE_NUM_XCD;
    const int n = q + (xcd < rem ? 1 : 0), first = xcd * q + min(xcd, rem);
    const int over = total % (MOE_NUM_XCD * XCD_CUS), half_round = MOE_NUM_XCD * XCD_CUS / 2;
    const int cut = over <= half_round ? n % XCD_CUS : 0, whole = n - cut;
    half = -1;
    if (loc < whole) return first + loc;
    const int j = loc - whole;
    if (j >= 2 * cut) return -1;
    half = j & 1;
    return first + whole + (j >> 1);
}

// Whether the up projection, whose whole items would be one round and up to half of another, runs all of them as halves (n_half
// to a token tile): two to three rounds.
// Two, where the last column tile is ragged and a half by itself: a cut list leaves its units idle after half of a round, and the
// halves of the last items wait for others (d = 2048, I = 1408, 258 items = 473 halves, cut / halves: 1 row to a tile 105 / 87 us, 16
// 106 / 86, 60 112 / 91, 128 127 / 101; 276 = 506: 107 / 90 to 130 / 105; with a third round, 294 = 539: 109 / 110 to 131 / 135; three column
// tiles, I = 640, tables of routed rows: 73 to 89 / 72 to 80, d = 1152 44 to 55 / 46 to 48).
// Three, where no tile is ragged and the tiles are short, so that a half takes half the time (d = 2048, I = 768 and 2048, 260 to 380
// items: 1 to 32 rows to a tile 1 to 3 % faster, 40 rows 0 to 2 % slower, 128 rows 1 to 4 %); with ragged ones only where the third
// round is more than half full (I = 1408, 1 to 16 rows: 294 to 342 items 0 to 1 % slower, 372 2 % faster, 384 3 %).
#define HALVES_ITEMS 384
#define HALVES_SHORT_ROWS 32
__device__ __forceinline__ bool up_runs_halves(int tiles, int n_ntc, int n_half, const moe_rows &r)
{
    const int items = tiles * n_ntc, halves = tiles * n_half;
    if (items <= 256 || items > HALVES_ITEMS) return false;
    if (halves <= 512) return true;
    return (halves == 2 * items || halves > 640) && wave_sum_int_dpp(r.c0 + r.c1) <= HALVES_SHORT_ROWS * tiles;
}

// Whether the up projection runs every expert's rows, 256 at most, as one tile of half the width (asked in launches of up to 256 rows per
// expert in the mean, masked-off ones counted, where an expert may be within that, and of a hidden size of 2048 or more): an expert has more
// than 128, such items fill one round of the compute units, three quarters of it or more, and the whole items would not all be cut.  A
// few last rows as a tile of their own take the whole time of its weights, and two tiles ask for them twice; but an item is 128 rows x
// 256 columns of LDS traffic more for half the products.  d = 4096, I = 14336, whole pass of 200 tokens, two experts of 139 and 95 rows (168
// items -> 224) 215 -> 192 us.  The launch alone, from cold caches, 2 to 100 experts of 14336 to 256 in seven mixtures of heights: over 129 to
// 240 whole items 1.03 times as fast in the mean at d = 2048 (0.93 to 1.16), 1.04 at 4096, 1.08 at 7168 (20 of 139 and 95 rows, I = 1408, 251 / 215,
// two of 256, I = 14336, d = 4096 164 / 155).  Lines: up to 128 whole items, which run as halves anyway, 0.97, 0.96 and 0.94 (129 rows and 15 times 40,
// I = 1536, d = 4096, 130 / 140); d = 1024 1.01, 0.92 to 1.07; fewer such items: one expert of 250 (112) 105 / 129, 20 of 200, I = 768 (120) 59 / 69.
#define TALL_MIN_ITEMS 192
#define TALL_MIN_D 2048
__device__ __forceinline__ bool up_runs_tall(const moe_rows &r, int whole, int n_half, int &experts)
{
    const int most = wave_max_int_dpp(max(r.c0, r.c1));
    experts = __popcll(__ballot(r.c0 > 0)) + __popcll(__ballot(r.c1 > 0));
    const int items = experts * n_half;
    return most > TM && most <= 2 * TM && items >= TALL_MIN_ITEMS && items <= MOE_NUM_XCD * XCD_CUS && whole > MOE_NUM_XCD * XCD_CUS / 2;
}

// NTT_MAX bounds the token subtiles a tile of this launch can need (from T); the block then runs the smallest
// body that covers its own rows, so a sparsely filled tile costs MFMA work for the rows it has.
template <int MODE, int NF, int NTT_MAX, bool DIRECT, int NSETS, bool FENCED, int WAVES, bool CAN_TALL>
__global__ __launch_bounds__(WAVES * 64, 2) void ffn_tiled_kernel(
    int d, int I, int k, int N, const uint16_t *__restrict__ xsrc,   // MODE 0: h [T,d]; MODE 1: act [R,I]
    const int32_t *__restrict__ perm, const int32_t *__restrict__ offsets, const int32_t *__restrict__ counts,
    const uint16_t *__restrict__ wa, const uint16_t *__restrict__ wb,   // MODE 0: packed w1, w3; MODE 1: packed w2, unused
    const uint8_t *__restrict__ mask,
    uint16_t *__restrict__ out,                                            // MODE 0: act [R,I]; MODE 1: y [R,d]
    int nsp_max, float *__restrict__ part, int R,   // MODE 1: up to nsp_max K splits per tile, partial sums in part [nsp,R,d] fp32
    int32_t *__restrict__ rival,                    // MODE 1, non-null: the long-K kernel follows; whether it is the one that works (wide_faster)
    int group)                                      // column tiles that alternate inside the item order of an expert (1: column tile major)
{
    // CAN_TALL: a launch that can run tiles of up to 256 rows at half width (up_runs_tall)
    __shared__ __attribute__((aligned(16))) uint16_t Xs[2][2][(CAN_TALL ? 2 : 1) * TM * 32];   // [buffer][k32 half][tokens x 32 k]
    __shared__ __attribute__((aligned(16))) char Ys[WAVES][2048];          // results on their way out
    // a launch that can run an item as two of half its width (cut_item_of)
    constexpr bool CAN_CUT = tiled_can_cut(MODE, NF, FENCED, WAVES);
    constexpr int NT_COLS = WAVES * 16 * (MODE == 0 ? NF / 2 : NF);
    const int n_ntc = ((MODE == 0 ? I : d) + NT_COLS - 1) / NT_COLS;   // column tiles
    const int n_half = ((MODE == 0 ? I : d) + NT_COLS / 2 - 1) / (NT_COLS / 2);
    int half = -1;
    bool halves = false;               // every item runs at half width

    // ---- which item: (expert, token tile, column tile, K split).  The number of K splits follows from the number of
    // tiles that have work, which only the device knows (counts and mask live there)
    MOE_TRACE_BEGIN();
    int e, mt, nt, nsp = 1, tmk = TM;      // tmk: token rows per tile of this launch
    int row0, nrows;
    if (DIRECT) {
        // at most one token tile per expert (T <= 128)
        const moe_work work = moe_working_experts(N, counts, offsets, mask);
        const int n_work = work.experts();
        if (MODE == 1) nsp = moe_dev_splits(n_work * n_ntc, nsp_max);
        halves = MODE == 0 && CAN_CUT && up_runs_halves(n_work, n_ntc, n_half, work.rows());
        if (halves) {
            if (!moe_item_of(work, n_half, blockIdx.x, e, nt)) return;
        } else if (CAN_CUT && nsp == 1) {
            const int L = cut_item_of(n_work * n_ntc, blockIdx.x, half);
            if (L < 0) return;
            moe_item_at(work, n_ntc, L, e, nt);
        } else if (!moe_item_of(work, n_ntc * nsp, blockIdx.x, e, nt)) {
            return;
        }
        mt = 0;
        row0 = work.first_row_of(e);
        nrows = work.rows_of(e);
    } else {
        const moe_rows rows = moe_masked_rows(N, counts, mask);
        const moe_tiles tiles = MODE == 0 ? tiles_128(rows) : down_tiles(rows, n_ntc, tmk);
        if constexpr (CAN_TALL) {
            int experts;
            if (up_runs_tall(rows, tiles.total * n_ntc, n_half, experts)) {
                const int items = experts * n_half;
                if ((int)blockIdx.x >= items) return;
                const int L = moe_xcd_run(items, blockIdx.x);
                int first, n;
                moe_find_tile(moe_rank_tiles(rows.c0 > 0, rows.c1 > 0), L / n_half, e, first, n);
                nt = L % n_half;
                row0 = offsets[e];
                nrows = counts[e];
#define TALL_BODY(n_) tile_body<MODE, NF / 2, n_, NSETS, FENCED, WAVES>(&Xs[0][0][0], Ys[__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)], d, I, k, xsrc, perm, wa, wb, out, e, nt, row0, nrows, 0, 1, part, R, threadIdx.x)
                if (nrows <= 32) TALL_BODY(2);
                else if (nrows <= 64) TALL_BODY(4);
                else if (nrows <= 96) TALL_BODY(6);
                else if (nrows <= 128) TALL_BODY(8);
                else if (nrows <= 160) TALL_BODY(10);
                else if (nrows <= 192) TALL_BODY(12);
                else TALL_BODY(16);
#undef TALL_BODY
                MOE_TRACE_END(MODE, e, nrows, nt);
                return;
            }
        }
        if (MODE == 1) nsp = moe_dev_splits(tiles.total * n_ntc, nsp_max);
        if (MODE == 1 && rival != nullptr) {
            const bool wide = wide_faster(wide_plan_of(rows, (d + WIDE_TN - 1) / WIDE_TN, I / 32), I / 32, tiles.total * n_ntc, tmk, NT_COLS);
            if (blockIdx.x == 0 && threadIdx.x == 0) *rival = wide;
            if (wide) return;
        }
        halves = MODE == 0 && CAN_CUT && up_runs_halves(tiles.total, n_ntc, n_half, rows);
        const int n_nt = halves ? n_half : n_ntc * nsp;
        const int total = tiles.total * n_nt;
        int L;
        if (CAN_CUT && nsp == 1 && !halves) {
            L = cut_item_of(total, blockIdx.x, half);
            if (L < 0) return;
        } else {
            if ((int)blockIdx.x >= total) return;
            L = moe_xcd_run(total, blockIdx.x);
        }
        int first, n;
        moe_find_tile(tiles, L / n_nt, e, first, n);
        const int local = L - first * n_nt;
        // Item order inside an expert: groups of `group` column tiles; inside a group the token tiles in turn, each with
        // the group's column tiles side by side.  Blocks that follow each other in the list start close in time, so the
        // blocks that share a token tile (same mt) and those that share a weight tile (same nt) both stay near each other.
        const int per_group = group * n;
        const int g0 = local / per_group, within = local - g0 * per_group;
        const int gsz = min(group, n_nt - g0 * group);         // the last group may hold fewer column tiles
        mt = within / gsz;
        nt = g0 * group + within % gsz;
        row0 = offsets[e] + mt * tmk;
        nrows = counts[e] - mt * tmk;
    }
    if (halves) {
        half = nt & 1;
        nt >>= 1;
    }
    const int sp = nt % nsp;      // column tile nt / nsp, K split nt % nsp
    nt /= nsp;
    nrows = nrows > tmk ? tmk : nrows;
#define BODY_NS(nf_, n, ns_) tile_body<MODE, nf_, n, ns_, FENCED, WAVES>(&Xs[0][0][0], Ys[__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)], d, I, k, xsrc, perm, wa, wb, out, e, nt, row0, nrows, sp, nsp, part, R, threadIdx.x)
#define BODY_NF(nf_, n) BODY_NS(nf_, n, NSETS)
    // tiles with few token rows do little arithmetic per weight byte: their speed is the speed of the weight stream, so
    // they prefetch further ahead (8 register sets instead of 4; the accumulators of a short tile leave the room)
#ifdef MOE_DEEP_SMALL
    const bool deep_ok = NSETS == 4 && WAVES == 8 && (((MODE == 0 ? d : I) / 32 / nsp) % 8) == 0;
#else
    const bool deep_ok = false;
#endif
#define BODY_SMALL(nf_, n)                                         \
    do {                                                           \
        if (deep_ok) BODY_NS(nf_, n, 8);                           \
        else BODY_NF(nf_, n);                                      \
    } while (0)
#define BODIES(nf_)                                                \
    do {                                                           \
        if (NTT_MAX == 1 || nrows <= 16) BODY_SMALL(nf_, 1);       \
        else if (NTT_MAX == 2 || nrows <= 32) BODY_SMALL(nf_, 2);  \
        else if (NTT_MAX == 4 || nrows <= 64) BODY_SMALL(nf_, 4);  \
        else if (nrows <= 96) BODY_NF(nf_, 6);                     \
        else if (MODE == 1 && nrows <= 112) BODY_NF(nf_, 7);       \
        else BODY_NF(nf_, 8);                                      \
    } while (0)
    if constexpr (CAN_CUT) {
        // a ragged last column tile that fits a half-width item has no second half; that of the up projection always runs as a
        // half-width item (I = 1408: five items of 256 + one of 128)
        if (nt == n_ntc - 1 && n_half < 2 * n_ntc) {
            if (half == 1) return;
            if (MODE == 0) half = 0;
        }
        if (__builtin_expect(half < 0, 1)) {
            BODIES(NF);
            MOE_TRACE_END(MODE, e, nrows, nt);
            return;
        }
        nt = 2 * nt + half;
        BODIES(NF / 2);
        MOE_TRACE_END(MODE, e, nrows, nt);
        return;
    }
    BODIES(NF);
    MOE_TRACE_END(MODE, e, nrows, nt);
#undef BODIES
#undef BODY_SMALL
#undef BODY_NF
#undef BODY_NS
}

// four columns of a row, the partial sums of all S splits on their way at once
template <int S>
__device__ __forceinline__ void add_splits(const float *__restrict__ partial, size_t p, int R, int d, int f, uint16_t *__restrict__ y)
{
    f32x4 v[S];
#pragma unroll
    for (int ks = 0; ks < S; ++ks) v[ks] = *reinterpret_cast<const f32x4 *>(partial + ((size_t)ks * R + p) * d + f);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 1; ks < S; ++ks) v[0] += v[ks];
    *reinterpret_cast<u32x2 *>(y + p * d + f) = u32x2{pack_bf16x2(v[0][0], v[0][1]), pack_bf16x2(v[0][2], v[0][3])};
}

// y[p,:] = bf16( sum over the K splits, in split order ), when the down projection of this launch split K (the same
// device-side decision as in ffn_tiled_kernel; nothing to do otherwise: the tiles wrote y themselves)
__global__ __launch_bounds__(256) void tiled_finish_kernel(int d, int R, int N, int n_ntc, int nsp_max, int direct,
                                                           const float *__restrict__ partial,
                                                           const int32_t *__restrict__ offsets, const int32_t *__restrict__ counts,
                                                           const uint8_t *__restrict__ mask, uint16_t *__restrict__ y)
{
    // Blocks walk the rows of their expert: with one for every token and expert, most had no row (3000 tokens, 16 experts: ranking
    // the tiles in all 48000 of them took 25 of 99 us), and where the launch did not split all of them ranked for nothing.
    const int e = blockIdx.y, c = counts[e];
    if ((int)blockIdx.x >= c || (mask != nullptr && mask[e] == 0)) return;
    int tiles;
    if (direct) {
        tiles = moe_working_experts(N, counts, offsets, mask).experts();
    } else {
        int tm;
        tiles = down_tiles(moe_masked_rows(N, counts, mask), n_ntc, tm).total;
    }
    const int nsp = moe_dev_splits(tiles * n_ntc, nsp_max);
    if (nsp == 1) return;
    const int f = (blockIdx.z * 256 + threadIdx.x) * 4;
    if (f >= d) return;
    const size_t row0 = offsets[e];
    for (int j = blockIdx.x; j < c; j += gridDim.x) {
        if (nsp == 2) add_splits<2>(partial, row0 + j, R, d, f, y);
        else if (nsp == 4) add_splits<4>(partial, row0 + j, R, d, f, y);
        else add_splits<8>(partial, row0 + j, R, d, f, y);
    }
}

#include "ffn_joint.h"

// measurement switch: how many column tiles alternate in the item order (see the kernel); 1 = column tile major
static int tiled_item_group(int mode)
{
    static const int up = getenv("MOE_TILED_GROUP_UP") ? atoi(getenv("MOE_TILED_GROUP_UP")) : 1;
    static const int dn = getenv("MOE_TILED_GROUP_DOWN") ? atoi(getenv("MOE_TILED_GROUP_DOWN")) : 1;
    const int g = mode == 0 ? up : dn;
    return g < 1 ? 1 : g;
}

template <int MODE, int NF, int NTT, bool DIRECT, int NSETS, bool FENCED, int WAVES>
static void launch_tiled(const moe_shape *s, long max_mt, const uint16_t *x, const int32_t *perm, const int32_t *offsets,
                         const int32_t *counts, const uint16_t *wa, const uint16_t *wb,
                         const uint8_t *mask, uint16_t *out, int nsp_max, float *part, int32_t *rival, hipStream_t st)
{
    constexpr int cols = WAVES * 16 * (MODE == 0 ? NF / 2 : NF);
    const long n_ntc = ((MODE == 0 ? s->I : s->d) + cols - 1) / cols;
    const int R = s->T * s->k;
    // blocks for the most items the device-side choice of K splits can produce: with every tile at work it takes the
    // fewest splits that reach 256 items, with fewer tiles at work there are fewer items, so this bound covers both
    const long n_e = s->N < (long)s->T * s->k ? s->N : (long)s->T * s->k;   // DIRECT: experts that can be non-empty
    const long tiles = DIRECT ? n_e : max_mt;
    long blocks = tiles * n_ntc * nsp_max;
    if (tiled_can_cut(MODE, NF, FENCED, WAVES)) {
        // and the items that run as two: those of a last round (cut_item_of), or all of them (up_runs_halves)
        const long halves = 2 * (blocks < HALVES_ITEMS ? blocks : HALVES_ITEMS);
        blocks += MOE_NUM_XCD * (XCD_CUS / 2);
        if (blocks < halves) blocks = halves;
    }
    const dim3 grid((unsigned)blocks);
#define LAUNCH(tall_) \
    hipLaunchKernelGGL((ffn_tiled_kernel<MODE, NF, NTT, DIRECT, NSETS, FENCED, WAVES, tall_>), grid, dim3(WAVES * 64), 0, st, s->d, s->I, s->k, \
                       s->N, x, perm, offsets, counts, wa, wb, mask, out, nsp_max, part, R, rival, tiled_item_group(MODE))
    if constexpr (MODE == 0 && !DIRECT && WAVES == 8) {
        // an instance of its own: with the tall bodies beside the others, 8192 tokens through 8 experts of I = 14336 took 1.4 % longer
        if (R <= 2 * TM * s->N && s->d >= TALL_MIN_D) {
            LAUNCH(true);
            return;
        }
    }
    LAUNCH(false);
#undef LAUNCH
}

// Weight fragments per wave (NF), 16-row token subtiles per tile (NTT) and weight register sets (NSETS).  An expert
// never receives more rows than there are tokens, so T bounds the subtiles in use, and up to 128 tokens every expert
// has at most one token tile, which needs no schedule; narrow weight tiles keep every compute unit busy when there
// are few token tiles, and since a narrow tile leaves a wave only NF KB per step to ask for, it prefetches further
// ahead (8 register sets, K permitting; 16 measured no better: the token loads, two stages ahead, sit between the
// weight loads in the in-order vmcnt queue and bound the useful depth).
template <int MODE>
static void dispatch_tiled(const moe_shape *s, int nf, int waves, long max_mt, const uint16_t *x, const int32_t *perm,
                           const int32_t *offsets, const int32_t *counts, const uint16_t *wa, const uint16_t *wb,
                           const uint8_t *mask, uint16_t *out, int nsp_max, float *part, int32_t *rival, hipStream_t st)
{
    const int K = MODE == 0 ? s->d : s->I;
    const bool deep = K % (256 * nsp_max) == 0 && K >= 2048;   // a short K does not pay for the longer prologue
#define GO(NF_, NTT_, D_, NS_, F_) launch_tiled<MODE, NF_, NTT_, D_, NS_, F_, 8>(s, max_mt, x, perm, offsets, counts, wa, wb, mask, out, nsp_max, part, rival, st)
    if (waves == 4) {
        // two independent 4-wave blocks per compute unit (scheduled launches with full-height tiles only)
        launch_tiled<MODE, 4, 8, false, 4, false, 4>(s, max_mt, x, perm, offsets, counts, wa, wb, mask, out, nsp_max, part, rival, st);
        return;
    }
#define GO3(NTT_, D_)                                                          \
    do {                                                                       \
        if constexpr (MODE == 1) {                                             \
            if (nf == 1) {                                                     \
                if (deep) GO(1, NTT_, D_, 8, false);                                  \
                else GO(1, NTT_, D_, 4, false);                                       \
                break;                                                         \
            }                                                                  \
            if (nf == 2) {                                                     \
                if (deep) GO(2, NTT_, D_, 8, false);                                  \
                else GO(2, NTT_, D_, 4, false);                                       \
                break;                                                         \
            }                                                                  \
        }                                                                      \
        if constexpr (MODE == 1 && !D_) {                                      \
            if (K >= 8192) {                                                   \
                GO(4, NTT_, D_, 4, true);                                      \
                break;                                                         \
            }                                                                  \
        }                                                                      \
        GO(4, NTT_, D_, 4, false);                                             \
    } while (0)
    if (s->T <= 16) GO3(1, true);
    else if (s->T <= 32) GO3(2, true);
    else if (s->T <= 64) GO3(4, true);
    else if (s->T <= TM) GO3(8, true);
    else GO3(8, false);
#undef GO3
#undef GO
}

int moe_ffn_tiled_impl(const moe_shape *s, const void *h, const int32_t *perm, const int32_t *offsets,
                       const int32_t *counts, const void *w1, const void *w3, const void *w2,
                       const uint8_t *expert_mask, void *y, void *workspace, int stages, hipStream_t st)
{
    const int d = s->d, I = s->I, N = s->N, k = s->k;
    const long R = (long)s->T * k;
    moe_ws_layout L = moe_ws(s);
    uint16_t *act = (uint16_t *)((char *)workspace + L.act);
    const long max_mt = R / TM + (N < R ? N : R), max_mt_down = R / MOE_TILE_M_MIN + (N < R ? N : R);
    // token tiles to expect: every expert that can be non-empty has one, large experts have several
    const long est_mt = (R + TM - 1) / TM > (N < R ? N : R) ? (R + TM - 1) / TM : (N < R ? N : R);

    // the down projection's tile shape
    int nf = s->T <= MOE_SKINNY_MAX_T ? 1
             : est_mt * ((d + 511) / 512) >= 256 ? 4 : est_mt * ((d + 255) / 256) >= 256 ? 2 : 1;
    // blocks of 4 waves, two of them per compute unit, for scheduled launches (experiment switch)
    static const int env_up = getenv("MOE_TILED_WAVES_UP") ? atoi(getenv("MOE_TILED_WAVES_UP")) : 0;
    static const int env_dn = getenv("MOE_TILED_WAVES_DOWN") ? atoi(getenv("MOE_TILED_WAVES_DOWN")) : 0;
    const int waves_up = s->T > TM && env_up == 4 ? 4 : 8;
    const int waves_down = s->T > TM && env_dn == 4 && nf == 4 ? 4 : 8;
    int32_t *const wide = moe_wide_down(s) ? (int32_t *)((char *)workspace + L.choice) : nullptr;
    if (stages & MOE_FFN_STAGE_UP) {
        dispatch_tiled<0>(s, 4, waves_up, max_mt, (const uint16_t *)h, perm, offsets, counts, (const uint16_t *)w1,
                          (const uint16_t *)w3, expert_mask, act, 1, nullptr, nullptr, st);
        MOE_CHECK_LAUNCH();
    }
    if (stages & MOE_FFN_STAGE_DOWN) {
        // nf: the widest weight tile that still leaves every compute unit a block (512 columns, then 256 columns), else
        // the narrowest (128 columns); and when even that leaves compute units idle -- few experts with rows, or few of
        // them masked on -- the K range of every tile is split over up to nsp_max items (decided on the device, which
        // knows counts and mask)
        const int nsp_max = moe_tiled_down_max_splits(s);
        float *part = (float *)((char *)workspace + L.partial);
        dispatch_tiled<1>(s, nf, waves_down, max_mt_down, (const uint16_t *)act, perm, offsets, counts, (const uint16_t *)w2,
                          (const uint16_t *)nullptr, expert_mask, (uint16_t *)y, nsp_max, part, wide, st);
        MOE_CHECK_LAUNCH();
        const int cols = 16 * waves_down * nf;      // of an item
        if (nsp_max > 1) {
            const int slices = (d + 1023) / 1024, blocks = 2048 / (N * slices);
            const int max_rows = s->T < (blocks > 64 ? blocks : 64) ? s->T : blocks > 64 ? blocks : 64;
            hipLaunchKernelGGL(tiled_finish_kernel, dim3(max_rows, N, slices), dim3(256), 0, st, d, (int)R, N, (d + cols - 1) / cols, nsp_max,
                               s->T <= TM ? 1 : 0, part, offsets, counts, expert_mask, (uint16_t *)y);
            MOE_CHECK_LAUNCH();
        }
        if (wide != nullptr) return moe_ffn_wide_down(s, offsets, counts, act, w2, y, expert_mask, part, wide, st);
    }
    return MOE_OK;
}

// Whether the FFNs of a layer run as a joint launch: the routed K not split (it has no partial sums), inner sizes the long-K kernel does not
// take, and enough items that filled last rounds pay for the clearing launch, the tickets and the activations' way past the caches; an
// up item is never cut there, so with about a round of them or less the separate launches end sooner.  masked: how many experts a mask
// leaves on is known to the device only; the lines are where a quarter of them is about level (30 random shapes within them: a quarter on 0.99 to
// 1.15 times as fast, half 1.00 to 1.23; next to the lines, 64 and 60 experts of 1408, 0.95 to 1.02 and 1.00 to 1.13).  Separate launches / joint in us:
// Routed experts alone, d = 2048, all on / half / a quarter.  64 experts, I = 1408, 512 tokens of 6 slots 227 / 224, 127 / 132, 84 / 91, 1024 256 /
// 244, 157 / 154, 119 / 116, 1400 269 / 262, 184 / 170, 130 / 133, 2048 328 / 299, 230 / 211, 174 / 160; 128 experts, I = 768, 384 tokens of 8 slots 234 / 223, 125 / 122, 70 / 87, 1000
// 251 / 240, 157 / 150, 92 / 96, 1531 282 / 260, 172 / 162, 114 / 107.  Beyond a quarter it loses still: an eighth of these 121 / 130 and 79 / 81.
// Few rows to an expert make short items: 128 of 384 at 8192 rows, 3/4 127 / 120, a quarter 54 / 64, at 12288 74 / 72.
// Other sizes, all on / a quarter, at 9216 to 16384 rows: 64 of 1024, d = 3072 302 / 272 and 141 / 131; 64 of 2048, d = 7168 1338 / 1286 and
// 718 / 633; 64 of 1024, d = 3072, 6144 rows (256 up items) a quarter 115 / 120; 75 of 640 (255) half 116 / 101, a quarter 72 / 77;
// 46 of 256, d = 7168 (110) 3/4 214 / 254, a quarter 161 / 185.
// Few experts: 8 of 4096, d = 4096, 4096 rows 426 / 415 and 155 / 159, 3072 rows (24 tiles) 323 / 370 and 132 / 170; 32 of 768, 4096 rows (96 up
// items) 89 / 93 and 45 / 63; 32 of 1408 with a quarter on, 12288 rows 125 / 137.  d = 1024: 32 of 2816, 8192 rows 203 / 196 and 96 / 115; d = 512:
// 64 of 512, 8192 rows 39 / 44 and 22 / 31.
// Together with shared experts there are four launches to join, on layers of d = 512 to 8192 at 17 to 4096 tokens 1.02 to 1.4 times as fast in
// nearly every call, masked or not; in some of few routed experts and at most 48 tokens not (16 of 3200, d = 4096, and one of 6400, half on, 206 / 210).
// Where the separate shared down projection would split its K, the joint launch ends with its long items: 60 of 1408 and a shared one
// of 5632, d = 2048, all on / half / a quarter: 64 tokens 224 / 191, 150 / 151, 103 / 116, 200 248 / 205, 167 / 153, 122 / 121, 512 267 / 220, 188 / 170,
// 138 / 149 (the one that loses), 1024 316 / 259, 228 / 178, 180 / 156; 10 of 3840 and one of 7680, 64 tokens 157 / 164, 125 / 133, 85 / 90, 512 250 / 222,
// 177 / 185, 138 / 135; d = 1024, 60 of 1408 and one of 5632: 200 tokens 145 / 129, 103 / 114, 80 / 89, 2048 240 / 217, 196 / 179, 162 / 145; d = 512:
// 200 99 / 98, 76 / 95, 66 / 82, 2048 150 / 136, 125 / 115, 112 / 107.
#define JOINT_MIN_ROWS 3072
#define JOINT_MIN_TILES 56
#define JOINT_MIN_UP_ITEMS 256
// under a mask, which leaves some of the experts
#define JOINT_MIN_ROWS_MASKED 6144
#define JOINT_MIN_EXPERT_ROWS_MASKED 72
#define JOINT_MIN_UP_ITEMS_MASKED 288
extern "C" bool moe_ffn_joint_ok(const moe_shape *s, const moe_shape *ss, bool masked)
{
    if (s->I >= 8192 || moe_tiled_down_max_splits(s) != 1) return false;
    if (ss != nullptr) {
        if (ss->I >= 8192 || s->T <= MOE_SKINNY_MAX_T) return false;
        if (moe_tiled_down_max_splits(ss) != 1) return s->T > TM && (s->d >= 2048 || s->T >= 2048);
        return s->T > TM || ss->I <= 2 * s->I;
    }
    const long R = (long)s->T * s->k, tiles = R / TM > s->N ? R / TM : s->N, up = tiles * ((s->I + JOINT_UP_COLS - 1) / JOINT_UP_COLS);
    if (s->d < 2048) return false;
    if (!masked) return R >= JOINT_MIN_ROWS && tiles >= JOINT_MIN_TILES && up >= JOINT_MIN_UP_ITEMS;
    return R >= JOINT_MIN_ROWS_MASKED && R >= JOINT_MIN_EXPERT_ROWS_MASKED * s->N && s->N >= JOINT_MIN_TILES && up >= JOINT_MIN_UP_ITEMS_MASKED;
}

static joint_experts joint_side(const moe_shape *s, const int32_t *perm, const int32_t *offsets, const int32_t *counts, const void *w1,
                                const void *w3, const void *w2, const uint8_t *mask, void *y, void *workspace)
{
    const moe_ws_layout L = moe_ws(s);
    int32_t *const counters = (int32_t *)((char *)workspace + L.partial) + MOE_JOINT_TICKETS;
    return {perm, offsets, counts, (const uint16_t *)w1, (const uint16_t *)w3, (const uint16_t *)w2, mask,
            (uint16_t *)((char *)workspace + L.act), (uint16_t *)y, counters, s->I, s->N, s->k};
}

// polls: the most looks at a counter, see ffn_joint.h (C linkage: with none at all every item takes the way of a wait that ran out)
extern "C" int moe_ffn_joint_impl(const moe_shape *s, const void *h, const int32_t *perm, const int32_t *offsets, const int32_t *counts, const void *w1,
                       const void *w3, const void *w2, const uint8_t *expert_mask, void *y, void *workspace, const moe_shape *ss,
                       const int32_t *s_perm, const int32_t *s_offsets, const int32_t *s_counts, const void *sw1, const void *sw3,
                       const void *sw2, void *shared_y, void *s_workspace, int polls, hipStream_t st)
{
    const auto est_tiles = [](const moe_shape *p) {
        const long R = (long)p->T * p->k, one = p->N < R ? p->N : R;
        return (R + TM - 1) / TM > one ? (R + TM - 1) / TM : one;
    };
    const int d = s->d;
    const joint_experts a = joint_side(s, perm, offsets, counts, w1, w3, w2, expert_mask, y, workspace);
    joint_experts b = {};
    if (ss != nullptr) b = joint_side(ss, s_perm, s_offsets, s_counts, sw1, sw3, sw2, nullptr, shared_y, s_workspace);
    int32_t *const tickets = (int32_t *)((char *)workspace + moe_ws(s).partial);
    const long na = moe_joint_max_tiles(s), nb = ss != nullptr ? moe_joint_max_tiles(ss) : 0, est = est_tiles(s) + (ss != nullptr ? est_tiles(ss) : 0);
    hipLaunchKernelGGL(joint_clear_kernel, dim3(1), dim3(256), 0, st, tickets, a.arrived, (int)na, b.arrived, (int)nb);
    MOE_CHECK_LAUNCH();
    // the widest weight tile of the down projection that leaves every compute unit a block
    const int nf = est * ((d + 511) / 512) >= 256 ? 4 : est * ((d + 255) / 256) >= 256 ? 2 : 1;
    const joint_args args = {{a, b}, (const uint16_t *)h, tickets, d, polls};
    const dim3 grid(MOE_NUM_XCD * JOINT_BLOCKS_PER_XCD);
    if (nf == 4) hipLaunchKernelGGL(ffn_joint_kernel<4>, grid, dim3(TILED_THREADS), 0, st, args);
    else if (nf == 2) hipLaunchKernelGGL(ffn_joint_kernel<2>, grid, dim3(TILED_THREADS), 0, st, args);
    else hipLaunchKernelGGL(ffn_joint_kernel<1>, grid, dim3(TILED_THREADS), 0, st, args);
    MOE_CHECK_LAUNCH();
    return MOE_OK;
}

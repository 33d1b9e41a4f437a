// Down projection of the grouped SwiGLU expert FFN over a long inner size on gfx950:
//   y[p, f] = act[p,:] . W2_e[f,:]        (K = I)
//
// A work item is (expert, 256 activation rows, 256 output columns): with K = 14336 an item runs for hundreds of
// microseconds, so what decides the duration of a launch is how well its items fill the compute units.
//   * The whole rounds of 256 items run as they are; the items of the last, partial round are cut along K into pieces
//     that fill the chip once more (fp32 partial sums, added in piece order by wide_finish_kernel).  Everything follows
//     from counts and mask on the device (wide_plan_of).
//   * 4 waves per block, one per SIMD, 256 accumulator registers per lane: the largest tile the register file holds
//     asks L2 for 32 KB per k32 step and 4.2 MFLOP (a little more than it holds: the epilogue of the 256-row body, with
//     the bf16 and the fp32 stores both live, parks 17 registers per lane in scratch).  A wave owns 64 output columns,
//     i.e. 4 weight fragments per step in the packed order of moe_pack_weights, loaded global -> VGPR seven steps ahead.
//   * Activation rows go straight from global memory to LDS (buffer_load ... lds, no VGPR, no LDS store): four buffers
//     of k64 stages, issued two and a half stages ahead.  The barrier that hands a stage over sits in the middle of the
//     stage before it, so that no wave meets it with an empty MFMA queue.
//   * Row r of a stage is 128 bytes in LDS with its 16-byte chunk c in slot c ^ (r & 7).  One instruction of the loader
//     fills 8 rows in slot order, so the lanes of a row still read one whole 128-byte line; a fragment read (served in
//     four passes of 16 lanes) hits 16 different 16-byte bank groups in every pass.
//   * The loads that run past the end of an item's K range are switched off by a buffer descriptor of zero bytes (no
//     branch, no traffic); all vector loads are bounds-checked by their descriptors.
// Measured (d = 4096, I = 14336, the down projection alone, against the tiles of ffn_tiled.hip): 3822 rows of six experts 617 ->
// 423 us (0.73 -> 1.06 PFLOP/s), 16384 rows of eight 1792 -> 1570 us (1.07 -> 1.23).  It is launched beside the tiled kernel, and
// which of the two works is decided on the device (wide_faster).  What bounds it: the matrix cores at the clock they get under
// load -- with every load a cache hit the same launch takes 338 us, with zeros for operands (no power limit) a fifth less.
#pragma once

#include "moe_common.h"

// Pieces: whole rounds of 256 items run as they are, the `rest` items beyond them are cut into S pieces each.  An item of
// few rows is shorter (measured at K = 14336: 166 us with up to 32 rows, 186, 215 and 288 with up to 64, 128 and 192, 360
// with more), so the whole rounds have room for some of the pieces: rest16 is what exceeds them, in sixteenths of a full
// item.  In k32 steps (0.7 us) an item takes `steps`, a piece steps / S plus about 14 for filling and draining its
// pipeline and writing its partial sums, the finishing pass about 25 plus what it reads (256 KB per piece; with the partial sums
// in register order it takes half of that, 35 -> 19 us for 256 pieces, and the estimate errs to the side of fewer pieces).
__device__ __forceinline__ int wide_cost16(int rows) { return rows <= 32 ? 7 : rows <= 64 ? 8 : rows <= 128 ? 10 : rows <= 192 ? 13 : 16; }

// Lane s weighs up s pieces; the cheapest, of equals the fewest, is taken.  All 64 lanes must call it.
__device__ __forceinline__ int wide_pieces(int rest, int rest16, int steps)
{
    const int s = threadIdx.x & 63;
    int cost = 0x7fffffff;
    if (s == 1) {
        cost = (steps + 14) << 5 | 1;
    } else if (s >= 2 && s <= WIDE_MAX_SPLIT && rest > 0 && rest * s <= WIDE_MAX_PIECES && steps >= 16 * s) {
        const int by_work = rest16 * s > 4096 + 256 ? (rest16 * s + 4095 - 256) / 4096 : 1;
        cost = ((1 + by_work) * (steps / s + 14) / 2 + 25 + rest * s / 7) << 5 | s;
    }
    return -wave_max_int_dpp(-cost) & 31;
}

// The items of a launch: row tiles, those items that run whole, pieces per item of the rest; work16: the work of all items in
// sixteenths of a full one.
struct wide_plan {
    moe_tiles tiles;
    int items, whole, pieces, work16;
};
__device__ __forceinline__ int wide_cost16_of(int c) { return c > 0 ? (c - 1) / WIDE_TM * 16 + wide_cost16((c - 1) % WIDE_TM + 1) : 0; }
__device__ __forceinline__ wide_plan wide_plan_of(const moe_rows &c, int n_nt, int steps)
{
    wide_plan p;
    p.tiles = moe_rank_tiles((c.c0 + WIDE_TM - 1) / WIDE_TM, (c.c1 + WIDE_TM - 1) / WIDE_TM);
    p.items = p.tiles.total * n_nt;
    const int rest = p.items % 256;
    p.work16 = wave_sum_int_dpp(wide_cost16_of(c.c0) + wide_cost16_of(c.c1)) * n_nt;
    p.pieces = wide_pieces(rest, p.work16 - (p.items - rest) * 16, steps);
    p.whole = p.pieces > 1 ? p.items - rest : p.items;
    return p;
}

// Whether this kernel or the tiled one (tiles of tm rows and cols columns, K unsplit) takes the down projection.  Which is
// faster follows from how well the items of either fill whole rounds of 256 compute units, so from the rows of every expert
// at work, which only the device knows: both are launched, every wave of the tiled one weighs them up from counts and mask, its
// first block writes the answer down, and the blocks of the slower one return.
// Durations, fitted to 6828 calls (d = 512 .. 8192, I = 8192 .. 28672, 2 to 128 experts, all, three, two or one quarter or one of
// them at work; 90 % of either within 10 %), in steps + 14 (filling and draining) times microseconds:
//   this kernel   0.40 a round + 0.40 a round's worth of work (fewer rows, less power, higher clock); with the rest cut
//                 0.575 a whole round + 0.19 its work + 0.47 the share of K of a piece + the finishing pass
//   tiled kernel  a a round + b a round's worth of items, a and b by the shape of its items (tiled_step_cost)
// This one has to come out 1 % ahead: 5380 of the calls go to it, median 1.17 times as fast as the tiled one, 4 of them below 0.96.
// With a line on the size of the activations alone, 1 call in 15 that it sent here was below 0.96, at worst 0.48.
// Those tiles were whole; items of 256 columns in a last round of half the units or less run as two of half the width now (cut_item_of),
// 0.80 of the time of such a launch, and are still charged as a whole round: 900 calls that take that width (d = 1024 .. 4096, I =
// 8192 .. 16384, 6 to 16 experts, skewed rows, masks) take 1.007 of the faster kernel's time in the mean, at worst 1.14, with 0.7 of a round
// 1.005 and 1.14, with 0.6 1.008 and 1.25; on 400 others 0.7 was level with a whole one (0.94 to 1.09).
// Down projection, tiled against this kernel, d = 4096, I = 14336: 1441 .. 190 rows of six experts 617 and 423 us, 1540 .. 126 rows of
// six (256 items of 256 x 256) 375 and 331, 8192 tokens through eight 1790 and 1570, but 280 .. 254 rows of six (256 items of 128 x
// 256, one exact round) 230 and 354 and 665 .. 596 rows of six (288 items of 256 x 256, 32 beyond one round) 374 and 442.
struct tiled_step_cost {
    int round, items;      // hundredths of a microsecond per k32 step
};
__device__ __forceinline__ tiled_step_cost tiled_step_cost_of(int cols, int tm)
{
    if (cols == 512) return tm == 96 ? tiled_step_cost{55, 14} : tm == 112 ? tiled_step_cost{50, 24} : tiled_step_cost{58, 22};
    if (cols == 256) return tm == 96 ? tiled_step_cost{26, 16} : tm == 112 ? tiled_step_cost{28, 18} : tiled_step_cost{36, 12};
    return tm == 96 ? tiled_step_cost{17, 9} : tm == 112 ? tiled_step_cost{19, 10} : tiled_step_cost{22, 9};
}
__device__ __forceinline__ bool wide_faster(const wide_plan &p, int steps, int items, int tm, int cols)
{
    // both in 1 / 51200 us
    const tiled_step_cost u = tiled_step_cost_of(cols, tm);
    const long long tiled = 2ll * (u.round * 256ll * ((items + 255) / 256) + (long long)u.items * items) * (steps + 14);
    const long long round = 256, rest = p.items % 256, work = p.work16 / 16;
    const long long wide = p.pieces == 1 ? 80 * (round * ((p.items + 255) / 256) + work) * (steps + 14)
                                         : (115 * round * (p.items / 256) + 38 * work) * (steps + 14) +
                                               round * (94 * (steps / p.pieces + 14) + 117 * (25 + rest * p.pieces / 7));
    return tiled * 100 > wide * 101;
}

#define WIDE_THREADS 256
#define WIDE_WAVES 4
#define WIDE_BUFS 4
#define WIDE_BUF_BYTES (WIDE_TM * 128)      // one k64 stage of activation rows
#define WIDE_SETS 8                          // weight register sets (k32 steps) ...
#define WIDE_AHEAD 7                         // ... of which this many are on their way

// 16 bytes per lane from buffer rsrc at voff + soff to LDS bytes lds_off + 16 * lane (all but voff wave-uniform).  Inline
// assembly, because the compiler waits for every LDS-direct load it knows of before the next LDS read; the waits for these
// are placed by hand (wait_vmem).  One wait state between the write of m0 and its use; m0 is a clobber, so that the compiler
// does not carry a value of its own in it past this (it warns because it never allocates m0, only sets it where it needs it).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void load_to_lds(u32x4 rsrc, uint32_t voff, uint32_t soff, uint32_t lds_off)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(lds_off), "v"(voff), "s"(rsrc), "s"(soff)
                 : "memory", "m0");
}
#pragma clang diagnostic pop

// at most N vector loads of this wave (register and LDS-direct alike, they complete in order) are still on their way.  Weight
// loads may be moved by the optimiser (it sinks those before the loop into it and drops those whose result is not used),
// so outside the main loop, where a set's load and its use are an iteration apart, N counts LDS-direct loads only.
template <int N> __device__ __forceinline__ void wait_vmem() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// acc += A B in place, accumulators in AGPRs.  Inline assembly, because left to itself the register allocator gives the
// result another quad of registers than the operand, and 256 accumulators fill all there are.
__device__ __forceinline__ void mfma_acc(f32x4 &acc, u32x4 a, u32x4 b)
{
    asm("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}

__device__ __forceinline__ u32x4 buffer_words(const void *p, uint32_t bytes)
{
    const uint64_t a = (uint64_t)p;
    return u32x4{(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)a), (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(a >> 32) & 0xffffu),
                 (uint32_t)__builtin_amdgcn_readfirstlane(bytes), 0x00027000u};
}

// NTT: 16-row subtiles computed (rows past nrows are clamped copies whose results are dropped).  The item covers the
// k32 steps [k0, k0 + nk) of K, nk a multiple of 4.
template <int NTT>
__device__ __forceinline__ void wide_body(char *lds, int d, int I, const uint16_t *__restrict__ act, const uint16_t *__restrict__ w2,
                                          int e, int nt, int row0, int nrows, int k0, int nk, uint16_t *__restrict__ y,
                                          float *__restrict__ part)
{
    constexpr int NF = WIDE_TN / WIDE_WAVES / 16;            // weight fragments per wave and step
    constexpr int P = NTT < 8 ? NTT : NTT % 8 == 0 ? 8 : 6;   // activation fragments read ahead of their MFMAs
    constexpr int DPS = NTT / 2;                              // LDS-direct loads per wave and k64 stage
    constexpr int D0 = (DPS + 1) / 2;                         // ... of which issued in the first of the two steps
    static_assert(NTT % P == 0, "the fragment ring restarts with every step");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, lg = lane >> 4;
    const int nst = nk / 2;                                   // k64 stages

    // ---- weights: 4 consecutive 16-row blocks of W2_e, 1 KB per block and step
    const int n0 = nt * WIDE_TN + wave * (WIDE_TN / WIDE_WAVES);
    const int col = n0 < d ? n0 : d - WIDE_TN / WIDE_WAVES;  // a wave past the ragged edge recomputes the last columns
    const uint32_t wbytes = (uint32_t)d * (uint32_t)I * 2u;   // < 4 GB: the launch checks
    const uint64_t wbase = (uint64_t)(w2 + (size_t)e * d * I);
    uint32_t wvo[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) wvo[f] = ((uint32_t)((col >> 4) + f) * (uint32_t)(I / 32) + (uint32_t)k0) * 1024u + lane * 16u;
    // ---- activation rows: instruction j of this wave fills rows 8 (4 j + wave) .. + 7 of the stage
    const u32x4 rx = buffer_words(act + (size_t)row0 * I, (uint32_t)nrows * (uint32_t)I * 2u);
    uint32_t xvo[DPS];
#pragma unroll
    for (int j = 0; j < DPS; ++j) {
        int r = (j * WIDE_WAVES + wave) * 8 + (lane >> 3);
        if (r >= nrows) r = nrows - 1;
        xvo[j] = ((uint32_t)r * (uint32_t)I + (uint32_t)k0 * 32u) * 2u + (uint32_t)((lane & 7) ^ (lane >> 3)) * 16u;
    }
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds) + wave * 1024u;
    const char *xr0 = lds + li * 128 + ((lg ^ (li & 7)) * 16);          // fragment reads, first and second k32 half of a stage
    const char *xr1 = lds + li * 128 + ((lg ^ 4 ^ (li & 7)) * 16);

    f32x4 acc[NF][NTT];
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int t = 0; t < NTT; ++t) acc[f][t] = f32x4{0.f, 0.f, 0.f, 0.f};

    // K is walked as a ring from an expert-dependent start, so that the items that share weights or rows stay in step
    const int st0 = (int)(((unsigned)e * 5u) % (unsigned)nst);
    u32x4 wr[WIDE_SETS][NF], xf[P];
    int kw = 2 * st0, kx = st0;             // the next weight step and activation stage to load ...
    int left_w = nk, left_x = nst;          // ... and how many are left
    uint32_t wsz = wbytes, xsz = rx.z;      // descriptor sizes: 0 once none is left

#define WLOAD(set, f)                                                                                                    \
    wr[set][f] = __builtin_amdgcn_raw_buffer_load_b128(__builtin_amdgcn_make_buffer_rsrc((void *)wbase, 0, wsz, 0x00027000), \
                                                       wvo[f], kw * 1024, 0)
#define WNEXT()                                   \
    do {                                          \
        kw = kw + 1 == nk ? 0 : kw + 1;           \
        wsz = --left_w > 0 ? wbytes : 0u;         \
    } while (0)
#define XLOAD(buf, j) load_to_lds(u32x4{rx.x, rx.y, xsz, rx.w}, xvo[j], kx * 128, lds0 + (buf) * WIDE_BUF_BYTES + (j) * 4096)
#define XNEXT()                                   \
    do {                                          \
        kx = kx + 1 == nst ? 0 : kx + 1;          \
        xsz = --left_x > 0 ? rx.z : 0u;           \
    } while (0)
#define XREAD(slot, buf, half, t) \
    xf[slot] = *reinterpret_cast<const u32x4 *>(((half) ? xr1 : xr0) + (buf) * WIDE_BUF_BYTES + (t) * 2048)

    // the descriptor words come from VALU instructions, and the compiler does not see the loads that read them next (5 wait
    // states)
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 7");
    // ---- stages 0 and 1 and the first half of stage 2 on their way, with the weights of 7 steps
#pragma unroll
    for (int s = 0; s < 3; ++s) {
#pragma unroll
        for (int j = 0; j < (s == 2 ? D0 : DPS); ++j) XLOAD(s, j);
        if (s < 2) XNEXT();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 2 * s; u < (s == 2 ? WIDE_AHEAD : 2 * s + 2); ++u) {
#pragma unroll
            for (int f = 0; f < NF; ++f) WLOAD(u, f);
            WNEXT();
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    wait_vmem<DPS + D0>();                                    // stage 0: followed by these, and maybe by weights
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < P; ++t) XREAD(t, 0, 0, t);

    // One k32 step: half `half` of the stage in buffer buf with weight set ws.  Every subtile is 4 MFMAs, one fragment
    // read P subtiles ahead and at most two loads; the fence keeps the compiler from bunching them.
#define STEP(buf, half, ws)                                                                                      \
    do {                                                                                                         \
        _Pragma("unroll") for (int t = 0; t < NTT; ++t) {                                                        \
            _Pragma("unroll") for (int f = 0; f < NF; ++f) mfma_acc(acc[f][t], wr[ws][f], xf[t % P]);            \
            if (t + P < NTT) XREAD(t % P, buf, half, t + P);                                                     \
            else if ((half) == 0) XREAD(t % P, buf, 1, t + P - NTT);                                             \
            else XREAD(t % P, ((buf) + 1) % WIDE_BUFS, 0, t + P - NTT);                                          \
            _Pragma("unroll") for (int f = 0; f < NF; ++f)                                                       \
                if (f * NTT / NF == t) WLOAD(((ws) + WIDE_AHEAD) % WIDE_SETS, f);                                \
            _Pragma("unroll") for (int j = 0; j < DPS; ++j)                                                      \
                if (((half) == 1) == (j < D0) && ((half) == 1 ? j : j - D0) * 2 + 1 == t)                        \
                    XLOAD(((buf) + ((half) == 1 ? 3 : 2)) % WIDE_BUFS, j);                                       \
            __builtin_amdgcn_sched_barrier(0);                                                                   \
        }                                                                                                        \
        WNEXT();                                                                                                 \
    } while (0)
    // One stage.  In its middle the next stage has landed (this wave's loads for it are followed by the DPS of the stage
    // after it and, in the main loop, by NF loads of weights in each of two steps) and every wave is done with the stage before, whose buffer
    // the loads of the second step overwrite.
#define STAGE(buf, ws, weights)                                                                                  \
    do {                                                                                                         \
        STEP(buf, 0, ws);                                                                                        \
        XNEXT();                                                                                                 \
        wait_vmem<DPS + (weights)>();                                                                            \
        __builtin_amdgcn_s_barrier();                                                                            \
        __builtin_amdgcn_sched_barrier(0);                                                                       \
        STEP(buf, 1, (ws) + 1);                                                                                  \
    } while (0)

    // The compiler does not know that mfma_acc delivers late, and may copy or store accumulators wherever control flow
    // joins: MFMAS_DONE stands before every such point (18 wait states are what reading a result needs at most).
#define MFMAS_DONE()                                   \
    do {                                               \
        asm volatile("s_nop 15\n\ts_nop 7");           \
        __builtin_amdgcn_sched_barrier(0);             \
    } while (0)
    for (int s = 0; s + WIDE_SETS <= nk; s += WIDE_SETS) {
        STAGE(0, 0, 2 * NF);
        STAGE(1, 2, 2 * NF);
        STAGE(2, 4, 2 * NF);
        STAGE(3, 6, 2 * NF);
        MFMAS_DONE();
    }
    if (nk & 4) {
        STAGE(0, 0, 0);
        STAGE(1, 2, 0);
        MFMAS_DONE();
    }
#undef MFMAS_DONE
#undef STAGE
#undef STEP
#undef XREAD
#undef XNEXT
#undef XLOAD
#undef WNEXT
#undef WLOAD
    wait_vmem<0>();                                    // no load may write LDS after the block has gone

    // ---- epilogue: a lane holds output columns 4 lg + 0..3 of row li of every 16x16 tile
    if (part == nullptr) __syncthreads();              // every wave is done with the stages, the ones past the edge of y among them
    if (n0 >= d) return;
    if (part != nullptr) {
        // the sums of a piece as they lie in the registers, 1 KB per tile (wide_finish_kernel knows the order): stored by rows,
        // neighbouring lanes in different rows, each of the 64 lanes is an access of its own
#pragma unroll
        for (int t = 0; t < NTT; ++t)
#pragma unroll
            for (int f = 0; f < NF; ++f)
                *reinterpret_cast<f32x4 *>(part + ((size_t)((wave * NF + f) * (WIDE_TM / 16) + t) * 64 + lane) * 4) = acc[f][t];
        return;
    }
    // rows of y go through LDS (2 KB of this wave's own), so that eight lanes store 128 bytes of a row; chunk c (16 bytes) of row i in
    // slot c ^ (i & 7)
    char *ys = lds + wave * 2048;
    const int yr = lane >> 3, yc = lane & 7;
#pragma unroll
    for (int t = 0; t < NTT; ++t) {
#pragma unroll
        for (int f = 0; f < NF; ++f)
            *reinterpret_cast<u32x2 *>(ys + li * 128 + (((f * 2 + (lg >> 1)) ^ (li & 7)) * 16) + (lg & 1) * 8) =
                u32x2{pack_bf16x2(acc[f][t][0], acc[f][t][1]), pack_bf16x2(acc[f][t][2], acc[f][t][3])};
        // the lanes of a wave exchange data: LDS serves a wave's accesses in order, the compiler keeps theirs
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int q = 0; q < 16; q += 8) {
            const int i = q + yr;
            const u32x4 v = *reinterpret_cast<const u32x4 *>(ys + i * 128 + ((yc ^ (i & 7)) * 16));
            if (t * 16 + i < nrows) *reinterpret_cast<u32x4 *>(y + (size_t)(row0 + t * 16 + i) * d + n0 + yc * 8) = v;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
}

struct wide_item {
    int e, nt, row0, nrows;
};

__device__ __forceinline__ wide_item wide_item_of(int L, int n_nt, const moe_tiles &tiles, const int32_t *__restrict__ offsets,
                                                  const int32_t *__restrict__ counts)
{
    int e, first, n;
    moe_find_tile(tiles, L / n_nt, e, first, n);
    const int local = L - first * n_nt;
    const int nt = local / n, mt = local - nt * n;             // the row tiles that share a weight tile follow each other
    const int rows = counts[e] - mt * WIDE_TM;
    return wide_item{e, nt, offsets[e] + mt * WIDE_TM, rows > WIDE_TM ? WIDE_TM : rows};
}

__global__ __launch_bounds__(WIDE_THREADS, 1) void ffn_wide_kernel(int d, int I, int N, const uint16_t *__restrict__ act,
                                                                   const int32_t *__restrict__ offsets, const int32_t *__restrict__ counts,
                                                                   const uint16_t *__restrict__ w2, const uint8_t *__restrict__ mask,
                                                                   uint16_t *__restrict__ y, float *__restrict__ partial, const int32_t *__restrict__ works)
{
    __shared__ __attribute__((aligned(1024))) char lds[WIDE_BUFS * WIDE_BUF_BYTES];
    const int n_nt = (d + WIDE_TN - 1) / WIDE_TN;
    if (*works == 0) return;
    const wide_plan plan = wide_plan_of(moe_masked_rows(N, counts, mask), n_nt, I / 32);
    const int items = plan.items, whole = plan.whole, S = plan.pieces;
    const int pid = blockIdx.x;
    int total = whole, base = 0, r = 1;
    if (pid >= whole) {                                        // pieces: all first pieces, then all second ones, ...
        r = items - whole;
        total = r * S;
        base = whole;
        if (pid - base >= total) return;
    }
    // a contiguous run of the list per XCD
    const int q = total / MOE_NUM_XCD, rem = total % MOE_NUM_XCD;
    const int xcd = (pid - base) % MOE_NUM_XCD, loc = (pid - base) / MOE_NUM_XCD;
    const int L = xcd < rem ? xcd * (q + 1) + loc : rem * (q + 1) + (xcd - rem) * q + loc;
    int item = L, k0 = 0, nk = I / 32;
    float *part = nullptr;
    if (pid >= whole) {
        const int sp = L / r, quads = I / 128;
        item = whole + L - sp * r;
        k0 = sp * quads / S * 4;
        nk = (sp + 1) * quads / S * 4 - k0;
        part = partial + (size_t)L * WIDE_TM * WIDE_TN;
    }
    const wide_item it = wide_item_of(item, n_nt, plan.tiles, offsets, counts);
    MOE_TRACE_BEGIN();
#define BODY(n) wide_body<n>(lds, d, I, act, w2, it.e, it.nt, it.row0, it.nrows, k0, nk, y, part)
    if (it.nrows <= 32) BODY(2);
    else if (it.nrows <= 64) BODY(4);
    else if (it.nrows <= 128) BODY(8);
    else if (it.nrows <= 192) BODY(12);
    else BODY(16);
#undef BODY
    MOE_TRACE_END(1, it.e, it.nrows, it.nt);
}

// y rows of the items that ran in pieces: the partial sums added in piece order.  A block takes 64 columns (a wave's share of the
// item) of 16 rows at a time, each wave one fragment of them; the rows are put together in LDS.
__global__ __launch_bounds__(256) void wide_finish_kernel(int d, int steps, int N, const int32_t *__restrict__ offsets,
                                                          const int32_t *__restrict__ counts, const uint8_t *__restrict__ mask, const float *__restrict__ partial,
                                                          uint16_t *__restrict__ y, const int32_t *__restrict__ works)
{
    __shared__ __attribute__((aligned(16))) char ys[2][2048];
    const int n_nt = (d + WIDE_TN - 1) / WIDE_TN;
    if (*works == 0) return;
    const wide_plan plan = wide_plan_of(moe_masked_rows(N, counts, mask), n_nt, steps);
    const int whole = plan.whole, S = plan.pieces, r = plan.items - whole;
    const int j = blockIdx.y, w = blockIdx.x % 4;
    if (S == 1 || j >= r) return;
    const wide_item it = wide_item_of(whole + j, n_nt, plan.tiles, offsets, counts);
    const int col = it.nt * WIDE_TN + w * 64;
    if (col >= d) return;
    const int lane = threadIdx.x & 63, f = threadIdx.x >> 6, li = lane & 15, lg = lane >> 4;
    const int nt16 = (it.nrows + 15) / 16;
    int b = 0;
    for (int t = blockIdx.x / 4; t < nt16; t += gridDim.x / 4, b ^= 1) {
        const float *p = partial + ((((size_t)j * 16 + w * 4 + f) * (WIDE_TM / 16) + t) * 64 + lane) * 4;
        f32x4 a = *reinterpret_cast<const f32x4 *>(p);
        for (int s = 1; s < S; ++s) {
            p += (size_t)r * WIDE_TM * WIDE_TN;
            a += *reinterpret_cast<const f32x4 *>(p);
        }
        *reinterpret_cast<u32x2 *>(ys[b] + li * 128 + (((f * 2 + (lg >> 1)) ^ (li & 7)) * 16) + (lg & 1) * 8) = u32x2{pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3])};
        __syncthreads();
        const int i = threadIdx.x >> 3, c = threadIdx.x & 7;
        if (i < 16 && t * 16 + i < it.nrows)
            *reinterpret_cast<u32x4 *>(y + (size_t)(it.row0 + t * 16 + i) * d + col + c * 8) = *reinterpret_cast<const u32x4 *>(ys[b] + i * 128 + ((c ^ (i & 7)) * 16));
    }
}

// works: whether this kernel or the tiled one, launched before it, takes the projection; written there
static int moe_ffn_wide_down(const moe_shape *s, const int32_t *offsets, const int32_t *counts, const void *act, const void *w2,
                      void *y, const uint8_t *mask, float *partial, const int32_t *works, hipStream_t st)
{
    const int d = s->d, I = s->I, N = s->N;
    const long max_items = (long)moe_wide_max_items(s);
    const long blocks = (max_items / 256 + 1) * 256;          // whole items in rounds of 256, then uncut ones or at most 256 pieces
    hipLaunchKernelGGL(ffn_wide_kernel, dim3((unsigned)blocks), dim3(WIDE_THREADS), 0, st, d, I, N, (const uint16_t *)act, offsets, counts,
                       (const uint16_t *)w2, mask, (uint16_t *)y, partial, works);
    MOE_CHECK_LAUNCH();
    const long cut = max_items < WIDE_MAX_PIECES / 2 ? max_items : WIDE_MAX_PIECES / 2;      // an item that is cut has two pieces or more
    hipLaunchKernelGGL(wide_finish_kernel, dim3(16, (unsigned)cut), dim3(256), 0, st, d, I / 32, N, offsets, counts, mask, partial, (uint16_t *)y, works);
    MOE_CHECK_LAUNCH();
    return MOE_OK;
}

// Both projections of the tiled expert FFN as one launch, of a layer's routed experts or of its routed and shared ones.
//
// A launch of the tiled kernel ends with a round of items that fills part of the chip, and the next one waits for all of it.  Here one
// block per compute unit takes item after item, those of the up projection first, and goes on with the down projection when none of
// them is left to take; a down item waits for the activations of its own token tile only.
//   * Every XCD has a queue of an eighth of the shared and, behind them, of the routed experts' up items, and one of their down items.
//     A block takes from its own XCD's queue, then from the others'.  Neighbouring XCDs walk the tiles in opposite directions: those on
//     the border of two shares are the first of both or the last of both, and few blocks ever wait.
//   * A block takes a down item only when all up items have been taken, and has none of them in hand while it waits: they are
//     being worked on by running blocks that wait for nothing.  That holds in whatever order blocks start, with fewer compute units
//     than blocks and with another such launch beside this one.  The wait has a bound all the same (MOE_JOINT_MAX_POLLS looks at the
//     counter, seconds; the waits seen are tens of microseconds).  A wave that reaches it has loaded rows that may be incomplete: the
//     rows of that item become NaN (joint_void).
//   * The ticket after an item is asked for between its last product and its stores, which hide the way to the counter and back.
//   * arrived[t] counts the up items of token tile t whose activations have been stored.  The activations are stored past the caches of
//     the XCD (sc1, device scope) and every wave waits for its stores before the block counts itself in, so the block that sees the
//     full count may read them.  It cannot find older contents in a cache: an activation is read by nothing before its tile is
//     complete (rows are whole 128-byte lines, rows past the tile's end are not touched), and a launch starts with clean caches.
//     With release and acquire fences in place of that (the whole L2 written back by each up item) an up item of 50 us took 56 to 65.
//   * Counters and tickets are cleared by a launch of one block ahead.
// Passes of whole layers, two or four launches / this: 2048 tokens of 6 slots, 32 of 64 experts, d = 2048, I = 1408, and two shared
// ones 356 / 309 us; 1531 tokens of 8 slots, 64 of 128 experts, I = 768 222 / 201; 4096 tokens of 4 slots, 60 experts, I = 1408, and a shared
// one of 5632 653 / 609.  The compute units are busy for 0.92 of the launch (0.78 to 0.85 of the separate ones); what an item takes is
// bound as in ffn_tiled.hip.
#pragma once

struct joint_experts {
    const int32_t *perm, *offsets, *counts;
    const uint16_t *w1, *w3, *w2;
    const uint8_t *mask;
    uint16_t *act, *y;
    int32_t *arrived;
    int I, N, k;                        // N = 0: none
};
struct joint_args {
    joint_experts x[2];                 // routed, shared
    const uint16_t *h;
    int32_t *tickets;                   // of the up items, then of the down items
    int d, polls;
};

#define JOINT_BLOCKS_PER_XCD 32         // a block to a compute unit

// tickets: of eight queues of up items and eight of down items (joint_ask); a, b: counters of the routed and of the shared experts' tiles
__global__ __launch_bounds__(256) void joint_clear_kernel(int32_t *tickets, int32_t *a, int na, int32_t *b, int nb)
{
    for (int i = threadIdx.x; i < na; i += 256) a[i] = 0;
    for (int i = threadIdx.x; i < nb; i += 256) b[i] = 0;
    if (threadIdx.x < 2 * MOE_NUM_XCD) tickets[threadIdx.x * MOE_JOINT_TICKET_STRIDE] = 0;
}

// items of a list of total that XCD xcd takes, and the first of them
__device__ __forceinline__ int joint_share(int total, int xcd) { return total / MOE_NUM_XCD + (xcd < total % MOE_NUM_XCD ? 1 : 0); }
__device__ __forceinline__ int joint_first(int total, int xcd) { return xcd * (total / MOE_NUM_XCD) + min(xcd, total % MOE_NUM_XCD); }

// Tickets of eight queues, 128 bytes apart (on one line the atomics of all blocks follow one another).  The next place in queue q is
// asked for ahead of its use, by lane 0.
__device__ __forceinline__ int joint_ask(int32_t *tickets, int q)
{
    return (threadIdx.x & 63) == 0 ? __hip_atomic_fetch_add(tickets + q * MOE_JOINT_TICKET_STRIDE, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
}

// The place that was asked for in queue `own`, or, where that is beyond its end, one of the next queue with an item left (q); -1 once
// all eight are empty.  length: items of the queues in the first eight lanes.  A whole wave calls it.
__device__ __forceinline__ int joint_get(int32_t *tickets, int asked, int own, int length, int &q)
{
    const int lane = threadIdx.x & 63;
    q = own;
    int place = __builtin_amdgcn_readfirstlane(asked);
    while (place >= __builtin_amdgcn_readlane(length, q)) {
        // all eight counters at once: most blocks that come here find that nothing is left
        int taken = 0x7fffffff;
        if (lane < MOE_NUM_XCD) taken = __hip_atomic_load(tickets + lane * MOE_JOINT_TICKET_STRIDE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned left = (unsigned)__ballot(taken < length);
        if (left == 0) return -1;
        const unsigned after = left >> q << q;
        q = __ffs(after != 0 ? after : left) - 1;
        place = __builtin_amdgcn_readfirstlane(joint_ask(tickets, q));
    }
    return place;
}

// The last routed down items of every queue run as two of half the width.  8 / 16 / 24 of them, two or four separate launches as the
// yardstick, 48 calls of 300 to 4096 tokens on three layer shapes: 1.122, 1.124 and 1.120 times as fast in the mean; 2048 tokens of 6
// slots, 32 of 64 experts, I = 1408 220 / 217 / 220 us, 900 tokens of 4 slots, 30 of 60 experts 135 / 143 / 144.
#define JOINT_CUT 16

// The arguments where the launch put them.  Read anew by every item: kept in registers across the items' loops they are more than
// there are.
typedef const __attribute__((address_space(4))) joint_args *joint_args_ptr;
__device__ __forceinline__ joint_args_ptr joint_arguments()
{
    joint_args_ptr p = (joint_args_ptr)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}

// What a block keeps of one set of experts: the places of their token tiles (moe_tiles of every lane), rows and first rows.  Read
// from memory by every item, counts and offsets were two trips ahead of its first load.
struct joint_table {
    int n[2][64], first[2][64], rows[128], row0[128], total;
};
// Filled by one wave: of an item's 35 to 60 us the two trips were 0.4 to 0.8 (passes 312.8 -> 308.4, 199.5 -> 198.2 and 612.1 -> 605.9 us).
__device__ __forceinline__ void joint_fill(joint_table &t, joint_args_ptr a, int shared)
{
    const int lane = threadIdx.x & 63, N = a->x[shared].N;
    moe_tiles m = {0, 0, 0, 0, 0};
    if (N > 0) {
        const int32_t *const offsets = a->x[shared].offsets;
        const int o0 = offsets[min(lane, N - 1)], o1 = offsets[min(lane + 64, N - 1)];
        const moe_rows r = moe_masked_rows(N, a->x[shared].counts, a->x[shared].mask);
        m = tiles_128(r);
        t.rows[lane] = r.c0;
        t.rows[lane + 64] = r.c1;
        t.row0[lane] = o0;
        t.row0[lane + 64] = o1;
    }
    t.n[0][lane] = m.n0;
    t.n[1][lane] = m.n1;
    t.first[0][lane] = m.first0;
    t.first[1][lane] = m.first1;
    if (lane == 0) t.total = m.total;
}

struct joint_item {
    int kind;      // bit 0 down, bit 1 shared, bits 2 and 3: 0 whole, 1 first half, 2 second half; -1: no item is left
    int e, nt, row0, nrows, tile;
};

#define JOINT_UP_COLS 256

// The item of the place that was asked for, or of the next queue (see the kernel).  The first wave of a block calls it.
template <int NFD>
__device__ __forceinline__ joint_item joint_next(const joint_table *tables, int asked, int own, bool &asks_down)
{
    constexpr int DOWN_COLS = 128 * NFD;
    constexpr bool CUT = NFD > 1;
    const joint_args_ptr a = joint_arguments();
    const int tiles_a = __builtin_amdgcn_readfirstlane(tables[0].total), tiles_b = __builtin_amdgcn_readfirstlane(tables[1].total);
    const int Ia = a->x[0].I, Ib = a->x[1].I, d = a->d;
    const int up_a = (Ia + JOINT_UP_COLS - 1) / JOINT_UP_COLS, up_b = (Ib + JOINT_UP_COLS - 1) / JOINT_UP_COLS, down_a = (d + DOWN_COLS - 1) / DOWN_COLS;
    // shared experts of a long inner size: their down items at half width, or one of them outlasts two rounds of the others
    const bool b_half = CUT && Ib > 2 * Ia;
    const int down_b = b_half ? (d + DOWN_COLS / 2 - 1) / (DOWN_COLS / 2) : down_a;
    const int ups_b = tiles_b * up_b, ups_a = tiles_a * up_a, downs_b = tiles_b * down_b, downs_a = tiles_a * down_a;
    const int lane = threadIdx.x & 63, qx = lane % MOE_NUM_XCD;
    int q = 0, place = -1;
    if (!asks_down) {
        place = joint_get(a->tickets, asked, own, joint_share(ups_b, qx) + joint_share(ups_a, qx), q);
        if (place < 0) {
            asks_down = true;
            asked = joint_ask(a->tickets + MOE_NUM_XCD * MOE_JOINT_TICKET_STRIDE, own);
        }
    }
    if (asks_down) {
        const int n = joint_share(downs_a, qx);
        place = joint_get(a->tickets + MOE_NUM_XCD * MOE_JOINT_TICKET_STRIDE, asked, own, joint_share(downs_b, qx) + n + (CUT ? min(n, JOINT_CUT) : 0), q);
    }
    if (place < 0) return joint_item{-1, 0, 0, 0, 0, 0};
    const int list_b = asks_down ? downs_b : ups_b, list_a = asks_down ? downs_a : ups_a;
    const int n_b = joint_share(list_b, q), n_a = joint_share(list_a, q);
    const bool sb = place < n_b;
    int half = 0;
    if (!sb) {
        place -= n_b;
        const int cut = min(n_a, JOINT_CUT), whole = n_a - cut;
        if (CUT && asks_down && place >= whole) {
            const int j = place - whole;
            half = 1 + (j & 1);
            place = whole + (j >> 1);
        }
    }
    const int n_q = sb ? n_b : n_a;
    const int L = joint_first(sb ? list_b : list_a, q) + ((q & 1) != 0 ? n_q - 1 - place : place);
    const int n_nt = asks_down ? (sb ? down_b : down_a) : sb ? up_b : up_a;
    const joint_table &t = tables[sb];
    joint_item it;
    int first, n;
    moe_find_tile(moe_tiles{t.n[0][lane], t.n[1][lane], t.first[0][lane], t.first[1][lane], 0}, L / n_nt, it.e, first, n);
    const int local = L - first * n_nt;
    it.nt = local / n;                         // the token tiles that share a weight tile follow each other
    const int mt = local - it.nt * n;
    if (sb && b_half && asks_down) {
        half = 1 + (it.nt & 1);
        it.nt >>= 1;
    }
    it.kind = (asks_down ? 1 : 0) | (sb ? 2 : 0) | half << 2;
    it.row0 = t.row0[it.e] + mt * TM;
    it.nrows = min(t.rows[it.e] - mt * TM, TM);
    it.tile = first + mt;
    return it;
}

// NaN into the results of a down item.  Called by a wave behind a barrier that follows the stores of all of them.
template <int NFD>
__device__ __forceinline__ void joint_void(const joint_item &it)
{
    const joint_args_ptr a = joint_arguments();
    const int half = it.kind >> 2, d = a->d, cols = half == 0 ? 128 * NFD : 64 * NFD;
    const int col0 = half == 0 ? it.nt * cols : (2 * it.nt + half - 1) * cols, end = min(col0 + cols, d);
    uint16_t *const y = a->x[it.kind >> 1 & 1].y;
    for (int r = 0; r < it.nrows; ++r)
        for (int c = col0 + (threadIdx.x & 63) * 8; c < end; c += 64 * 8)
            *reinterpret_cast<u32x4 *>(y + (size_t)(it.row0 + r) * d + c) = u32x4{0x7fc07fc0u, 0x7fc07fc0u, 0x7fc07fc0u, 0x7fc07fc0u};
}

// NFD: weight fragments per wave of the down projection (128 output columns each)
template <int NFD>
__global__ __launch_bounds__(TILED_THREADS, 2) void ffn_joint_kernel(joint_args)
{
    __shared__ joint_item next, given_up[8];       // given_up: of every wave, the item whose activations it did not wait for any longer
    __shared__ joint_table tables[2];
    __shared__ __attribute__((aligned(16))) uint16_t Xs[2][2][TM * 32];
    __shared__ __attribute__((aligned(16))) char Ys[8][2048];
    constexpr int DOWN_COLS = 128 * NFD;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), own = blockIdx.x % MOE_NUM_XCD;
    bool asks_down = false;
    int asked = 0;
    const auto ask = [&]() {
        if (wave == 0) asked = joint_ask(joint_arguments()->tickets + (asks_down ? MOE_NUM_XCD * MOE_JOINT_TICKET_STRIDE : 0), own);
    };
    const auto get = [&]() {
        if (wave == 0) {
            const joint_item it = joint_next<NFD>(tables, asked, own, asks_down);
            if (threadIdx.x == 0) next = it;
        }
        __syncthreads();
    };
    // the first tickets are taken like the others: dealt by the block id, they would belong to blocks that may not have started
    ask();
    if (wave < 2) joint_fill(tables[wave], joint_arguments(), wave);
    __syncthreads();
    get();
    while (true) {
        const int kind = __builtin_amdgcn_readfirstlane(next.kind);
        if (kind < 0) return;
        const int e = __builtin_amdgcn_readfirstlane(next.e), row0 = __builtin_amdgcn_readfirstlane(next.row0);
        const int nrows = __builtin_amdgcn_readfirstlane(next.nrows), tile = __builtin_amdgcn_readfirstlane(next.tile);
        int nt = __builtin_amdgcn_readfirstlane(next.nt), tid = threadIdx.x;
        asm volatile("" : "+v"(tid));                   // what the bodies derive from it is not kept across the items
        const joint_args_ptr args = joint_arguments();
        const auto x = &args->x[kind >> 1 & 1];
        const int d = args->d, I = x->I, k = x->k, half = kind >> 2;
        bool gave_up = false;
        uint16_t *const act = x->act;
        char *const ys = Ys[wave];
#define BODY(mode_, nf_, n_, x_, perm_, wa_, wb_, out_) \
    tile_body<mode_, nf_, n_, 4, false, 8, mode_ == 0>(&Xs[0][0][0], ys, d, I, k, x_, perm_, wa_, wb_, out_, e, nt, row0, nrows, 0, 1, nullptr, 0, tid, ask)
#define BODIES(mode_, nf_, ...)                                  \
    do {                                                         \
        if (nrows <= 16) BODY(mode_, nf_, 1, __VA_ARGS__);       \
        else if (nrows <= 32) BODY(mode_, nf_, 2, __VA_ARGS__);  \
        else if (nrows <= 64) BODY(mode_, nf_, 4, __VA_ARGS__);  \
        else if (nrows <= 96) BODY(mode_, nf_, 6, __VA_ARGS__);  \
        else BODY(mode_, nf_, 8, __VA_ARGS__);                   \
    } while (0)
        if ((kind & 1) == 0) {
            const int32_t *const perm = x->perm;
            const uint16_t *const h = args->h, *const w1 = x->w1, *const w3 = x->w3;
            // a ragged last column tile is a half-width item (I is a multiple of 128)
            if (__builtin_expect(nt < I / JOINT_UP_COLS, 1)) {
                BODIES(0, 4, h, perm, w1, w3, act);
            } else {
                nt *= 2;
                BODIES(0, 2, h, perm, w1, w3, act);
            }
            // every wave's stores have left, then one thread reports
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            if (threadIdx.x == 0) __hip_atomic_fetch_add(joint_arguments()->x[kind >> 1 & 1].arrived + tile, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            const uint16_t *const w2 = x->w2;
            uint16_t *const y = x->y;
            int32_t *const arrived = x->arrived + tile;
            const int want = (I + JOINT_UP_COLS - 1) / JOINT_UP_COLS, most = args->polls;
            int polls = 0;
            while (polls < most && __builtin_amdgcn_readfirstlane(__hip_atomic_load(arrived, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) < want) {
                __builtin_amdgcn_s_sleep(8);
                ++polls;
            }
            gave_up = polls == most;
            if (__builtin_expect(gave_up, 0)) given_up[wave] = next;
            const uint16_t *act_in = act;
            asm volatile("" : "+s"(act_in)::"memory");      // no read of the activations moves ahead of the wait
            if (NFD == 1 || half == 0) {
                BODIES(1, NFD, act_in, nullptr, w2, nullptr, y);
            } else if constexpr (NFD > 1) {
                nt = 2 * nt + half - 1;
                if (nt * (DOWN_COLS / 2) < d) {
                    BODIES(1, NFD / 2, act_in, nullptr, w2, nullptr, y);
                } else {                                     // a ragged last column tile may have no second half
                    ask();
                    __syncthreads();                         // every wave has read `next`; elsewhere a body's barriers see to that
                }
            }
        }
        get();
        if (__builtin_expect(gave_up, 0)) joint_void<NFD>(given_up[wave]);
    }
#undef BODIES
#undef BODY
}

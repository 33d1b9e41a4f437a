// Gate, top-k, workload histogram, token permutation and next-layer workload prediction for gfx950.
//
// moe_route (Eq. 1 and the expert workload of Section "Greedy Assignment Strategy"):
//   gate_topk_kernel      16 tokens per block, all experts; logits by bf16 MFMA 16x16x32 straight from global memory
//                         (K split over the 16 waves, reduced through LDS), then softmax and top-k per token
//                         inside one wavefront: k rounds of a DPP max reduction + ballot.
//   hist_scan_perm_kernel one block per expert: ballot counts of the selections below / equal to the expert
//                         (= its offset and workload), then a ballot-based stable compaction of its rows.
//   Decode-sized batches (T <= 16, T*k <= 128) need no second kernel: the selecting block builds a 16-bit
//   token mask per expert in LDS, and workload, scan and permutation are popcounts of it.  With more than 16
//   experts the gate product of such a batch is first spread over one block per 16 experts and select_decode_kernel
//   (one wavefront per token) selects from the stored logits.
// moe_predict_workload (Section "Residual-Based Prefetching"):
//   the same kernels on the next layer's gate with bias'[e] = bias[e] + res_vec . W[e], so that
//   (h + res_vec) . W + bias = h . W + bias'.  res_vec runs through the gate product as three more token rows (its exact split
//   into three bf16 numbers), so the fold costs no pass over the gate matrix.  Decode-sized: the selecting block emits the
//   workloads and their p largest.  Larger: hist_top_block.
// moe_route_predict: both gates as two "jobs" of the same launches (blockIdx.z); beyond decode sizes the histogram of the
// prediction is one more block of hist_scan_perm_kernel.
#include "moe_common.h"

#define ROUTE_TOKENS 16      // tokens per block of gate_topk_kernel
#define ROUTE_THREADS 1024
#define ROUTE_SEGS 16
// The residual vector of a gate is three more rows of the product.  RES_IN_TILE: rows 13 .. 15 of a block's 16, which takes 13 tokens
// (blocks that walk token tiles convert them once).  RES_BESIDE: an operand of their own, so that a block still takes 16 tokens.
#define RES_NONE 0
#define RES_IN_TILE 1
#define RES_BESIDE 2
#define FOLD_ROW 13

// The p largest workloads by descending value, equal values by ascending index; one wavefront, lane l holding the
// workloads c0 of expert l and c1 of expert l + 64.  A workload is at most T < 2^24 (T d < 2^31, d >= 128), so workload and
// index fit one int whose maximum is the next entry: p maxima on the DPP crossbar (through LDS shuffles of workload and
// index, 8 of 128 took 3 us of a decode step).
__device__ __forceinline__ void top_p_of(int c0, int c1, int N, int p, int32_t *__restrict__ top, int lane)
{
    int k0 = lane < N ? (c0 << 7 | (127 - lane)) : -1;
    int k1 = lane + 64 < N ? (c1 << 7 | (63 - lane)) : -1;
    for (int s = 0; s < p; ++s) {
        const int best = wave_max_int_dpp(k0 > k1 ? k0 : k1);
        if (k0 == best) k0 = -1;
        if (k1 == best) k1 = -1;
        if (lane == 0) top[s] = 127 - (best & 127);
    }
}

// ---------------------------------------------------------------------------------------------------
// Softmax + top-k of one token inside a wavefront: lane l holds the logits v0 of expert l and v1 of expert l + 64.  k rounds of:
// wave-wide max on the DPP crossbar, then the lowest expert index holding that value (ballot + find-first-set; the lower 64
// experts are asked first), which is the tie rule "equal scores by ascending index".  Lane s < k returns the s-th selection and its
// softmax score; sel = sum of the k scores.
// The rounds compare integers that order as the logits do: floats cost a canonicalisation per maximum, and four waves of a
// SIMD share its issue slots (16 tokens of 64 experts, 6 slots: 2.3 us of a 5.6 us launch).  A logit that is no number comes
// after every other one.
#define NO_EXPERT ((int)0x80000000u)
__device__ __forceinline__ int logit_key(float v)
{
    const int b = __float_as_int(v + 0.f);                                    // -0 and 0 are equal
    return v != v ? NO_EXPERT + 1 : b ^ (b >> 31 & 0x7fffffff);
}
__device__ __forceinline__ float key_logit(int key)
{
    return key == NO_EXPERT + 1 ? __int_as_float(0x7fc00000) : __int_as_float(key ^ (key >> 31 & 0x7fffffff));
}
__device__ __forceinline__ void select_token(float v0, float v1, int N, int k, int lane, int &my_idx, float &my_p, float &sel)
{
    int k0 = lane < N ? logit_key(v0) : NO_EXPERT, k1 = lane + 64 < N ? logit_key(v1) : NO_EXPERT;
    int best = wave_max_int_dpp(N > 64 ? max(k0, k1) : k0), my_best = best;
    const float m = key_logit(best);
    const float NEG = -__builtin_huge_valf();
    const float p0 = lane < N && v0 > NEG ? expf(v0 - m) : 0.f;
    const float p1 = lane + 64 < N && v1 > NEG ? expf(v1 - m) : 0.f;
    const float den = wave_sum_dpp(p0 + p1);
    my_idx = 0;
    if (N > 64) {
        for (int s = 0; s < k; ++s) {
            if (s > 0) best = wave_max_int_dpp(max(k0, k1));
            const unsigned long long b0 = __ballot(k0 == best), b1 = __ballot(k1 == best);
            const int bi = b0 != 0ull ? __ffsll((long long)b0) - 1 : 63 + __ffsll((long long)b1);
            if (lane == bi) k0 = NO_EXPERT;
            if (lane + 64 == bi) k1 = NO_EXPERT;
            if (lane == s) { my_idx = bi; my_best = best; }
        }
    } else {
        for (int s = 0; s < k; ++s) {
            if (s > 0) best = wave_max_int_dpp(k0);
            const int bi = __ffsll((long long)__ballot(k0 == best)) - 1;
            if (lane == bi) k0 = NO_EXPERT;
            if (lane == s) { my_idx = bi; my_best = best; }
        }
    }
    // the k scores at once, one per lane
    my_p = expf(key_logit(my_best) - m) / den;
    sel = 0.f;
    for (int s = 0; s < k; ++s) sel += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_p), s));
}

// Weight of a sigmoid-gated shared expert for one token, by one wavefront: c = 1 / (1 + exp(-(x . w_sg))).  One
// definition for every caller, so the value does not depend on which kernel evaluates it.
__device__ __forceinline__ float sigmoid_gate_of(const uint16_t *__restrict__ x, const uint16_t *__restrict__ w_sg, int d, int lane)
{
    float acc = 0.f;
    for (int j = lane * 8; j < d; j += 512) {
        uint4 a = *reinterpret_cast<const uint4 *>(x + j);
        uint4 b = *reinterpret_cast<const uint4 *>(w_sg + j);
        acc = fmaf(bf16_lo(a.x), bf16_lo(b.x), acc); acc = fmaf(bf16_hi(a.x), bf16_hi(b.x), acc);
        acc = fmaf(bf16_lo(a.y), bf16_lo(b.y), acc); acc = fmaf(bf16_hi(a.y), bf16_hi(b.y), acc);
        acc = fmaf(bf16_lo(a.z), bf16_lo(b.z), acc); acc = fmaf(bf16_hi(a.z), bf16_hi(b.z), acc);
        acc = fmaf(bf16_lo(a.w), bf16_lo(b.w), acc); acc = fmaf(bf16_hi(a.w), bf16_hi(b.w), acc);
    }
    acc = wave_sum(acc);
    return 1.0f / (1.0f + expf(-acc));
}

// Outputs of the wider layer (N + S experts, k + S slots per token: the S always-on shared experts appended, as
// append_shared_kernel writes them) that the selecting block of a decode-sized batch can write itself; S = 0: none.
struct shared_tail {
    int S, d;
    const uint16_t *h, *w_sg;          // w_sg null: weight 1
    float *gate;                       // [T] the sigmoid gates, by a plane of the gate launch; null: evaluated by the selecting block
    int32_t *x_idx;
    float *x_w;
    int32_t *x_counts, *x_offsets, *x_perm, *x_inv;
};

// Histogram, scan and stable permutation of a decode-sized batch (T <= 16, R = T*k <= 128 selections in sel_idx, LDS)
// by one block.  A token selects an expert at most once, so the rows of expert e are one per selecting token, in
// token order: a 16-bit token mask per expert gives the workload (its popcount) and the rank of a row within its
// expert (the popcount below the token's bit) without any serial pass.  With perm == nullptr (a prediction) the
// workloads and the p largest of them are written instead.  Every thread of the block must call it.
// With X.S > 0 (routing only) the tables of the layer with its shared experts appended follow from the same LDS state:
// sel_w holds the combine weights of the R selections, cs is room for T floats.  What depends on the thread alone is worked
// out beforehand (decode_prep), while the logits are on their way.
struct decode_prep {
    int t, s;             // token and slot of selection threadIdx.x
    int xj, xt;           // shared expert and token of the appended slot threadIdx.x
    float xc;             // its weight, where that is known beforehand
};
__device__ __forceinline__ decode_prep decode_prepare(int T, int k, const shared_tail &X)
{
    decode_prep p;
    p.t = threadIdx.x / k;
    p.s = threadIdx.x - p.t * k;
    p.xj = threadIdx.x / T;
    p.xt = threadIdx.x - p.xj * T;
    p.xc = X.S > 0 && X.w_sg != nullptr && X.gate != nullptr ? X.gate[p.xt] : 1.0f;
    return p;
}
__device__ __forceinline__ void decode_tables(const int *sel_idx, unsigned *tokmask, int *off_s, int T, int N, int k,
                                              int32_t *__restrict__ counts, int32_t *__restrict__ offsets,
                                              int32_t *__restrict__ perm, int32_t *__restrict__ inv_perm,
                                              int32_t *__restrict__ top, int p, const float *sel_w, float *cs,
                                              const shared_tail &X, const decode_prep &D)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int R = T * k;
    if (threadIdx.x < MOE_MAX_EXPERTS) tokmask[threadIdx.x] = 0u;
    __syncthreads();
    int my_e = -1, my_t = 0;
    if ((int)threadIdx.x < R) {
        my_e = sel_idx[threadIdx.x];
        my_t = D.t;
        atomicOr(&tokmask[my_e], 1u << my_t);
    }
    __syncthreads();
    if (wave == 0) {
        // workloads of experts lane and lane + 64, and their exclusive prefix sums over all 128 slots
        const int c0 = lane < N ? __popc(tokmask[lane]) : 0;
        const int c1 = lane + 64 < N ? __popc(tokmask[lane + 64]) : 0;
        int s0 = c0, s1 = c1;
        const int tot0 = wave_scan_int_dpp(s0);
        if (N > 64) wave_scan_int_dpp(s1);
        if (lane < N) counts[lane] = c0;
        if (lane + 64 < N) counts[lane + 64] = c1;
        if (perm == nullptr) {
            // prediction: the workloads and the p largest of them (equal workloads by ascending index)
            top_p_of(c0, c1, N, p, top, lane);
        } else {
            off_s[lane] = s0 - c0;
            off_s[lane + 64] = tot0 + s1 - c1;
            if (lane < N) offsets[lane] = s0 - c0;
            if (lane + 64 < N) offsets[lane + 64] = tot0 + s1 - c1;
            if (lane == 0) offsets[N] = R;
        }
    }
    if (perm == nullptr) return;
    __syncthreads();
    int pos = 0;
    if ((int)threadIdx.x < R) {
        pos = off_s[my_e] + __popc(tokmask[my_e] & ((1u << my_t) - 1u));
        perm[pos] = threadIdx.x;
        inv_perm[threadIdx.x] = pos;
    }
    if (X.S <= 0) return;
    // ---- the same layer as N + S experts with k + S slots per token (what append_shared_kernel derives from the tables)
    const int S = X.S, kx = k + S, tid = threadIdx.x, nthreads = blockDim.x;
    const bool gates_here = X.w_sg != nullptr && X.gate == nullptr;
    if (gates_here) {
        for (int t = wave; t < T; t += nthreads >> 6) {
            const float c = sigmoid_gate_of(X.h + (size_t)t * X.d, X.w_sg, X.d, lane);
            if (lane == 0) cs[t] = c;
        }
        __syncthreads();
    }
    if (tid < R) {                                             // routed slots keep their order; slot ids move to the wider stride
        const int o = my_t * kx + D.s;
        X.x_idx[o] = my_e;
        X.x_w[o] = sel_w[tid];
        X.x_inv[o] = pos;
        X.x_perm[pos] = tid + my_t * S;
    }
    if (tid < T * S) {                                         // shared expert j takes slot k + j of every token
        const int o = D.xt * kx + k + D.xj, row = R + tid;
        X.x_idx[o] = N + D.xj;
        X.x_w[o] = gates_here ? cs[D.xt] : D.xc;
        X.x_inv[o] = row;
        X.x_perm[row] = o;
    }
    for (int e = tid; e < N + S; e += nthreads) {
        X.x_counts[e] = e < N ? __popc(tokmask[e]) : T;
        X.x_offsets[e] = e < N ? off_s[e] : R + (e - N) * T;
    }
    if (tid == 0) X.x_offsets[N + S] = R + S * T;
}

// One gate to evaluate: the layer's own (routing) or the next layer's (prediction).  A launch carries two jobs and
// blockIdx.z picks one, so that a decode step can route and predict in the same pair of launches.
struct gate_job {
    const uint16_t *gate_w;    // [N,d] bf16
    const float *bias;         // [N] or null
    const float *res_vec;      // non-null: add res_vec . W[e] to the logit of expert e
    int norm_mode;
    int32_t *topk_idx;         // [T,k]
    float *topk_w;             // [T,k]
    int32_t *counts;           // non-null: single-block launch that also does the histogram (and, with perm, scan and permutation)
    int32_t *offsets, *perm, *inv_perm;
    float *logits;             // [T,N] between gate_logits_kernel and the kernel that selects
    int32_t *top;              // with counts and without perm: the p largest workloads
    int p;
    shared_tail x;             // x.S > 0 (with perm, decode-sized launches only): also write the tables with the shared experts appended
};

// picked by index, so that a block reads the one it works on: with the choice between two arguments every field of both
// was held in scalar registers and some spilled
struct gate_jobs {
    gate_job job[2];
};

// Eight elements of row `part` of the residual's exact split x = hi + mid + lo into bf16 numbers (8 bits of its 24 each, cut off,
// so that both differences are exact).  What is not finite stays in hi.
__device__ __forceinline__ u32x4 residual_rows(float4 r0, float4 r1, int part)
{
    const float x[8] = {r0.x, r0.y, r0.z, r0.w, r1.x, r1.y, r1.z, r1.w};
    u32x4 o;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        uint32_t w[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const float v = x[2 * j + q];
            const bool finite = __builtin_fabsf(v) < __builtin_huge_valf();
            uint32_t hi = __float_as_uint(v) & 0xffff0000u;
            if (v != v) hi = 0x7fc00000u;
            const float rem = finite ? v - __uint_as_float(hi) : 0.f;
            const uint32_t mid = __float_as_uint(rem) & 0xffff0000u;
            const uint32_t lo = __float_as_uint(rem - __uint_as_float(mid));
            w[q] = part == 0 ? hi : part == 1 ? mid : lo;
        }
        o[j] = w[0] >> 16 | (w[1] & 0xffff0000u);
    }
    return o;
}

// res_vec . W from the products of its three parts.  Where the first is not finite it is the whole result: hi is zero only where the
// residual is (or is below the smallest bf16 number), the lower parts are zero wherever hi is exact, and zero times an infinite
// weight would turn the infinity into NaN.
__device__ __forceinline__ float residual_sum(float hi, float mid, float lo)
{
    return __builtin_fabsf(hi) < __builtin_huge_valf() ? (lo + mid) + hi : hi;
}

// 16 rows x 32 k, lane l holding chunk l % 4 of row l / 4, to an MFMA operand (row l % 16, chunk l / 16); from_lane: four times the
// lane this one's data comes from
__device__ __forceinline__ bf16x8 rows_to_frag(u32x4 v, int from_lane)
{
    u32x4 o;
#pragma unroll
    for (int j = 0; j < 4; ++j) o[j] = (uint32_t)__builtin_amdgcn_ds_bpermute(from_lane, (int)v[j]);
    return as_frag(o);
}

// The gate product of one block: 16 token rows (with a residual vector 13 and its three rows) times the 16 NT experts from e_base.
// Rows are read four lanes to a row, 64 contiguous bytes, and put into fragment order by a lane permutation: read in
// fragment order (neighbouring lanes in different rows) every lane is an access of its own, 38 GB/s per compute unit against 147
// from L2 and 30 against 58 from HBM.  K is cut into ROUTE_SEGS runs by d alone and the sums of the runs are added as a tree, so
// that a logit is the same number whatever the batch size and the number of jobs.
// RES: how the rows of a residual vector are held, if the gate has one.
template <int NT, int RES> struct gate_tile {
    static constexpr int NP = NT * 16;                       // padded expert count
    static constexpr int G = NT <= 4 ? NT : 4;               // expert groups of a wave, ...
    static constexpr int KW = NT <= 4 ? 16 : 8;              // ... waves K is dealt to, ...
    static constexpr int SEGS = ROUTE_SEGS / KW;             // ... runs of a wave
    static constexpr int ROWS = RES == RES_BESIDE ? ROUTE_TOKENS + 3 : ROUTE_TOKENS;
    static constexpr int RES_ROW = RES == RES_BESIDE ? ROUTE_TOKENS : FOLD_ROW;
    const char *hb, *wb;
    const float *res_vec;
    uint32_t wo[G];                                          // byte offsets: T*d < 2^31 elements keeps them in 32 bits
    int T, d, nsteps, per, kw, g0, row, chunk, frag_lane;

    __device__ __forceinline__ gate_tile(int T_, int d_, int N, const uint16_t *h, const gate_job &J, int e_base)
    {
        const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        T = T_;
        d = d_;
        hb = reinterpret_cast<const char *>(h);
        wb = reinterpret_cast<const char *>(J.gate_w);
        res_vec = RES != RES_NONE ? J.res_vec : nullptr;
        kw = wave % KW;
        g0 = wave / KW * G;
        row = lane >> 2;
        chunk = lane & 3;
        frag_lane = ((lane & 15) * 4 + (lane >> 4)) * 4;
        nsteps = d >> 5;
        per = (nsteps + ROUTE_SEGS - 1) / ROUTE_SEGS;
#pragma unroll
        for (int j = 0; j < G; ++j) wo[j] = ((uint32_t)min(e_base + (g0 + j) * 16 + row, N - 1) * (uint32_t)d + chunk * 8) * 2u;
    }
    __device__ __forceinline__ bool fold_row() const { return RES == RES_IN_TILE && res_vec != nullptr && row >= FOLD_ROW; }
    __device__ __forceinline__ uint32_t row_offset(int t0) const { return ((uint32_t)min(t0 + row, T - 1) * (uint32_t)d + chunk * 8) * 2u; }
    // n steps from s on (a step beyond the last one reads that again); along the rows first: the halves of a line follow each other
    template <int n> __device__ __forceinline__ void load_tokens(u32x4 (&a)[n], int t0, int s, int last) const
    {
        const uint32_t ho = row_offset(t0);
        if (!fold_row()) {
#pragma unroll
            for (int u = 0; u < n; ++u) a[u] = *reinterpret_cast<const u32x4 *>(hb + ho + min(s + u, last) * 64);
        }
    }
    template <int n> __device__ __forceinline__ void load_residual(u32x4 (&a)[n], int s, int last) const
    {
        if (fold_row()) {
#pragma unroll
            for (int u = 0; u < n; ++u) {
                const float4 *r = reinterpret_cast<const float4 *>(res_vec + min(s + u, last) * 32 + chunk * 8);
                a[u] = residual_rows(r[0], r[1], row - FOLD_ROW);
            }
        }
    }
    template <int n> __device__ __forceinline__ void load_gate(u32x4 (&b)[n][G], int s, int last) const
    {
#pragma unroll
        for (int j = 0; j < G; ++j)
#pragma unroll
            for (int u = 0; u < n; ++u) b[u][j] = *reinterpret_cast<const u32x4 *>(wb + wo[j] + min(s + u, last) * 64);
    }
    __device__ __forceinline__ bf16x8 gate_frag(bf16x8 b) const { return b; }
    __device__ __forceinline__ bf16x8 gate_frag(u32x4 b) const { return rows_to_frag(b, frag_lane); }
    // b: gate rows as loaded, or fragments
    template <int n, class B> __device__ __forceinline__ void mfmas(f32x4 (&acc)[G], const u32x4 (&a)[n], const B (&b)[n][G], int steps) const
    {
#pragma unroll
        for (int u = 0; u < n; ++u) {
            if (u >= steps) break;                           // uniform
            const bf16x8 af = rows_to_frag(a[u], frag_lane);
#pragma unroll
            for (int j = 0; j < G; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, gate_frag(b[u][j]), acc[j], 0, 0, 0);
        }
    }
    // the steps [s, s_end) of a run, n on their way at once
    template <int n> __device__ __forceinline__ void walk(f32x4 (&acc)[G], int t0, int s, int s_end) const
    {
        for (; s < s_end; s += n) {
            u32x4 a[n], b[n][G];
            load_tokens(a, t0, s, s_end - 1);
            load_gate(b, s, s_end - 1);
            load_residual(a, s, s_end - 1);
            __builtin_amdgcn_sched_barrier(0);               // every load of the batch is on its way
            mfmas(acc, a, b, s_end - s);
        }
    }
    // the same for the only run of a wave, with the residual's rows beside the tokens: lane l converts elements 8l .. 8l + 7 of the run
    // (512 at most) while the tokens and gate rows are on their way; rr, of this wave's own, holds them as chunks of the three parts
    template <int n> __device__ __forceinline__ void walk_beside(f32x4 (&acc)[G], f32x4 (&res)[G], u32x4 (&rr)[3][64], int t0, int s0, int s_end) const
    {
        const int lane = threadIdx.x & 63, r = lane & 15, c = lane >> 4;
        const bool mine = res_vec != nullptr && lane < (s_end - s0) * 4;
        float4 r0, r1;
        if (mine) {
            r0 = *reinterpret_cast<const float4 *>(res_vec + s0 * 32 + lane * 8);
            r1 = *reinterpret_cast<const float4 *>(res_vec + s0 * 32 + lane * 8 + 4);
        }
        for (int s = s0; s < s_end; s += n) {
            u32x4 a[n], b[n][G];
            load_tokens(a, t0, s, s_end - 1);
            load_gate(b, s, s_end - 1);
            __builtin_amdgcn_sched_barrier(0);
            if (mine && s == s0) {
#pragma unroll
                for (int p = 0; p < 3; ++p) rr[p][lane] = residual_rows(r0, r1, p);
            }
            // the lanes of a wave exchange data: LDS serves a wave's accesses in order, the compiler keeps theirs
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
            for (int u = 0; u < n; ++u) {
                if (s + u >= s_end) break;                   // uniform
                const bf16x8 af = rows_to_frag(a[u], frag_lane);
                u32x4 rf = u32x4{0, 0, 0, 0};
                if (res_vec != nullptr && r < 3) rf = rr[r][(s + u - s0) * 4 + c];
#pragma unroll
                for (int j = 0; j < G; ++j) {
                    const bf16x8 bf = gate_frag(b[u][j]);
                    acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, bf, acc[j], 0, 0, 0);
                    res[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_frag(rf), bf, res[j], 0, 0, 0);
                }
            }
        }
    }
    __device__ __forceinline__ void store(float (&part)[ROUTE_SEGS][ROWS][NP + 1], int seg, const f32x4 (&acc)[G]) const
    {
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int j = 0; j < G; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (g0 + j < NT) part[seg][4 * (lane >> 4) + r][(g0 + j) * 16 + (lane & 15)] = acc[j][r];
    }
    __device__ __forceinline__ void store_res(float (&part)[ROUTE_SEGS][ROWS][NP + 1], int seg, const f32x4 (&res)[G]) const
    {
        const int lane = threadIdx.x & 63;
        if (lane >= 16) return;                              // rows 0 .. 3 of the result
#pragma unroll
        for (int j = 0; j < G; ++j)
#pragma unroll
            for (int r = 0; r < 3; ++r) part[seg][RES_ROW + r][(g0 + j) * 16 + lane] = res[j][r];
    }
    // the sums of the runs; ends with a barrier
    static __device__ __forceinline__ void reduce(const float (&part)[ROUTE_SEGS][ROWS][NP + 1], float (&lg)[ROWS][NP + 4])
    {
        for (int idx = threadIdx.x; idx < ROWS * NP; idx += ROUTE_THREADS) {
            const int tt = idx / NP, e = idx % NP;
            float v[ROUTE_SEGS];
#pragma unroll
            for (int w = 0; w < ROUTE_SEGS; ++w) v[w] = part[w][tt][e];
#pragma unroll
            for (int o = 1; o < ROUTE_SEGS; o *= 2)
#pragma unroll
                for (int w = 0; w < ROUTE_SEGS; w += 2 * o) v[w] += v[w + o];
            lg[tt][e] = v[0];
        }
        __syncthreads();
    }
    // logit of a token's row: the bias with the residual vector folded in is added, (h + res_vec).W + b = h.W + (res_vec.W + b)
    __device__ __forceinline__ float logit(const float (&lg)[ROWS][NP + 4], const float (&bias_s)[NP], int tt, int e) const
    {
        float b = bias_s[e];
        if (RES != RES_NONE && res_vec != nullptr) b = residual_sum(lg[RES_ROW][e], lg[RES_ROW + 1][e], lg[RES_ROW + 2][e]) + b;
        return lg[tt][e] + b;
    }
    static __device__ __forceinline__ void load_bias(float (&bias_s)[NP], const float *bias, int e_base, int N)
    {
        const int e = threadIdx.x;
        if (e < NP) bias_s[e] = bias != nullptr && e_base + e < N ? bias[e_base + e] : 0.f;
    }
};

// Logits of 16 NT experts per blockIdx.y.  Bound by the latency of its reads at decode sizes and by what one compute unit takes in
// beyond: a block keeps its gate rows in registers (all of them up to d = 2048) and walks token tiles, so that the gate matrix is
// read once per block, not once per 16 tokens.  KEEP: how many of its run's steps a wave keeps, no more than a run has: with four of
// a run of one, each with the residual's conversion, a decode prediction took 8.7 us, now 6.6 (d = 256, 64 experts; 4096 tokens 17.3 / 14.3).  With fragment-order reads by 8 waves (16 x 32 tiles, the residual folded by waves of
// their own) and now: 16 tokens of 64 experts 5.7 / 4.6 us, 16 of two gates of 128 with a residual 8.2 / 6.3, 77 of 128 8.0 / 5.4,
// 2048 of 64 10.4 / 7.3, 4096 of 60 17.3 / 9.8, 1531 of two gates of 128 22 / 13.6 (d = 2048).
template <int NT, int KEEP>
__global__ __launch_bounds__(ROUTE_THREADS) void gate_logits_kernel(int T, int d, int N, const uint16_t *__restrict__ h, gate_jobs jobs)
{
    const gate_job &J = jobs.job[blockIdx.z == 0 ? 0 : 1];
    if (J.x.gate != nullptr && blockIdx.z == gridDim.z - 1) {
        // the sigmoid gates of the shared experts, one wave per token
        const int t = threadIdx.x >> 6, lane = threadIdx.x & 63;
        if (blockIdx.y == 0 && t < T) {
            const float c = sigmoid_gate_of(h + (size_t)t * d, J.x.w_sg, d, lane);
            if (lane == 0) J.x.gate[t] = c;
        }
        return;
    }
    const int tokens = J.res_vec != nullptr ? FOLD_ROW : ROUTE_TOKENS;
    int t0 = blockIdx.x * tokens;
    if (t0 >= T) return;
    constexpr int NP = NT * 16;
    __shared__ float part[ROUTE_SEGS][ROUTE_TOKENS][NP + 1];    // partial logits
    __shared__ __attribute__((aligned(16))) float lg[ROUTE_TOKENS][NP + 4];   // reduced logits, rows 16-byte aligned
    __shared__ float bias_s[NP];
    const int e_base = blockIdx.y * NP;
    const gate_tile<NT, RES_IN_TILE> G(T, d, N, h, J, e_base);
    static_assert(G.SEGS == 1, "one run per wave");
    const int s0 = G.kw * G.per, s_end = min(s0 + G.per, G.nsteps), last = max(min(s_end, G.nsteps) - 1, 0);
    u32x4 a[KEEP], b[KEEP][G.G];
    G.load_tokens(a, t0, s0, last);
    G.load_gate(b, s0, last);
    G.load_residual(a, s0, last);
    G.load_bias(bias_s, J.bias, e_base, N);
    bf16x8 bf[KEEP][G.G];
#pragma unroll
    for (int u = 0; u < KEEP; ++u)
#pragma unroll
        for (int j = 0; j < G.G; ++j) bf[u][j] = rows_to_frag(b[u][j], G.frag_lane);
    float *__restrict__ out = J.logits;
    for (; t0 < T; t0 += gridDim.x * tokens) {
        f32x4 acc[G.G];
#pragma unroll
        for (int j = 0; j < G.G; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        G.mfmas(acc, a, bf, s_end - s0);
        G.template walk<2>(acc, t0, s0 + KEEP, s_end);
        G.store(part, G.kw, acc);
        G.load_tokens(a, t0 + gridDim.x * tokens, s0, last);     // of the next tile (of the last token beyond the last tile)
        __syncthreads();
        G.reduce(part, lg);
        const int n = min(tokens, T - t0) * NP;
        for (int idx = threadIdx.x; idx < n; idx += ROUTE_THREADS) {
            const int tt = idx / NP, e = idx % NP;
            if (e_base + e < N) out[(size_t)(t0 + tt) * N + e_base + e] = G.logit(lg, bias_s, tt, e);
        }
    }
}

// Gate and selection of 16 tokens, NT = ceil(N / 16); with TABLES (a decode-sized batch, one block) the tables too.  (One kernel for
// all held the fields of every path in scalar registers and spilled them.)  Before and now, d = 4096, 8 experts: 200 tokens 10.9 /
// 7.8 us, 8192 23 / 19.
// RES_BESIDE where the gate may have a residual: with 13 tokens to a block, 4096 of them are 316 blocks for 256 compute units.  Prediction,
// RES_IN_TILE / RES_BESIDE, d = 4096, 8 experts: 17 tokens 10.8 / 9.5 us, 4096 21 / 14.5, 16384 50 / 41; d = 2048, 48 experts: 4096 21 / 14.4.
// With up to 16 experts two blocks of 64 registers per lane share a compute unit (20 bytes spill; one of 66: 16384 tokens 45 us).
template <int NT, bool TABLES, int RES>
__global__ __launch_bounds__(ROUTE_THREADS, !TABLES && RES == RES_BESIDE && NT == 1 ? 8 : 4) void gate_topk_kernel(
    int T, int d, int N, int k, const uint16_t *__restrict__ h, gate_jobs jobs)
{
    const gate_job &J = jobs.job[blockIdx.z == 0 ? 0 : 1];
    const int t0 = blockIdx.x * ROUTE_TOKENS;
    if (t0 >= T) return;
    constexpr int NP = NT * 16;
    typedef gate_tile<NT, RES> tile;
    __shared__ float part[ROUTE_SEGS][tile::ROWS][NP + 1];
    __shared__ __attribute__((aligned(16))) float lg[tile::ROWS][NP + 4];
    __shared__ float bias_s[NP];
    const tile G(T, d, N, h, J, 0);
    G.load_bias(bias_s, J.bias, 0, N);
    for (int seg = G.kw * G.SEGS; seg < (G.kw + 1) * G.SEGS; ++seg) {
        f32x4 acc[G.G];
#pragma unroll
        for (int j = 0; j < G.G; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        const int s0 = seg * G.per, s_end = min((seg + 1) * G.per, G.nsteps);
        if constexpr (RES == RES_BESIDE) {
            static_assert(G.SEGS == 1, "one run per wave");
            __shared__ u32x4 rr[ROUTE_SEGS][3][64];
            f32x4 res[G.G];
#pragma unroll
            for (int j = 0; j < G.G; ++j) res[j] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (TABLES && G.per > 2) G.template walk_beside<8>(acc, res, rr[seg], t0, s0, s_end);
            else G.template walk_beside<TABLES ? 2 : 4>(acc, res, rr[seg], t0, s0, s_end);
            G.store_res(part, seg, res);
        } else {
            G.template walk<TABLES && NT == 1 ? 8 : NT <= 3 ? 4 : 2>(acc, t0, s0, s_end);
        }
        G.store(part, seg, acc);
    }
    __syncthreads();
    G.reduce(part, lg);

    // softmax + top-k: one wave per token, lane l owns experts l and l + 64
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (wave < min(ROUTE_TOKENS, T - t0)) {
        const int t = t0 + wave;
        const float v0 = G.logit(lg, bias_s, wave, min(lane, N - 1));
        const float v1 = NT > 4 ? G.logit(lg, bias_s, wave, min(lane + 64, N - 1)) : v0;
        int my_idx;
        float my_p, sel;
        select_token(v0, v1, N, k, lane, my_idx, my_p, sel);
        if (lane < k) {
            const float wgt = J.norm_mode == MOE_NORM_RENORM ? my_p / sel : my_p;
            J.topk_idx[(size_t)t * k + lane] = my_idx;
            J.topk_w[(size_t)t * k + lane] = wgt;
            if (TABLES) {
                reinterpret_cast<int *>(&part[0][0][0])[wave * k + lane] = my_idx;
                (&part[1][0][0])[wave * k + lane] = wgt;
            }
        }
    }
    if constexpr (!TABLES) return;
    __syncthreads();
    __shared__ unsigned tokmask[MOE_MAX_EXPERTS];
    __shared__ int off_s[MOE_MAX_EXPERTS];
    decode_tables(reinterpret_cast<const int *>(&part[0][0][0]), tokmask, off_s, T, N, k, J.counts, J.offsets, J.perm, J.inv_perm, J.top, J.p,
                  &part[1][0][0], &part[2][0][0], J.x, decode_prepare(T, k, J.x));
}

// Selection for a decode-sized batch from stored logits [T, N] (bias already added): one wavefront per token, then
// the tables of decode_tables.  One block of 16 waves per job (blockIdx.z).
#define SELECT_THREADS 1024
__global__ __launch_bounds__(SELECT_THREADS) void select_decode_kernel(int T, int N, int k, gate_jobs jobs)
{
    const gate_job &J = jobs.job[blockIdx.z == 0 ? 0 : 1];
    __shared__ int sel_idx[ROUTE_TOKENS * MOE_MAX_TOPK];
    __shared__ float sel_w[ROUTE_TOKENS * MOE_MAX_TOPK], cs[ROUTE_TOKENS];
    __shared__ unsigned tokmask[MOE_MAX_EXPERTS];
    __shared__ int off_s[MOE_MAX_EXPERTS];
    const int lane = threadIdx.x & 63, t = threadIdx.x >> 6;
    // all arguments at once: read where they are used, each line of them is a round trip of its own (0.4 us)
    asm volatile("" ::"s"(J.topk_idx), "s"(J.topk_w), "s"(J.counts), "s"(J.offsets), "s"(J.perm), "s"(J.inv_perm), "s"(J.norm_mode), "s"(J.x.S),
                 "s"(J.x.gate), "s"(J.x.x_idx), "s"(J.x.x_w), "s"(J.x.x_counts), "s"(J.x.x_offsets), "s"(J.x.x_perm), "s"(J.x.x_inv));
    const float *row = J.logits + (size_t)min(t, T - 1) * N;
    const float v0 = row[min(lane, N - 1)], v1 = row[min(lane + 64, N - 1)];
    const decode_prep prep = decode_prepare(T, k, J.x);
    if (t < T) {
        int my_idx;
        float my_p, sel;
        select_token(v0, v1, N, k, lane, my_idx, my_p, sel);
        if (lane < k) {
            J.topk_idx[(size_t)t * k + lane] = my_idx;
            const float wgt = J.norm_mode == MOE_NORM_RENORM ? my_p / sel : my_p;
            J.topk_w[(size_t)t * k + lane] = wgt;
            sel_idx[t * k + lane] = my_idx;
            sel_w[t * k + lane] = wgt;
        }
    }
    __syncthreads();
    decode_tables(sel_idx, tokmask, off_s, T, N, k, J.counts, J.offsets, J.perm, J.inv_perm, J.top, J.p, sel_w, cs, J.x, prep);
}

// Selection from stored logits [T, N] for any batch size: one wavefront per token, 16 tokens per block.
__global__ __launch_bounds__(SELECT_THREADS) void select_rows_kernel(int T, int N, int k, gate_jobs jobs)
{
    const gate_job &J = jobs.job[blockIdx.z == 0 ? 0 : 1];
    const int lane = threadIdx.x & 63;
    const int t = blockIdx.x * (SELECT_THREADS / 64) + (threadIdx.x >> 6);
    if (t >= T) return;
    const float *row = J.logits + (size_t)t * N;
    const float v0 = row[min(lane, N - 1)], v1 = row[min(lane + 64, N - 1)];
    int my_idx;
    float my_p, sel;
    select_token(v0, v1, N, k, lane, my_idx, my_p, sel);
    if (lane < k) {
        J.topk_idx[(size_t)t * k + lane] = my_idx;
        J.topk_w[(size_t)t * k + lane] = J.norm_mode == MOE_NORM_RENORM ? my_p / sel : my_p;
    }
}

// ---------------------------------------------------------------------------------------------------
// A prediction's histogram: R selections idx, the N workloads and the p largest of them.
struct top_job {
    const int32_t *idx;
    int32_t *pred_counts, *top;
    int p;
};

// Workload histogram of R predicted selections and its p largest entries.  One block of 16 wavefronts, each with a
// private LDS histogram (one shared set of 128 bins serialises on the popular experts), summed in wave order.
#define HT_THREADS 1024
#define HT_BATCH 8           // selections on their way per thread, so that 8192 of them cost one read latency
__device__ __forceinline__ void hist_top_block(int R, int N, const top_job &J)
{
    __shared__ int sub[HT_THREADS / 64][MOE_MAX_EXPERTS];
    __shared__ int hist[MOE_MAX_EXPERTS];
    const int wave = threadIdx.x >> 6;
    for (int j = threadIdx.x; j < (HT_THREADS / 64) * MOE_MAX_EXPERTS; j += HT_THREADS) (&sub[0][0])[j] = 0;
    __syncthreads();
    for (int r0 = threadIdx.x; r0 < R; r0 += HT_BATCH * HT_THREADS) {
        int v[HT_BATCH];
#pragma unroll
        for (int j = 0; j < HT_BATCH; ++j) v[j] = r0 + j * HT_THREADS < R ? J.idx[r0 + j * HT_THREADS] : -1;
#pragma unroll
        for (int j = 0; j < HT_BATCH; ++j)
            if (v[j] >= 0) atomicAdd(&sub[wave][v[j] & (MOE_MAX_EXPERTS - 1)], 1);
    }
    __syncthreads();
    if (threadIdx.x < MOE_MAX_EXPERTS) {
        int c = 0;
#pragma unroll
        for (int w = 0; w < HT_THREADS / 64; ++w) c += sub[w][threadIdx.x];
        hist[threadIdx.x] = c;
        if ((int)threadIdx.x < N) J.pred_counts[threadIdx.x] = c;
    }
    __syncthreads();
    if (threadIdx.x < 64) top_p_of(hist[threadIdx.x], hist[threadIdx.x + 64], N, J.p, J.top, threadIdx.x);
}

__global__ __launch_bounds__(HT_THREADS) void hist_top_kernel(int R, int N, top_job J) { hist_top_block(R, N, J); }

// One block of 16 waves per expert e.  Every wave takes a contiguous run of 64 PT selections, so that its workload is the
// popcount of PT ballots and one number per wave is all the block has to exchange: the selections below e (their
// block-wide sum is offsets[e]) and equal to e (counts[e], and the positions of a wave's rows).  No global zero-fill, no
// cross-block atomics, stable and the same on every run.  R up to 1024 PT selections stay in registers between counting and
// placing; more are read a second time, 16 K at a time.
// What bounds it is latency (a launch, two dependent reads, one barrier), so PT follows R: with 64 entries a thread whatever
// R was, 400 selections of 8 experts took 12.4 us and 12288 of 64 took 14.3 us; now 4.9 and 5.5 us.
#define HSP_THREADS 1024
#define HSP_WAVES (HSP_THREADS / 64)
template <int PT>
__global__ __launch_bounds__(HSP_THREADS) void hist_scan_perm_kernel(
    int R, int N, const int32_t *__restrict__ topk_idx, int32_t *__restrict__ counts,
    int32_t *__restrict__ offsets, int32_t *__restrict__ perm, int32_t *__restrict__ inv_perm, top_job top /* block N, if any */)
{
    static_assert(HSP_THREADS == HT_THREADS, "one block size for both");
    if ((int)blockIdx.x == N) {
        hist_top_block(R, N, top);
        return;
    }
    __shared__ int tot[2][HSP_WAVES];
    const int e = blockIdx.x;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    constexpr int SUPER = HSP_THREADS * PT;

    // entry j of this thread in super-chunk c0: r = c0 + wave * 64 PT + j * 64 + lane
    int v[PT];
    auto load_super = [&](int c0) {
#pragma unroll
        for (int j = 0; j < PT; ++j) {
            const int r = c0 + (wave * PT + j) * 64 + lane;
            v[j] = r < R ? topk_idx[r] : -1;
        }
    };
    int below = 0, equal = 0;                               // of this wave, uniform
    for (int c0 = 0; c0 < R; c0 += SUPER) {
        load_super(c0);
#pragma unroll
        for (int j = 0; j < PT; ++j) {
            below += __popcll(__ballot((unsigned)v[j] < (unsigned)e));   // padding entries are -1 = huge unsigned
            equal += __popcll(__ballot(v[j] == e));
        }
    }
    if (lane == 0) { tot[0][wave] = below; tot[1][wave] = equal; }
    __syncthreads();
    int off = 0, cnt = 0, before = 0;                       // before: rows of e in the waves below this one
#pragma unroll
    for (int w = 0; w < HSP_WAVES; ++w) {
        off += tot[0][w];
        before += w < wave ? tot[1][w] : 0;
        cnt += tot[1][w];
    }
    if (threadIdx.x == 0) {
        counts[e] = cnt;
        offsets[e] = off;
        if (e == N - 1) offsets[N] = off + cnt;
    }
    const unsigned long long lower = (1ull << lane) - 1ull;
    auto place = [&](int c0, int pos) {
#pragma unroll
        for (int j = 0; j < PT; ++j) {
            const unsigned long long b = __ballot(v[j] == e);
            if (v[j] == e) {
                const int r = c0 + (wave * PT + j) * 64 + lane;
                const int p = pos + __popcll(b & lower);
                perm[p] = r;
                inv_perm[r] = p;
            }
            pos += __popcll(b);
        }
    };
    if (R <= SUPER) {
        place(0, off + before);
        return;
    }
    for (int c0 = 0; c0 < R; c0 += SUPER) {                 // off: running output position of the super-chunk, uniform
        load_super(c0);
        equal = 0;
#pragma unroll
        for (int j = 0; j < PT; ++j) equal += __popcll(__ballot(v[j] == e));
        __syncthreads();                                    // the totals of the chunk before have been read
        if (lane == 0) tot[1][wave] = equal;
        __syncthreads();
        before = cnt = 0;
#pragma unroll
        for (int w = 0; w < HSP_WAVES; ++w) {
            before += w < wave ? tot[1][w] : 0;
            cnt += tot[1][w];
        }
        place(c0, off + before);
        off += cnt;
    }
}

// top: the histogram of a prediction of the same size in the same launch, or null
static int launch_hist_scan_perm(int R, int N, const int32_t *topk_idx, int32_t *counts, int32_t *offsets, int32_t *perm,
                                 int32_t *inv_perm, const top_job *top, hipStream_t st)
{
    const top_job none = {};
#define HSP(pt)                                                                                                        \
    hipLaunchKernelGGL(hist_scan_perm_kernel<pt>, dim3(N + (top != nullptr ? 1 : 0)), dim3(HSP_THREADS), 0, st, R, N, topk_idx, \
                       counts, offsets, perm, inv_perm, top != nullptr ? *top : none)
    if (R <= HSP_THREADS) HSP(1);
    else if (R <= 4 * HSP_THREADS) HSP(4);
    else HSP(16);
#undef HSP
    MOE_CHECK_LAUNCH();
    return MOE_OK;
}

// ---------------------------------------------------------------------------------------------------
__global__ void dense_route_kernel(int T, int S, int32_t *__restrict__ counts, int32_t *__restrict__ offsets,
                                   int32_t *__restrict__ perm)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p < T * S) {
        int e = p / T, t = p - e * T;
        perm[p] = t * S + e;
    }
    if (p < S) { counts[p] = T; offsets[p] = p * T; }
    if (p == 0) offsets[S] = S * T;
}

__global__ __launch_bounds__(256) void shared_gate_kernel(int T, int d, const uint16_t *__restrict__ h,
                                                          const uint16_t *__restrict__ w_sg, float *__restrict__ scale)
{
    const int lane = threadIdx.x & 63;
    const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (t >= T) return;
    const float c = sigmoid_gate_of(h + (size_t)t * d, w_sg, d, lane);
    if (lane == 0) scale[t] = c;
}

// Tables of the layer seen as N + S experts with k + S slots per token: the S always-on experts become experts
// N .. N + S - 1 and take the last S slots of every token (weight 1, or the sigmoid gate of the token), so that one
// grouped launch computes routed and shared experts alike.  One wave per token; the routed rows keep their order and
// only their slot ids move to the wider stride.
__global__ __launch_bounds__(256) void append_shared_kernel(
    int T, int d, int N, int k, int S, const uint16_t *__restrict__ h, const uint16_t *__restrict__ w_sg,
    const int32_t *__restrict__ idx, const float *__restrict__ w, const int32_t *__restrict__ counts,
    const int32_t *__restrict__ offsets, const int32_t *__restrict__ perm, const int32_t *__restrict__ inv,
    int32_t *__restrict__ x_idx, float *__restrict__ x_w, int32_t *__restrict__ x_counts, int32_t *__restrict__ x_offsets,
    int32_t *__restrict__ x_perm, int32_t *__restrict__ x_inv)
{
    const int lane = threadIdx.x & 63;
    const int R = T * k, kx = k + S;
    const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (t < T) {
        float c = 1.0f;
        if (w_sg != nullptr) c = sigmoid_gate_of(h + (size_t)t * d, w_sg, d, lane);
        if (lane < kx) {
            const int o = t * kx + lane;
            if (lane < k) {
                x_idx[o] = idx[t * k + lane];
                x_w[o] = w[t * k + lane];
                x_inv[o] = inv[t * k + lane];
            } else {
                const int row = R + (lane - k) * T + t;
                x_idx[o] = N + lane - k;
                x_w[o] = c;
                x_inv[o] = row;
                x_perm[row] = o;
            }
        }
    }
    for (int i = blockIdx.x * 256 + threadIdx.x; i < R; i += gridDim.x * 256) {
        const int v = perm[i];
        x_perm[i] = v + (v / k) * S;
    }
    if (blockIdx.x == 0) {
        for (int e = threadIdx.x; e < N + S; e += 256) {
            x_counts[e] = e < N ? counts[e] : T;
            x_offsets[e] = e < N ? offsets[e] : R + (e - N) * T;
        }
        if (threadIdx.x == 0) x_offsets[N + S] = R + S * T;
    }
}

// ---------------------------------------------------------------------------------------------------
// host side
static gate_job make_job(const void *gate_w, const float *bias, int norm_mode, int32_t *topk_idx, float *topk_w)
{
    gate_job j = {};
    j.gate_w = (const uint16_t *)gate_w;
    j.bias = bias;
    j.norm_mode = norm_mode;
    j.topk_idx = topk_idx;
    j.topk_w = topk_w;
    return j;
}

// Token tiles are dealt to as many blocks as make one round of compute units
static unsigned gate_streams(unsigned tiles, unsigned slices)
{
    const unsigned n = slices >= 256 ? 1 : 256 / slices;
    return tiles < n ? tiles : n;
}

template <int NT>
static void launch_gate_logits(const moe_shape *s, const uint16_t *h, dim3 grid, hipStream_t st, const gate_jobs &jobs)
{
    const int run = (s->d / 32 + ROUTE_SEGS - 1) / ROUTE_SEGS;        // steps of a wave
    const dim3 block(ROUTE_THREADS);
    if (run == 1) hipLaunchKernelGGL((gate_logits_kernel<NT, 1>), grid, block, 0, st, s->T, s->d, s->N, h, jobs);
    else if (run == 2) hipLaunchKernelGGL((gate_logits_kernel<NT, 2>), grid, block, 0, st, s->T, s->d, s->N, h, jobs);
    else hipLaunchKernelGGL((gate_logits_kernel<NT, 4>), grid, block, 0, st, s->T, s->d, s->N, h, jobs);
}

// Launches the gate kernels for one job, or for two jobs side by side (both of the same size, so they take the same
// path).  ws_logits[i]: [max(T, 16), N] scratch of job i for the paths that store logits, or null (a job with a residual always has one).
static int launch_gate_topk(const moe_shape *s, const void *h, hipStream_t st, int n_jobs, gate_job *jobs, float *const *ws_logits)
{
    const int NT = (s->N + 15) / 16;
    gate_jobs two = {{jobs[0], jobs[n_jobs - 1]}};
    const bool fold = jobs[n_jobs - 1].res_vec != nullptr;
    const int tokens = fold ? FOLD_ROW : ROUTE_TOKENS;
    dim3 grid((s->T + tokens - 1) / tokens, 1, n_jobs), block(ROUTE_THREADS);
    const uint16_t *hp = (const uint16_t *)h;
    if (s->T <= ROUTE_TOKENS && NT >= 2 && ws_logits[0] != nullptr) {
        // decode-sized batch with many experts: one block would stream the whole gate matrix alone, so the gate product is spread
        // over one block per 16 experts and the selection runs from the stored logits.  (Up to 16 experts one block is faster, with a
        // residual too: prediction at d = 4096, 8 experts, 1 token 7.8 us against 10.8 as two launches, 13 tokens 8.4 / 11.5, 16 8.7 / 12.3)
        for (int i = 0; i < 2; ++i) two.job[i].logits = ws_logits[i < n_jobs ? i : n_jobs - 1];
        grid.y = NT;
        if (two.job[0].x.gate != nullptr) grid.z += 1;
        launch_gate_logits<1>(s, hp, grid, st, two);
        MOE_CHECK_LAUNCH();
        // T <= 16 and k <= 8: at most 128 selections, so the selecting block also builds the tables
        hipLaunchKernelGGL(select_decode_kernel, dim3(1, 1, n_jobs), dim3(SELECT_THREADS), 0, st, s->T, s->N, s->k, two);
        MOE_CHECK_LAUNCH();
        return MOE_OK;
    }
    const int blocks = (s->T + ROUTE_TOKENS - 1) / ROUTE_TOKENS * n_jobs;
    if (s->T > ROUTE_TOKENS && (NT >= 4 || (fold && NT >= 2 && s->d <= 4096 && blocks > 512)) && ws_logits[0] != nullptr) {
        // many experts: a block that evaluated all of them for its tokens would leave half the chip idle and spend its time on the
        // gate rows, so the gate product runs as (token blocks x 32-expert slices) and the selection, one wavefront per token,
        // reads the stored logits.  With 17 to 48 experts and a residual also where the blocks that select would be more than two rounds
        // (prediction, those / stored: d = 2048, 32 experts, 8192 tokens 22.9 / 24.1 us, 16384 44 / 37; d = 1024, 20 experts 17.5 / 18.2,
        // 31 / 27), but not for gate rows that do not stay in registers (d = 8192, 48 experts, 16384 tokens 98 / 153).
        for (int i = 0; i < 2; ++i) two.job[i].logits = ws_logits[i < n_jobs ? i : n_jobs - 1];
        grid.y = (s->N + 31) / 32;
        grid.x = gate_streams(grid.x, grid.y * n_jobs);
        launch_gate_logits<2>(s, hp, grid, st, two);
        MOE_CHECK_LAUNCH();
        hipLaunchKernelGGL(select_rows_kernel, dim3((s->T + SELECT_THREADS / 64 - 1) / (SELECT_THREADS / 64), 1, n_jobs),
                           dim3(SELECT_THREADS), 0, st, s->T, s->N, s->k, two);
        MOE_CHECK_LAUNCH();
        return MOE_OK;
    }
    two.job[0].x.gate = nullptr;      // the block that selects evaluates the shared experts' gates too
    grid.x = (s->T + ROUTE_TOKENS - 1) / ROUTE_TOKENS;
    const bool tables = two.job[0].counts != nullptr;
#define GT(n, tables_, res) hipLaunchKernelGGL((gate_topk_kernel<n, tables_, res>), grid, block, 0, st, s->T, s->d, s->N, s->k, hp, two)
    if (fold) {                        // a residual comes with a workspace: 48 experts at most, and 16 in a decode-sized batch
        if (tables) GT(1, true, RES_BESIDE);
        else if (NT == 1) GT(1, false, RES_BESIDE);
        else if (NT == 2) GT(2, false, RES_BESIDE);
        else GT(3, false, RES_BESIDE);
        MOE_CHECK_LAUNCH();
        return MOE_OK;
    }
    // Without a residual both ways of compiling the block are right.  With the code of the residual's rows it has up to 28 more registers
    // and its token loads stay ahead of the branches of the steps: faster (d = 8192, 8 experts, 16384 tokens 53 / 58 us, 48 experts 94 /
    // 105), but for 17 to 32 experts, where the 58 registers without it let two blocks share a compute unit (d = 1024, 20 experts,
    // 16384 tokens 27.8 / 21.8 us; d = 2048, 32 experts 46.1 / 37.7, 200 tokens 8.8 / 8.6).
#define GTN(n)                              \
    case n:                                 \
        if (tables) GT(n, true, RES_NONE);  \
        else GT(n, false, n == 2 ? RES_NONE : RES_IN_TILE); \
        break;
    switch (NT) {
        GTN(1) GTN(2) GTN(3) GTN(4) GTN(5) GTN(6) GTN(7) GTN(8)
    default:
        return MOE_EUNSUPPORTED;
    }
#undef GTN
#undef GT
    MOE_CHECK_LAUNCH();
    return MOE_OK;
}

// [max(T, 16), N] fp32 logits scratch number `which` (0: routing, 1: prediction) inside the routing workspace
static float *route_logits_scratch(const moe_shape *s, void *workspace, int which)
{
    if (workspace == nullptr) return nullptr;
    moe_ws_layout L = moe_ws(s);
    return (float *)((char *)workspace + L.route + moe_align256(MOE_MAX_EXPERTS * 4) + 2 * moe_align256((size_t)s->T * s->k * 4) +
                     (size_t)which * moe_logits_scratch_bytes(s));
}

static bool single_block_routing(const moe_shape *s) { return s->T <= ROUTE_TOKENS && s->T * s->k <= 128; }

static gate_job route_job(const moe_shape *s, const void *gate_w, const float *gate_bias, int norm_mode, int32_t *topk_idx,
                          float *topk_w, int32_t *counts, int32_t *offsets, int32_t *perm, int32_t *inv_perm)
{
    gate_job j = make_job(gate_w, gate_bias, norm_mode, topk_idx, topk_w);
    if (single_block_routing(s)) {     // one block: histogram, scan and permutation in the same launch
        j.counts = counts;
        j.offsets = offsets;
        j.perm = perm;
        j.inv_perm = inv_perm;
    }
    return j;
}

// prediction job: at decode sizes the selecting block does histogram and top-p; beyond, they follow in a launch of their own
static gate_job predict_job(const moe_shape *s, const float *res_vec, const void *next_gate_w, const float *next_gate_bias, int p,
                            int32_t *pred_counts, int32_t *top_experts, void *workspace)
{
    moe_ws_layout L = moe_ws(s);
    char *ws = (char *)workspace + L.route;
    const size_t R = (size_t)s->T * s->k;
    int32_t *idx = (int32_t *)(ws + moe_align256(MOE_MAX_EXPERTS * 4));
    float *w = (float *)(ws + moe_align256(MOE_MAX_EXPERTS * 4) + moe_align256(R * 4));
    gate_job j = make_job(next_gate_w, next_gate_bias, MOE_NORM_NONE, idx, w);
    j.res_vec = res_vec;
    if (single_block_routing(s)) {
        j.counts = pred_counts;
        j.top = top_experts;
        j.p = p;
    }
    return j;
}

int moe_route_impl(const moe_shape *s, const void *h, const void *gate_w, const float *gate_bias, int norm_mode,
                   int32_t *topk_idx, float *topk_w, int32_t *counts, int32_t *offsets, int32_t *perm,
                   int32_t *inv_perm, void *workspace, hipStream_t st)
{
    gate_job j = route_job(s, gate_w, gate_bias, norm_mode, topk_idx, topk_w, counts, offsets, perm, inv_perm);
    float *wl[1] = {route_logits_scratch(s, workspace, 0)};
    int rc = launch_gate_topk(s, h, st, 1, &j, wl);
    if (rc != MOE_OK || single_block_routing(s)) return rc;
    return launch_hist_scan_perm(s->T * s->k, s->N, topk_idx, counts, offsets, perm, inv_perm, nullptr, st);
}

int moe_predict_impl(const moe_shape *s, const void *h, const float *res_vec, const void *next_gate_w,
                     const float *next_gate_bias, int p, int32_t *pred_counts, int32_t *top_experts, void *workspace,
                     hipStream_t st)
{
    gate_job j = predict_job(s, res_vec, next_gate_w, next_gate_bias, p, pred_counts, top_experts, workspace);
    float *wl[1] = {route_logits_scratch(s, workspace, 1)};
    int rc = launch_gate_topk(s, h, st, 1, &j, wl);
    if (rc != MOE_OK || single_block_routing(s)) return rc;
    const top_job top = {j.topk_idx, pred_counts, top_experts, p};
    hipLaunchKernelGGL(hist_top_kernel, dim3(1), dim3(HT_THREADS), 0, st, s->T * s->k, s->N, top);
    MOE_CHECK_LAUNCH();
    return MOE_OK;
}

// Routing of this layer and workload prediction of the next in one pass: the two gates are evaluated by the same launches
// (blockIdx.z = 0 routes, 1 predicts).  Beyond decode sizes that is three launches: 1531 tokens, 128 experts 25 us.
int moe_route_predict_impl(const moe_shape *s, const void *h, const void *gate_w, const float *gate_bias, int norm_mode,
                           int32_t *topk_idx, float *topk_w, int32_t *counts, int32_t *offsets, int32_t *perm,
                           int32_t *inv_perm, const float *res_vec, const void *next_gate_w, const float *next_gate_bias,
                           int p, int32_t *pred_counts, int32_t *top_experts, void *workspace, hipStream_t st)
{
    gate_job jobs[2] = {route_job(s, gate_w, gate_bias, norm_mode, topk_idx, topk_w, counts, offsets, perm, inv_perm),
                        predict_job(s, res_vec, next_gate_w, next_gate_bias, p, pred_counts, top_experts, workspace)};
    float *wl[2] = {route_logits_scratch(s, workspace, 0), route_logits_scratch(s, workspace, 1)};
    int rc = launch_gate_topk(s, h, st, 2, jobs, wl);
    if (rc != MOE_OK || single_block_routing(s)) return rc;
    const top_job top = {jobs[1].topk_idx, pred_counts, top_experts, p};
    return launch_hist_scan_perm(s->T * s->k, s->N, topk_idx, counts, offsets, perm, inv_perm, &top, st);
}

int moe_dense_route_impl(const moe_shape *s, int32_t *counts, int32_t *offsets, int32_t *perm, hipStream_t st)
{
    int n = s->T * s->N;
    hipLaunchKernelGGL(dense_route_kernel, dim3((n + 255) / 256), dim3(256), 0, st, s->T, s->N, counts, offsets, perm);
    MOE_CHECK_LAUNCH();
    return MOE_OK;
}

int moe_append_shared_impl(const moe_shape *, int, const void *, const void *, const int32_t *, const float *, const int32_t *,
                           const int32_t *, const int32_t *, const int32_t *, int32_t *, float *, int32_t *, int32_t *, int32_t *,
                           int32_t *, hipStream_t);

// moe_route followed by moe_append_shared; at decode sizes the selecting block writes both sets of tables
int moe_route_shared_impl(const moe_shape *s, int n_shared, const void *h, const void *gate_w, const float *gate_bias, int norm_mode,
                          const void *w_sg, int32_t *topk_idx, float *topk_w, int32_t *counts, int32_t *offsets, int32_t *perm,
                          int32_t *inv_perm, int32_t *x_topk_idx, float *x_topk_w, int32_t *x_counts, int32_t *x_offsets,
                          int32_t *x_perm, int32_t *x_inv_perm, void *workspace, hipStream_t st)
{
    if (!single_block_routing(s)) {
        int rc = moe_route_impl(s, h, gate_w, gate_bias, norm_mode, topk_idx, topk_w, counts, offsets, perm, inv_perm, workspace, st);
        if (rc != MOE_OK) return rc;
        return moe_append_shared_impl(s, n_shared, h, w_sg, topk_idx, topk_w, counts, offsets, perm, inv_perm, x_topk_idx, x_topk_w,
                                      x_counts, x_offsets, x_perm, x_inv_perm, st);
    }
    gate_job j = route_job(s, gate_w, gate_bias, norm_mode, topk_idx, topk_w, counts, offsets, perm, inv_perm);
    j.x.S = n_shared;
    j.x.d = s->d;
    j.x.h = (const uint16_t *)h;
    j.x.w_sg = (const uint16_t *)w_sg;
    if (w_sg != nullptr && workspace != nullptr) j.x.gate = (float *)((char *)workspace + moe_ws(s).route);
    j.x.x_idx = x_topk_idx;
    j.x.x_w = x_topk_w;
    j.x.x_counts = x_counts;
    j.x.x_offsets = x_offsets;
    j.x.x_perm = x_perm;
    j.x.x_inv = x_inv_perm;
    float *wl[1] = {route_logits_scratch(s, workspace, 0)};
    return launch_gate_topk(s, h, st, 1, &j, wl);
}

int moe_shared_gate_impl(const moe_shape *s, const void *h, const void *w_sg, float *scale, hipStream_t st)
{
    hipLaunchKernelGGL(shared_gate_kernel, dim3((s->T + 3) / 4), dim3(256), 0, st, s->T, s->d, (const uint16_t *)h,
                       (const uint16_t *)w_sg, scale);
    MOE_CHECK_LAUNCH();
    return MOE_OK;
}

int moe_append_shared_impl(const moe_shape *s, int n_shared, const void *h, const void *w_sg, const int32_t *topk_idx,
                           const float *topk_w, const int32_t *counts, const int32_t *offsets, const int32_t *perm,
                           const int32_t *inv_perm, int32_t *x_topk_idx, float *x_topk_w, int32_t *x_counts,
                           int32_t *x_offsets, int32_t *x_perm, int32_t *x_inv_perm, hipStream_t st)
{
    hipLaunchKernelGGL(append_shared_kernel, dim3((s->T + 3) / 4), dim3(256), 0, st, s->T, s->d, s->N, s->k, n_shared,
                       (const uint16_t *)h, (const uint16_t *)w_sg, topk_idx, topk_w, counts, offsets, perm, inv_perm, x_topk_idx,
                       x_topk_w, x_counts, x_offsets, x_perm, x_inv_perm);
    MOE_CHECK_LAUNCH();
    return MOE_OK;
}

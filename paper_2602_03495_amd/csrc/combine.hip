// Weighted combine of the expert outputs (Eq. 2 restricted to the experts placed on this GPU) for gfx950.
// One block per token and 2048 columns; each thread owns 8 consecutive hidden features (one 16-byte bf16 load per source row),
// sums in fp32 in slot order and rounds once to bf16.  A gather, so no atomics and no ordering effects.
#include "moe_common.h"

__device__ __forceinline__ void fma8(float (&acc)[8], float w, uint4 v)
{
    acc[0] = fmaf(w, bf16_lo(v.x), acc[0]); acc[1] = fmaf(w, bf16_hi(v.x), acc[1]);
    acc[2] = fmaf(w, bf16_lo(v.y), acc[2]); acc[3] = fmaf(w, bf16_hi(v.y), acc[3]);
    acc[4] = fmaf(w, bf16_lo(v.z), acc[4]); acc[5] = fmaf(w, bf16_hi(v.z), acc[5]);
    acc[6] = fmaf(w, bf16_lo(v.w), acc[6]); acc[7] = fmaf(w, bf16_hi(v.w), acc[7]);
}

// The next B source rows of the set bits of `on` (slot order), all of them on their way before the first sum.
template <int B>
__device__ __forceinline__ void add_rows(float (&acc)[8], unsigned long long &on, int p, float w, const uint16_t *__restrict__ yf, int d)
{
    uint4 v[B];
    float wj[B];
#pragma unroll
    for (int j = 0; j < B; ++j) {
        const int l = __ffsll(on) - 1;
        on &= on - 1;
        wj[j] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w), l));
        v[j] = *reinterpret_cast<const uint4 *>(yf + (size_t)__builtin_amdgcn_readlane(p, l) * d);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < B; ++j) fma8(acc, wj[j], v[j]);
}

// Bound by latency at decode sizes, by the reads beyond.  Every wave holds the slots of its token in its first lanes, finds
// those placed on this GPU by a ballot and reads all their rows at once: with a loop over the slots that skipped the others,
// the reads of up to 8 rows followed one another (16 tokens, 8 slots, d = 2048: 3.7 us, now 2.5).
// MASKED: two kernels, because without a mask the rows need not wait for the experts of the slots (2.42 us, and 2.55 where they do; 1100
// tokens of 6 slots 4.36 / 4.76) and a branch on it inside costs either (2.54 and 2.65 with a mask).
template <bool MASKED>
__global__ __launch_bounds__(256) void combine_kernel(int T, int d, int N, int k, const uint16_t *__restrict__ y,
                                                      const int32_t *__restrict__ topk_idx, const float *__restrict__ topk_w,
                                                      const int32_t *__restrict__ inv_perm, const uint8_t *__restrict__ mask,
                                                      const uint16_t *__restrict__ shared_y, int n_shared,
                                                      const float *__restrict__ shared_scale, uint16_t *__restrict__ out)
{
    const int t = blockIdx.x, lane = threadIdx.x & 63;
    int p = 0;
    float w = 0.f;
    bool mine = lane < k;
    unsigned long long on_lo = 0, on_hi = 0;
    if (MASKED) {                       // the whole of it, beside the slots: looked up by expert it was a round trip after them
        const int m0 = mask[min(lane, N - 1)], m1 = mask[min(lane + 64, N - 1)];
        on_lo = __ballot(m0 != 0);
        on_hi = __ballot(m1 != 0);
    }
    if (mine) {
        const size_t r = (size_t)t * k + lane;
        const int e = MASKED ? topk_idx[r] : 0;
        w = topk_w[r];
        p = inv_perm[r];
        if (MASKED) mine = ((e < 64 ? on_lo : on_hi) >> (e & 63) & 1ull) != 0;
    }
    unsigned long long on = __ballot(mine);
    const float sc = (n_shared > 0 && shared_scale != nullptr) ? shared_scale[t] : 1.0f;
    const int f = (blockIdx.y * 256 + threadIdx.x) * 8;
    if (blockIdx.y * 2048 + (threadIdx.x & ~63) * 8 >= d) return;          // the whole wave is beyond the row
    const int fr = f < d ? f : 0;                                          // lanes beyond it read column 0 and write nothing
    uint4 sh[2];
#pragma unroll
    for (int m = 0; m < 2; ++m)
        if (m < n_shared) sh[m] = *reinterpret_cast<const uint4 *>(shared_y + ((size_t)m * T + t) * d + fr);
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const uint16_t *yf = y + fr;
    switch (__popcll(on)) {            // at most MOE_MAX_TOPK
    case 1: add_rows<1>(acc, on, p, w, yf, d); break;
    case 2: add_rows<2>(acc, on, p, w, yf, d); break;
    case 3: add_rows<3>(acc, on, p, w, yf, d); break;
    case 4: add_rows<4>(acc, on, p, w, yf, d); break;
    case 5: add_rows<5>(acc, on, p, w, yf, d); break;
    case 6: add_rows<6>(acc, on, p, w, yf, d); break;
    case 7: add_rows<7>(acc, on, p, w, yf, d); break;
    case 8: add_rows<8>(acc, on, p, w, yf, d); break;
    }
#pragma unroll
    for (int m = 0; m < 2; ++m)
        if (m < n_shared) fma8(acc, sc, sh[m]);
    for (int m = 2; m < n_shared; ++m)
        fma8(acc, sc, *reinterpret_cast<const uint4 *>(shared_y + ((size_t)m * T + t) * d + fr));
    if (f < d) {
        uint4 o;
        o.x = pack_bf16x2(acc[0], acc[1]);
        o.y = pack_bf16x2(acc[2], acc[3]);
        o.z = pack_bf16x2(acc[4], acc[5]);
        o.w = pack_bf16x2(acc[6], acc[7]);
        *reinterpret_cast<uint4 *>(out + (size_t)t * d + f) = o;
    }
}

// The same sums for many tokens with few slots: a block walks the columns of its token, whose tables it reads once for all of them.
__global__ __launch_bounds__(256) void combine_walk_kernel(int T, int d, int k, const uint16_t *__restrict__ y,
                                                           const int32_t *__restrict__ topk_idx, const float *__restrict__ topk_w,
                                                           const int32_t *__restrict__ inv_perm, const uint8_t *__restrict__ mask,
                                                           const uint16_t *__restrict__ shared_y, int n_shared,
                                                           const float *__restrict__ shared_scale, uint16_t *__restrict__ out)
{
    const int t = blockIdx.x;
    __shared__ float w_s[MOE_MAX_TOPK];
    __shared__ int p_s[MOE_MAX_TOPK];
    if (threadIdx.x < k) {
        const size_t r = (size_t)t * k + threadIdx.x;
        const int e = topk_idx[r];
        const bool on = mask == nullptr || mask[e] != 0;
        w_s[threadIdx.x] = topk_w[r];
        p_s[threadIdx.x] = on ? inv_perm[r] : -1;
    }
    __syncthreads();
    const float sc = (n_shared > 0 && shared_scale != nullptr) ? shared_scale[t] : 1.0f;
    for (int f = threadIdx.x * 8; f < d; f += 256 * 8) {
        float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        for (int s = 0; s < k; ++s) {
            const int p = p_s[s];
            if (p >= 0) fma8(acc, w_s[s], *reinterpret_cast<const uint4 *>(y + (size_t)p * d + f));
        }
        for (int m = 0; m < n_shared; ++m)
            fma8(acc, sc, *reinterpret_cast<const uint4 *>(shared_y + ((size_t)m * T + t) * d + f));
        uint4 o;
        o.x = pack_bf16x2(acc[0], acc[1]);
        o.y = pack_bf16x2(acc[2], acc[3]);
        o.z = pack_bf16x2(acc[4], acc[5]);
        o.w = pack_bf16x2(acc[6], acc[7]);
        *reinterpret_cast<uint4 *>(out + (size_t)t * d + f) = o;
    }
}

// combine_kernel's speed over combine_walk_kernel's, no mask / a quarter to half of the experts on.  d = 8192, 2 slots: 1030 tokens 1.03 /
// 1.03 to 1.08, 12000 1.02 / 0.72, 40000 0.99 / 0.93 to 1.05; 3 slots, 12000 tokens 1.00 / 0.74 to 1.00; 1 slot 0.98 / 0.83.  d = 4096: 2
// slots, 1030 tokens 1.11 / 1.04, 12000 1.09 / 0.99; 1 slot 1.03 / 0.86, 40000 0.97 / 0.80.  d = 1152: 1.06 to 1.28 / 1.0 to 1.18.
// With 5 slots or more, and up to 1024 columns, it was level or ahead with 5 waves on a SIMD already (0.94 to 2.4); with 4, 0.88 to 1.65.
// The line was drawn where combine_kernel ran 5 waves on a SIMD (d = 4096, 2 slots, 1500 tokens 0.95 / 0.88); with the 8 it has
// now it gains where rows are many, up to a few microseconds, and loses up to a quarter where few are on.
static bool combine_walks(const moe_shape *s) { return s->k <= 3 && s->d > 1024 && s->T > 1024; }

int moe_combine_impl(const moe_shape *s, const void *y, const int32_t *topk_idx, const float *topk_w,
                     const int32_t *inv_perm, const uint8_t *expert_mask, const void *shared_y, int n_shared,
                     const float *shared_scale, void *out, hipStream_t st)
{
    // rows shorter than a block's 2048 columns: only the waves that have some (20000 tokens of 128 columns, 1 slot, 2 shared
    // experts: 13.2 us with all four, 7.3 with one)
    const unsigned threads = s->d >= 2048 ? 256 : (unsigned)(s->d + 511) / 512 * 64;
#define COMBINE(kernel, grid, ...)                                                                                              \
    hipLaunchKernelGGL(kernel, grid, dim3(threads), 0, st, s->T, s->d, __VA_ARGS__, (const uint16_t *)y, topk_idx, topk_w, inv_perm, \
                       expert_mask, (const uint16_t *)shared_y, shared_y ? n_shared : 0, shared_scale, (uint16_t *)out)
    const dim3 tiles(s->T, (s->d + 2047) / 2048);
    if (combine_walks(s)) COMBINE(combine_walk_kernel, dim3(s->T), s->k);
    else if (expert_mask != nullptr) COMBINE(combine_kernel<true>, tiles, s->N, s->k);
    else COMBINE(combine_kernel<false>, tiles, s->N, s->k);
#undef COMBINE
    MOE_CHECK_LAUNCH();
    return MOE_OK;
}

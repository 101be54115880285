// Element-wise multiplication weights (Sec. 3.2, "Codebook Optimization for Element-wise
// Multiplication") and the token-shift mix that consumes them (Eq. "time mixing r/k/v", Eq.
// "channel mixing r/k"):
//   clip_mean_kernel      the representative activation of a calibration batch: per position, the
//                         samples limited to their [p, 100 - p] percentile range, then averaged;
//   mu_kmeans_kernel      X^2-weighted Lloyd iterations on the weight's 2-vectors (the loss of Eq.
//                         "quantization loss of mul"), one workgroup per weight tensor;
//   token_shift_mix_kernel  mu_hat * x_t + (1 - mu_hat) * x_{t-1} for all projections of a layer
//                         in one pass over the activations, mu_hat looked up in its codebook.
// Every decision (argmin, percentile rank) is taken on binary32 / binary64 values computed with one
// rounding per operation in a fixed formula, so that any implementation of the same steps takes
// the same decisions.
#include "common.h"

#include <algorithm>
#include <type_traits>
#include <utility>
#include <vector>

namespace rwkvq {

// ---------------------------------------------------------------------------------- clip_mean
// clip_mean_select_kernel<NS> (B <= 16 NS): a workgroup takes 16 consecutive positions, sixteen lanes (a DPP row) each; a
// lane holds NS samples of its position as order-preserving keys.  The percentiles need order statistics by value only (ties
// have one value), so the k-th is built bit by bit: bit t of it is set when at most k keys lie below the prefix with that
// bit - a count over the row per bit, 16 bits for 16-bit samples, 32 for binary32, both percentiles in one count.  Its
// successor is the same value again or the least key above.  One thread per position then forms the clipped mean as a binary64
// sum in sample order.  Ranking every sample by B comparisons (the kernel this replaces: 64 workgroups for 4096 positions, B^2
// comparisons each position) took 119 us for 128 x 4096 bf16 samples, this 8.8 us: the chain of 128 binary64 additions and
// the trips to memory are what is left.  Up to 32 samples a lane counts the keys below and up to each of its own in fifteen row
// rotations instead of 32 counts in a row (20480 positions, 16 binary32 samples: 12.5 -> 6.8 us).
constexpr int kClipP = 16;                           // positions per workgroup
constexpr int kClipMaxB = 1024;                      // sixteen lanes of 64 samples
__device__ __forceinline__ int clip_at(int b, int p) { return b * kClipP + (p ^ (b & 15)); }   // sixteen samples of a position: sixteen banks
__device__ __forceinline__ int row_sum(int v) {      // over the sixteen lanes of a DPP row, in every lane
    v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, true);      // quad_perm [1, 0, 3, 2]
    v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, true);      // quad_perm [2, 3, 0, 1]
    v += __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, true);     // row_half_mirror
    return v + __builtin_amdgcn_update_dpp(0, v, 0x140, 0xF, 0xF, true);
}
__device__ __forceinline__ uint32_t row_min(uint32_t v) {
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true));
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true));
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, true));
    return min(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, true));
}
template <int... R>                                  // over the sixteen values o of the DPP row: how many are below v, how many at most v
__device__ __forceinline__ void row_rank(uint32_t o, uint32_t v, int& below, int& at_most, std::integer_sequence<int, R...>) {
    auto other = [&](uint32_t t) { below += t < v ? 1 : 0; at_most += t <= v ? 1 : 0; };
    other(o);
    (other((uint32_t)__builtin_amdgcn_update_dpp(0, (int)o, 0x121 + R, 0xF, 0xF, true)), ...);     // row_ror 1 .. 15
}
template <int NS>
__global__ void __launch_bounds__(256) clip_mean_select_kernel(const void* __restrict__ x, int dt, int B, int n, int k_lo,
                                                               double f_lo, int k_hi, double f_hi, float* __restrict__ out) {
    extern __shared__ uint32_t tile[];               // [B][16] bit patterns (16-bit samples: in the high half)
    __shared__ float stat[4][kClipP];
    const int tid = threadIdx.x, j0 = blockIdx.x * kClipP;
    {
        // all of a thread's loads before the first store (one trip to memory instead of B / 16)
        const int p = tid % kClipP, j = min(j0 + p, n - 1), b0 = tid / kClipP;
        constexpr int kAt = NS < 16 ? NS : 16;
        for (int i0 = 0; i0 < NS; i0 += kAt) {
            uint32_t v[kAt];
            if (dt == DT_F32) {
#pragma unroll
                for (int i = 0; i < kAt; ++i) v[i] = ((const uint32_t*)x)[(size_t)min(b0 + 16 * (i0 + i), B - 1) * n + j];
            } else {
#pragma unroll
                for (int i = 0; i < kAt; ++i) v[i] = ((const uint16_t*)x)[(size_t)min(b0 + 16 * (i0 + i), B - 1) * n + j];
            }
#pragma unroll
            for (int i = 0; i < kAt; ++i) {
                const int b = b0 + 16 * (i0 + i);
                if (b < B) tile[clip_at(b, p)] = dt == DT_F32 ? v[i] : v[i] << 16;
            }
        }
    }
    __syncthreads();
    const int p = tid >> 4, l = tid & 15;
    uint32_t key[NS];
#pragma unroll
    for (int i = 0; i < NS; ++i) {
        const int b = l + 16 * i;
        const uint32_t v = tile[clip_at(min(b, B - 1), p)];
        const uint32_t k = (v & 0x80000000u) ? ~v & (dt == DT_F32 ? 0xFFFFFFFFu : 0xFFFF0000u) : v | 0x80000000u;
        key[i] = b < B ? k : 0xFFFFFFFFu;            // above every finite sample
    }
    auto value = [&](uint32_t k) {
        const uint32_t v = (k & 0x80000000u) ? k & 0x7FFFFFFFu : ~k & (dt == DT_F32 ? 0xFFFFFFFFu : 0xFFFF0000u);
        return dt == DT_F32 ? __uint_as_float(v) : dt == DT_BF16 ? __uint_as_float(v) : f16_bits_to_f32((uint16_t)(v >> 16));
    };
    if constexpr (NS <= 2) {
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            int below = 0, at_most = 0;
#pragma unroll
            for (int j = 0; j < NS; ++j) row_rank(key[j], key[i], below, at_most, std::make_integer_sequence<int, 15>{});
            auto is = [&](int k) { return below <= k && k < at_most; };   // the k-th, k < B (lanes that tie store the same value)
            const float v = value(key[i]);
            if (is(k_lo)) stat[0][p] = v;
            if (is(min(k_lo + 1, B - 1))) stat[1][p] = v;
            if (is(k_hi)) stat[2][p] = v;
            if (is(min(k_hi + 1, B - 1))) stat[3][p] = v;
        }
    } else {
        uint32_t lo = 0, hi = 0;                         // keys of the k_lo-th and k_hi-th sample
        for (int bit = 31; bit >= (dt == DT_F32 ? 0 : 16); --bit) {
            const uint32_t tl = lo | (1u << bit), th = hi | (1u << bit);
            int c = 0;                                   // samples below tl, and below th in the high half
#pragma unroll
            for (int i = 0; i < NS; ++i) c += (key[i] < tl ? 1 : 0) + (key[i] < th ? 0x10000 : 0);
            c = row_sum(c);
            if ((c & 0xFFFF) <= k_lo) lo = tl;
            if ((c >> 16) <= k_hi) hi = th;
        }
        int at_most = 0;
        uint32_t next_lo = 0xFFFFFFFFu, next_hi = 0xFFFFFFFFu;
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            at_most += (key[i] <= lo ? 1 : 0) + (key[i] <= hi ? 0x10000 : 0);
            if (key[i] > lo) next_lo = min(next_lo, key[i]);
            if (key[i] > hi) next_hi = min(next_hi, key[i]);
        }
        at_most = row_sum(at_most);
        next_lo = row_min(next_lo);
        next_hi = row_min(next_hi);
        if ((at_most & 0xFFFF) > k_lo + 1 || k_lo + 1 >= B) next_lo = lo;
        if ((at_most >> 16) > k_hi + 1 || k_hi + 1 >= B) next_hi = hi;
        if (l == 0) { stat[0][p] = value(lo); stat[1][p] = value(next_lo); stat[2][p] = value(hi); stat[3][p] = value(next_hi); }
    }
    __syncthreads();
    const double f_v = (double)stat[0][p], f_w = (double)stat[2][p];
    const double dlo = __dadd_rn(f_v, __dmul_rn(f_lo, __dsub_rn((double)stat[1][p], f_v)));
    const double dhi = __dadd_rn(f_w, __dmul_rn(f_hi, __dsub_rn((double)stat[3][p], f_w)));
    auto clipped = [&](uint32_t w, double at_least, double at_most) {
        double v = (double)(dt == DT_F16 ? f16_bits_to_f32((uint16_t)(w >> 16)) : __uint_as_float(w));
        v = v < at_least ? at_least : v;
        return v > at_most ? at_most : v;
    };
    // The sum is in sample order, one binary64 addition after another: clipped by all threads first, so that the one thread
    // per position only adds (14 -> 8.8 us; B <= 256, the doubles of more would not fit).
    double* const limited = (double*)(tile + B * kClipP);
    if constexpr (NS <= 16) {
#pragma unroll
        for (int i = 0; i < NS; ++i)
            if (l + 16 * i < B) limited[clip_at(l + 16 * i, p)] = clipped(tile[clip_at(l + 16 * i, p)], dlo, dhi);
    } else {
        if (l == 0) { limited[p] = dlo; limited[kClipP + p] = dhi; }
    }
    __syncthreads();
    if (tid < kClipP && j0 + tid < n) {
        double acc = 0.0;
        if constexpr (NS <= 16) {
#pragma unroll 16
            for (int b = 0; b < B; ++b) acc = __dadd_rn(acc, limited[clip_at(b, tid)]);
        } else {
            const double at_least = limited[tid], at_most = limited[kClipP + tid];
#pragma unroll 8
            for (int b = 0; b < B; ++b) acc = __dadd_rn(acc, clipped(tile[clip_at(b, tid)], at_least, at_most));
        }
        out[j0 + tid] = (float)(acc / (double)B);
    }
}

// clip_mean_ends_kernel<NS> (32 < B <= 32 NS): the same where both percentiles are within a few samples of the ends (k_lo + 2 and
// B - k_hi at most kClipEnds): the distinct values are taken from either end, a minimum and a count over the position's 32 lanes per
// step, instead of a count per bit.  A minimum above m without a compare: keys up to m wrap to the top in key - (m + 1).
// What bounds it: start-up (2.5 us of a launch that moves nothing), the trips to memory, and the chain of B binary64 additions.
// 4096 positions x 128 bf16 samples 8.5 -> 5.0 us, 5120 x 256 15.3 -> 10.9, 2560 x 64 5.7 -> 3.7.  The line: a step costs about as much
// as two bits of the other way, which has 16 of them for 16-bit samples.
constexpr int kClipEnds = 6, kClipLanes = 32, kClipThreads = kClipLanes * kClipP;
__device__ __forceinline__ uint32_t lanes32_min(uint32_t v) {
    v = row_min(v);
    const auto both = __builtin_amdgcn_permlane16_swap(v, v, false, false);      // the pair's even row twice, its odd row twice
    return min((uint32_t)both[0], (uint32_t)both[1]);
}
__device__ __forceinline__ int lanes32_sum(int v) {
    v = row_sum(v);
    const auto both = __builtin_amdgcn_permlane16_swap((uint32_t)v, (uint32_t)v, false, false);
    return (int)both[0] + (int)both[1];
}
// The values of ranks k and k + 1 (k + 1 < B, or ignored) among the position's keys, the least first, from two sets of keys side by side
// (each step is a chain of exchanges between lanes; one set after the other takes 1.026 times as long in the median of 192 calls of 33 to
// 256 samples x 768 to 8192 positions, 0.99 to 1.05: 33 x 8192 4.32 us, here 4.19, 200 x 3328 6.64 and 6.48; calls issued one by one
// follow each other every 6.4 us and do not show it); steps past a set's need change nothing.
struct Ranks { uint32_t m, before, at_k, at_k1; };           // m: the value taken last, before: keys up to it
template <int NS>
__device__ __forceinline__ void lowest(const uint32_t (&low)[NS], int k_low, Ranks& l, const uint32_t (&high)[NS], int k_high, Ranks& h, int steps) {
    l = h = Ranks{0xFFFFFFFFu, 0u, 0u, 0u};
    for (int s = 0; s < steps; ++s) {
        uint32_t dl[NS], dh[NS], least_l = 0xFFFFFFFFu, least_h = 0xFFFFFFFFu;
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            dl[i] = low[i] - (l.m + 1u); least_l = min(least_l, dl[i]);
            dh[i] = high[i] - (h.m + 1u); least_h = min(least_h, dh[i]);
        }
        least_l = lanes32_min(least_l);
        least_h = lanes32_min(least_h);
        int c = 0;                                   // both counts (up to 256 each) in one sum
#pragma unroll
        for (int i = 0; i < NS; ++i) c += (dl[i] == least_l ? 1 : 0) + (dh[i] == least_h ? 0x10000 : 0);
        c = lanes32_sum(c);
        auto take = [](Ranks& r, uint32_t least, uint32_t count, int k) {
            r.m += least + 1u;
            if ((int)r.before <= k) r.at_k = r.m;
            if ((int)r.before <= k + 1) r.at_k1 = r.m;
            r.before += count;
        };
        take(l, least_l, (uint32_t)c & 0xFFFFu, k_low);
        take(h, least_h, (uint32_t)c >> 16, k_high);
    }
}
template <int NS>
__global__ void __launch_bounds__(kClipThreads) clip_mean_ends_kernel(const void* __restrict__ x, int dt, int B, int n, int k_lo, double f_lo,
                                                                      int k_hi, double f_hi, float* __restrict__ out) {
    extern __shared__ uint32_t tile[];               // as in clip_mean_select_kernel
    const int tid = threadIdx.x;
    // The 32 or 64 bytes that a workgroup reads of a sample are a part of a cache line: neighbours go to one XCD, whose L2 then
    // fetches the line once (workgroups are dealt to the eight XCDs in turn).
    const int per_xcd = gridDim.x >> 3, blk = (gridDim.x & 7) ? (int)blockIdx.x : (int)((blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3));
    const int j0 = blk * kClipP;
    {
        const int p = tid % kClipP, j = min(j0 + p, n - 1), b0 = tid / kClipP;
        uint32_t v[NS];
        if (dt == DT_F32) {
#pragma unroll
            for (int i = 0; i < NS; ++i) v[i] = ((const uint32_t*)x)[(size_t)min(b0 + kClipLanes * i, B - 1) * n + j];
        } else {
#pragma unroll
            for (int i = 0; i < NS; ++i) v[i] = ((const uint16_t*)x)[(size_t)min(b0 + kClipLanes * i, B - 1) * n + j];
        }
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            const int b = b0 + kClipLanes * i;
            if (b < B) tile[clip_at(b, p)] = dt == DT_F32 ? v[i] : v[i] << 16;
        }
    }
    __syncthreads();
    const int p = tid / kClipLanes, l = tid % kClipLanes;
    uint32_t bits[NS], low[NS], high[NS];            // ranks from below and from above; not a sample: above every one
#pragma unroll
    for (int i = 0; i < NS; ++i) {
        const int b = l + kClipLanes * i;
        bits[i] = tile[clip_at(min(b, B - 1), p)];
        const uint32_t k = (bits[i] & 0x80000000u) ? ~bits[i] & (dt == DT_F32 ? 0xFFFFFFFFu : 0xFFFF0000u) : bits[i] | 0x80000000u;
        low[i] = b < B ? k : 0xFFFFFFFFu;
        high[i] = b < B ? ~k : 0xFFFFFFFFu;
    }
    auto value = [&](uint32_t k) {
        const uint32_t v = (k & 0x80000000u) ? k & 0x7FFFFFFFu : ~k & (dt == DT_F32 ? 0xFFFFFFFFu : 0xFFFF0000u);
        return dt == DT_F32 ? __uint_as_float(v) : dt == DT_BF16 ? __uint_as_float(v) : f16_bits_to_f32((uint16_t)(v >> 16));
    };
    const int from_top = B - 1 - k_hi;               // rank of the k_hi-th from above; the next one up is rank from_top - 1
    Ranks from_low, from_high;
    lowest<NS>(low, k_lo, from_low, high, from_top - 1, from_high, max(k_lo + 2, from_top + 1));
    const uint32_t lo = from_low.at_k, hi = from_high.at_k1;
    uint32_t lo1 = from_low.at_k1, hi1 = from_high.at_k;
    if (k_lo + 1 >= B) lo1 = lo;
    if (from_top == 0) hi1 = hi;
    const double f_v = (double)value(lo), f_w = (double)value(~hi);
    const double dlo = __dadd_rn(f_v, __dmul_rn(f_lo, __dsub_rn((double)value(lo1), f_v)));
    const double dhi = __dadd_rn(f_w, __dmul_rn(f_hi, __dsub_rn((double)value(~hi1), f_w)));
    double* const limited = (double*)(tile + B * kClipP);
#pragma unroll
    for (int i = 0; i < NS; ++i) {
        const int b = l + kClipLanes * i;
        double v = (double)(dt == DT_F16 ? f16_bits_to_f32((uint16_t)(bits[i] >> 16)) : __uint_as_float(bits[i]));
        v = v < dlo ? dlo : v;
        v = v > dhi ? dhi : v;
        if (b < B) limited[clip_at(b, p)] = v;
    }
    __syncthreads();
    if (tid < kClipP && j0 + tid < n) {
        double acc = 0.0;
#pragma unroll 32
        for (int b = 0; b < B; ++b) acc = __dadd_rn(acc, limited[clip_at(b, tid)]);
        out[j0 + tid] = (float)(acc / (double)B);
    }
}

// One thread per position, samples re-read from memory: any batch size.
__global__ void __launch_bounds__(256) clip_mean_kernel(const void* __restrict__ x, int dt, int B, int n, int k_lo,
                                                        double f_lo, int k_hi, double f_hi, float* __restrict__ out) {
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= n) return;
    const int k_lo1 = k_lo + 1 < B ? k_lo + 1 : B - 1, k_hi1 = k_hi + 1 < B ? k_hi + 1 : B - 1;
    float v_lo = 0.f, v_lo1 = 0.f, v_hi = 0.f, v_hi1 = 0.f;
    for (int i = 0; i < B; ++i) {
        const float vi = load_as_f32(x, (size_t)i * n + j, dt);
        int rank = 0;
        for (int b = 0; b < B; ++b) {
            const float vb = load_as_f32(x, (size_t)b * n + j, dt);
            rank += (vb < vi || (vb == vi && b < i)) ? 1 : 0;
        }
        if (rank == k_lo) v_lo = vi;
        if (rank == k_lo1) v_lo1 = vi;
        if (rank == k_hi) v_hi = vi;
        if (rank == k_hi1) v_hi1 = vi;
    }
    // linear interpolation between neighbouring order statistics, binary64, one rounding per step
    const double lo = __dadd_rn((double)v_lo, __dmul_rn(f_lo, __dsub_rn((double)v_lo1, (double)v_lo)));
    const double hi = __dadd_rn((double)v_hi, __dmul_rn(f_hi, __dsub_rn((double)v_hi1, (double)v_hi)));
    double acc = 0.0;
    for (int b = 0; b < B; ++b) {                       // sample order: the sum is reproducible
        double v = (double)load_as_f32(x, (size_t)b * n + j, dt);
        v = v < lo ? lo : v;
        v = v > hi ? hi : v;
        acc = __dadd_rn(acc, v);
    }
    out[j] = (float)(acc / (double)B);
}

hipError_t launch_clip_mean(const void* x, int dt, int B, int n, int k_lo, double f_lo, int k_hi, double f_hi,
                            float* out, hipStream_t s) {
    // a tile of B x 16 words, and up to B = 256 as many doubles (beyond, two limits per position)
    const dim3 grid((n + kClipP - 1) / kClipP), wg(256);
    const size_t lds = (size_t)B * kClipP * 4 + (B <= 256 ? (size_t)B * kClipP * 8 : 2 * kClipP * 8);
    if (B > 2 * kClipP && B <= 256 && k_lo + 2 <= kClipEnds && B - k_hi <= kClipEnds) {
        const dim3 wide(kClipThreads);
        if (B <= 64) hipLaunchKernelGGL(clip_mean_ends_kernel<2>, grid, wide, lds, s, x, dt, B, n, k_lo, f_lo, k_hi, f_hi, out);
        else if (B <= 128) hipLaunchKernelGGL(clip_mean_ends_kernel<4>, grid, wide, lds, s, x, dt, B, n, k_lo, f_lo, k_hi, f_hi, out);
        else hipLaunchKernelGGL(clip_mean_ends_kernel<8>, grid, wide, lds, s, x, dt, B, n, k_lo, f_lo, k_hi, f_hi, out);
    } else if (B <= 16) hipLaunchKernelGGL(clip_mean_select_kernel<1>, grid, wg, lds, s, x, dt, B, n, k_lo, f_lo, k_hi, f_hi, out);
    else if (B <= 32) hipLaunchKernelGGL(clip_mean_select_kernel<2>, grid, wg, lds, s, x, dt, B, n, k_lo, f_lo, k_hi, f_hi, out);
    else if (B <= 64) hipLaunchKernelGGL(clip_mean_select_kernel<4>, grid, wg, lds, s, x, dt, B, n, k_lo, f_lo, k_hi, f_hi, out);
    else if (B <= 128) hipLaunchKernelGGL(clip_mean_select_kernel<8>, grid, wg, lds, s, x, dt, B, n, k_lo, f_lo, k_hi, f_hi, out);
    else if (B <= 256) hipLaunchKernelGGL(clip_mean_select_kernel<16>, grid, wg, lds, s, x, dt, B, n, k_lo, f_lo, k_hi, f_hi, out);
    else if (B <= kClipMaxB) {
        // (the tile of the largest B takes all of the 64 KB that need no asking; one thread per position, the kernel below, is
        // a hundred times slower there)
        static std::atomic<unsigned long long> raised{0ull};
        const hipError_t e = raise_lds((const void*)clip_mean_select_kernel<64>, kClipMaxB * kClipP * 4 + 2 * kClipP * 8, raised);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(clip_mean_select_kernel<64>, grid, wg, lds, s, x, dt, B, n, k_lo, f_lo, k_hi, f_hi, out);
    } else hipLaunchKernelGGL(clip_mean_kernel, dim3((n + 255) / 256), dim3(256), 0, s, x, dt, B, n, k_lo, f_lo, k_hi, f_hi, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------- weighted KMeans
constexpr int kMuMaxTensors = 64;
struct MuTensor {
    const void* mu;          // n elements, storage type of the launch
    const float* xbar;       // n representative activations
    uint16_t* cb;            // in: initial entries, out: final entries; fp16 [E][2]
    uint8_t* idx;            // out: n / 2 indices
    int n, pad;
};
struct MuArgs {
    MuTensor t[kMuMaxTensors];
    int dt, kbits, iters, pad;
};

// binary64 -> fp16 with a single rounding: truncate to binary32, keep inexactness in the last bit
// (round to odd), then let the binary32 -> fp16 conversion round to nearest even.
__device__ __forceinline__ uint16_t f64_to_f16_bits(double d) {
    float f = __double2float_rz(d);
    if ((double)f != d) f = __uint_as_float(__float_as_uint(f) | 1u);
    return f32_to_f16_bits(f);
}

// One workgroup per weight tensor.  The vectors go through LDS in chunks of 2048: every vector of a chunk is
// assigned to its cheapest entry, then the sums of an entry's coordinate are continued by S = 1024 / (2 E) threads, each
// over a contiguous share of the chunk in index order; after the last chunk the S partial sums are added in share order.
// Binary64 sums in a fixed order: a call gives the same codebook every time.
// A share's vectors are first put in order of their entries (stable, so an entry's vectors keep index order): one wavefront
// per share counts rounds of 64 with ballots over the entry's bits, a running sum over the entries gives their first slots.
// A thread then adds only its entry's vectors; scanning the whole share for them (what this replaces) was most of the time:
// 28 tensors of 4096 weights, 64 entries, 10 iterations 290 -> 131 us (6 iterations with every vector at one entry 183 -> 143;
// one vector's look-ups after the other there: 198).  Up to 4096 vectors stay in LDS over the iterations, and a thread compares both of
// its vectors with an entry that it has read (131 -> 107, 256 entries 395 -> 331).
// What bounds it: vector ALU of the one compute unit a tensor has, 5.6 of 9.7 us per iteration in the ten instructions per
// vector and entry, near the rate that four wavefronts per SIMD retire.
__device__ __forceinline__ unsigned long long same_entry_lanes(uint32_t e, int bits, bool valid) {
    unsigned long long m = __builtin_amdgcn_ballot_w64(valid);
    for (int b = 0; b < bits; ++b) {
        const bool bit = (e >> b) & 1u;
        const unsigned long long set = __builtin_amdgcn_ballot_w64(bit);
        m &= bit ? set : ~set;
    }
    return m;
}
constexpr int kMuChunk = 2048, kMuHeld = 4096;        // vectors of a chunk; most vectors that stay in LDS over the iterations
template <int E>
__global__ void __launch_bounds__(1024) mu_kmeans_kernel(MuArgs a, int hold) {
    constexpr int S = 1024 / (2 * E);                 // threads per (entry, coordinate) = shares of a chunk
    constexpr int kChunk = kMuChunk, kPer = kChunk / S;   // vectors per chunk and per share
    constexpr int kBits = E == 64 ? 6 : 8, kH = kChunk / 1024;
    static_assert(S <= 16 && kPer % 64 == 0, "a wavefront per share, rounds of 64 vectors");
    extern __shared__ float4_t held[];                // the weight's two elements and their two squared activations, per vector
    __shared__ __attribute__((aligned(16))) float cb[E][2];
    __shared__ uint16_t s_idx[kChunk], s_at[kChunk];  // entry of a vector; vectors of a share in order of their entries
    __shared__ uint32_t first[S][E];                  // a share's first slot of an entry; while counting: vectors seen
    __shared__ uint32_t count[S][E];
    __shared__ double num[2 * E][S], den[2 * E][S];
    const MuTensor t = a.t[blockIdx.x];
    const int V = t.n >> 1, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int e = tid; e < E; e += 1024) {
        cb[e][0] = f16_bits_to_f32(t.cb[2 * e]);
        cb[e][1] = f16_bits_to_f32(t.cb[2 * e + 1]);
    }
    __syncthreads();
    const int pair = tid / S, seg = tid % S;          // update phase: pair = 2 e + coordinate
    for (int it = 0; it <= a.iters; ++it) {
        const bool last = it == a.iters;
        double sn = 0.0, sd = 0.0;
        for (int c0 = 0; c0 < V; c0 += kChunk) {
            const int in_chunk = V - c0 < kChunk ? V - c0 : kChunk;
            float4_t* const chunk = held + (hold ? c0 : 0);
            if (it == 0 || !hold) {
                if (!hold && it + c0 > 0) __syncthreads();
#pragma unroll
                for (int h = 0; h < kH; ++h) {
                    const int vl = h * 1024 + tid, v = min(c0 + vl, V - 1);
                    const float x0 = t.xbar[2 * (size_t)v], x1 = t.xbar[2 * (size_t)v + 1];
                    chunk[vl] = float4_t{load_as_f32(t.mu, 2 * (size_t)v, a.dt), load_as_f32(t.mu, 2 * (size_t)v + 1, a.dt),
                                         __fmul_rn(x0, x0), __fmul_rn(x1, x1)};
                }
            }
            auto assign = [&](auto count) {           // a thread's own vectors, the entries read once for all of them
                constexpr int H = decltype(count)::value;
                float4_t v[H];
                int best[H];
                float bestc[H];
#pragma unroll
                for (int h = 0; h < H; ++h) { v[h] = chunk[h * 1024 + tid]; best[h] = 0; bestc[h] = __builtin_inff(); }
#pragma unroll 4
                for (int e = 0; e < E; e += 2) {
                    const float4_t two = *(const float4_t*)&cb[e][0];
#pragma unroll
                    for (int k = 0; k < 2; ++k)
#pragma unroll
                        for (int h = 0; h < H; ++h) {
                            const float t0 = __fsub_rn(v[h].x, k ? two.z : two.x), t1 = __fsub_rn(v[h].y, k ? two.w : two.y);
                            const float c = __fadd_rn(__fmul_rn(v[h].z, __fmul_rn(t0, t0)), __fmul_rn(v[h].w, __fmul_rn(t1, t1)));
                            if (c < bestc[h]) { bestc[h] = c; best[h] = e + k; }
                        }
                }
#pragma unroll
                for (int h = 0; h < H; ++h) {
                    const int vl = h * 1024 + tid;
                    if (vl >= in_chunk) continue;
                    if (last) t.idx[c0 + vl] = (uint8_t)best[h];
                    else s_idx[vl] = (uint16_t)best[h];
                }
            };
            if (1024 + 64 * wave < in_chunk) assign(std::integral_constant<int, kH>{});
            else if (64 * wave < in_chunk) assign(std::integral_constant<int, 1>{});
            if (last) continue;                       // the final pass only assigns
            if (tid < S * E) (&count[0][0])[tid] = 0u;
            __syncthreads();
            if (wave < S) {                           // order share `wave` by entries
                uint32_t e[kPer / 64], rank[kPer / 64];
#pragma unroll
                for (int r = 0; r < kPer / 64; ++r) {
                    const int vl = wave * kPer + 64 * r + lane;
                    const bool valid = vl < in_chunk;
                    e[r] = valid ? s_idx[vl] : 0u;
                    const unsigned long long m = same_entry_lanes(e[r], kBits, valid);
                    const uint32_t below = (uint32_t)__builtin_popcountll(m & ((1ull << lane) - 1ull)), old = count[wave][e[r]];
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");     // a wavefront's LDS accesses are served in order
                    __builtin_amdgcn_wave_barrier();
                    if (valid && below == 0u) count[wave][e[r]] = old + (uint32_t)__builtin_popcountll(m);
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                    rank[r] = old + below;
                }
                uint32_t run = 0;                     // first slots: running sum over the entries, 64 at a time
#pragma unroll
                for (int e0 = 0; e0 < E; e0 += 64) {
                    const uint32_t c = count[wave][e0 + lane];
                    uint32_t incl = c;
#pragma unroll
                    for (int off = 1; off < 64; off <<= 1) {
                        const uint32_t up = __shfl_up(incl, off, 64);
                        if (lane >= off) incl += up;
                    }
                    first[wave][e0 + lane] = run + incl - c;
                    run += __shfl(incl, 63, 64);
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
                for (int r = 0; r < kPer / 64; ++r) {
                    const int vl = wave * kPer + 64 * r + lane;
                    if (vl < in_chunk) s_at[wave * kPer + first[wave][e[r]] + rank[r]] = (uint16_t)vl;
                }
            }
            __syncthreads();
            {
                const int c = pair & 1;
                const uint32_t at = seg * kPer + first[seg][pair >> 1], cnt = count[seg][pair >> 1];
#pragma unroll 8
                for (uint32_t i = 0; i < cnt; ++i) {  // eight vectors' look-ups at a time: an entry may hold a whole share
                    const int vl = s_at[at + i];
                    const float* vec = (const float*)&chunk[vl];
                    const double w = (double)vec[2 + c];
                    sn += w * (double)vec[c];    // the product of two binary32 values is exact in binary64
                    sd += w;
                }
            }
            __syncthreads();
        }
        if (last) break;
        num[pair][seg] = sn;
        den[pair][seg] = sd;
        __syncthreads();
        for (int p = tid; p < 2 * E; p += 1024) {
            double tn = 0.0, td = 0.0;
#pragma unroll
            for (int g = 0; g < S; ++g) { tn += num[p][g]; td += den[p][g]; }
            if (td > 0.0) (&cb[0][0])[p] = f16_bits_to_f32(f64_to_f16_bits(tn / td));
        }
        __syncthreads();
    }
    __syncthreads();
    for (int e = tid; e < 2 * E; e += 1024) t.cb[e] = f32_to_f16_bits((&cb[0][0])[e]);
}

hipError_t launch_mu_codebook(const void* const* mus, const float* const* xbars, const int* n_elems, int n_tensors,
                              int dt, int kbits, int iters, void* const* cbs, uint8_t* const* idx, hipStream_t s) {
    for (int base = 0; base < n_tensors; base += kMuMaxTensors) {
        MuArgs a;
        const int cnt = n_tensors - base < kMuMaxTensors ? n_tensors - base : kMuMaxTensors;
        for (int i = 0; i < kMuMaxTensors; ++i) {
            const int k = base + (i < cnt ? i : 0);
            a.t[i] = MuTensor{mus[k], xbars[k], (uint16_t*)cbs[k], idx[k], n_elems[k], 0};
        }
        a.dt = dt; a.kbits = kbits; a.iters = iters; a.pad = 0;
        int most = 0;
        for (int i = 0; i < cnt; ++i) most = std::max(most, n_elems[base + i] / 2);
        const int hold = most <= kMuHeld, chunks = hold ? (most + kMuChunk - 1) / kMuChunk : 1, lds = chunks * kMuChunk * 16;
        static std::atomic<unsigned long long> raised[2];
        hipError_t e = raise_lds(kbits == 6 ? (const void*)mu_kmeans_kernel<64> : (const void*)mu_kmeans_kernel<256>, kMuHeld * 16, raised[kbits == 6]);
        if (e != hipSuccess) return e;
        if (kbits == 6) hipLaunchKernelGGL(mu_kmeans_kernel<64>, dim3(cnt), dim3(1024), lds, s, a, hold);
        else hipLaunchKernelGGL(mu_kmeans_kernel<256>, dim3(cnt), dim3(1024), lds, s, a, hold);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---------------------------------------------------------------------------------- token-shift mix
constexpr int kMixMaxProj = 8;
struct MixArgs {
    const void* x;           // [M][d]
    const void* x_prev;      // [d]: the token before row 0
    const uint8_t* idx[kMixMaxProj];    // [d / 2] per projection
    const uint16_t* cb[kMixMaxProj];    // fp16 [E][2] per projection
    void* out[kMixMaxProj];             // [M][d] per projection
    int M, d, dt, n_proj, E, pad;
};

// A thread owns 8 consecutive channels of one row: one 16-byte load of x_t, one of x_{t-1}, and per
// projection four index bytes, four codebook look-ups (codebooks staged in LDS) and one 16-byte
// store.  HBM-bound: 2 (n_proj + 1) bytes per element (x_{t-1} is x_t's neighbouring row, a cache hit).
template <bool BF16> struct MixElem;
template <> struct MixElem<true> {
    static __device__ __forceinline__ void widen(uint32_t w, float& lo, float& hi) {
        lo = __uint_as_float(w << 16); hi = __uint_as_float(w & 0xFFFF0000u);
    }
    static __device__ __forceinline__ uint32_t narrow(float lo, float hi) {      // v_cvt_pk_bf16_f32: nearest even
        typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
        bf2 v = {(__bf16)lo, (__bf16)hi};
        return __builtin_bit_cast(uint32_t, v);
    }
};
template <> struct MixElem<false> {
    static __device__ __forceinline__ void widen(uint32_t w, float& lo, float& hi) {
        const half2_t h = __builtin_bit_cast(half2_t, w);
        const half_t a = h.x, b = h.y;
        lo = (float)a; hi = (float)b;
    }
    static __device__ __forceinline__ uint32_t narrow(float lo, float hi) {
        half2_t v = {(half_t)lo, (half_t)hi};
        return __builtin_bit_cast(uint32_t, v);
    }
};

template <bool BF16>
__global__ void __launch_bounds__(256) token_shift_mix_kernel(MixArgs a) {
    __shared__ uint32_t cbs[kMixMaxProj][256];
    for (int i = threadIdx.x; i < a.n_proj * a.E; i += 256) {
        const int p = i / a.E, e = i - p * a.E;
        cbs[p][e] = ((const uint32_t*)a.cb[p])[e];
    }
    __syncthreads();
    const int chunks = a.d >> 3;
    // Workgroups are dealt round-robin to the 8 XCDs, each with its own L2: give every XCD one
    // contiguous range of rows, so that x_{t-1} (the row above) is in the L2 that just read it as x_t
    // (with the plain order the two reads of a row came from different XCDs: twice the fetches).
    const int per_xcd = gridDim.x >> 3;                    // the grid is a multiple of 8 workgroups
    const long long blk = (long long)(blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    const long long g = blk * 256 + threadIdx.x;
    if (g >= (long long)a.M * chunks) return;
    const int row = (int)(g / chunks), c = (int)(g - (long long)row * chunks);
    const uint4_t xt = ((const uint4_t*)a.x)[(size_t)row * chunks + c];
    const uint4_t xp = row == 0 ? ((const uint4_t*)a.x_prev)[c] : ((const uint4_t*)a.x)[(size_t)(row - 1) * chunks + c];
    const uint32_t xtw[4] = {xt.x, xt.y, xt.z, xt.w}, xpw[4] = {xp.x, xp.y, xp.z, xp.w};
    float t[8], u[8];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        MixElem<BF16>::widen(xtw[q], t[2 * q], t[2 * q + 1]);
        MixElem<BF16>::widen(xpw[q], u[2 * q], u[2 * q + 1]);
    }
    for (int p = 0; p < a.n_proj; ++p) {
        const uint32_t four = ((const uint32_t*)a.idx[p])[c];      // channels 8c..8c+7 = vectors 4c..4c+3
        uint32_t ow[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float m0, m1;
            MixElem<false>::widen(cbs[p][(four >> (8 * q)) & 255u], m0, m1);
            const float o0 = __fadd_rn(__fmul_rn(m0, t[2 * q]), __fmul_rn(__fsub_rn(1.0f, m0), u[2 * q]));
            const float o1 = __fadd_rn(__fmul_rn(m1, t[2 * q + 1]), __fmul_rn(__fsub_rn(1.0f, m1), u[2 * q + 1]));
            ow[q] = MixElem<BF16>::narrow(o0, o1);
        }
        // written once, read by a later launch: stored with the non-temporal hint, so that the outputs do not
        // displace the rows of x (each read twice, as x_t and as x_{t-1}) from the L2
        __builtin_nontemporal_store(uint4_t{ow[0], ow[1], ow[2], ow[3]}, (uint4_t*)a.out[p] + (size_t)row * chunks + c);
    }
}

hipError_t launch_token_shift_mix(const void* x, const void* x_prev, int dt, int M, int d, const uint8_t* const* idx,
                                  const void* const* cbs, int kbits, int n_proj, void* const* outs, hipStream_t s) {
    MixArgs a;
    a.x = x; a.x_prev = x_prev;
    for (int p = 0; p < kMixMaxProj; ++p) {
        const int k = p < n_proj ? p : 0;
        a.idx[p] = idx[k]; a.cb[p] = (const uint16_t*)cbs[k]; a.out[p] = outs[k];
    }
    a.M = M; a.d = d; a.dt = dt; a.n_proj = n_proj; a.E = 1 << kbits; a.pad = 0;
    const long long threads = (long long)M * (d >> 3);
    const dim3 grid((unsigned)((((threads + 255) / 256) + 7) / 8 * 8));
    if (dt == DT_BF16) hipLaunchKernelGGL(token_shift_mix_kernel<true>, grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL(token_shift_mix_kernel<false>, grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace rwkvq

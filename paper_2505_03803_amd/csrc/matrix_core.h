// What the matrix-core kernels for large batches share: operand types, the decoding of packed words into operands
// (Deq(W) of Sec. 2.2 rounded once to the type of x) and the layout of an activation tile in LDS.
#pragma once
#include "common.h"

#include <algorithm>

namespace rwkvq {

// How long a launch runs, in column tiles (256 columns of W) that a compute unit works through one after another: workgroups
// go to 256 compute units, those with a long K first.  `tail`: how much of the shortest workgroup the end of the launch leaves
// some compute units without work.
struct LaunchLoad {
    long long wgs = 0;
    double work = 0.0;
    int longest = 0, shortest = 0x7FFFFFFF;
    void add(long long n, int K) {
        const int k = K >> 8;
        wgs += n; work += (double)n * k;
        longest = std::max(longest, k); shortest = std::min(shortest, k);
    }
    double columns(double tail) const {
        if (longest == shortest && wgs <= 512) return (double)(longest * ((wgs + 255) / 256));
        return wgs <= 256 ? (double)longest : std::max((double)longest, work / 256.0 + tail * shortest);
    }
};

constexpr int kRowBytes = 128;                 // a row of an operand tile in LDS: 64 k * 2 B

// s_waitcnt immediates (gfx9 encoding): only the named counter is waited for.
#define RWKVQ_WAIT_VM0_LGKM0() __builtin_amdgcn_s_waitcnt(0x0070)   /* vmcnt(0) lgkmcnt(0) */
#define RWKVQ_WAIT_VM8_LGKM0() __builtin_amdgcn_s_waitcnt(0x0078)   /* vmcnt(8) lgkmcnt(0) */
#define RWKVQ_WAIT_VM4_LGKM0() __builtin_amdgcn_s_waitcnt(0x0074)   /* vmcnt(4) lgkmcnt(0) */
// Publish LDS writes (ds_write and load-unit copies) to the workgroup: the caller has waited for
// its own writes; the barrier orders them against the other wavefronts' reads.
#define RWKVQ_BARRIER() asm volatile("s_barrier" ::: "memory")

template <bool BF16> struct Elem;
template <> struct Elem<true> {
    // accumulate in place; the "a" constraint pins the accumulator to the AGPR half of the
    // register file (left to itself the allocator starts it in VGPRs and shuffles it all loop long)
    static __device__ __forceinline__ void mfma(uint4_t a, uint4_t b, float4_t& c) {
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
    }
    static __device__ __forceinline__ uint32_t pack(float lo, float hi) {   // v_cvt_pk_bf16_f32
        typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
        bf2 v = {(__bf16)lo, (__bf16)hi};
        return __builtin_bit_cast(uint32_t, v);
    }
    static __device__ __forceinline__ uint32_t from_f16x2(uint32_t h) {
        half2_t v = __builtin_bit_cast(half2_t, h);
        return pack((float)v.x, (float)v.y);
    }
};
template <> struct Elem<false> {
    static __device__ __forceinline__ void mfma(uint4_t a, uint4_t b, float4_t& c) {
        asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
    }
    static __device__ __forceinline__ uint32_t pack(float lo, float hi) {
        half2_t v = {(half_t)lo, (half_t)hi};
        return __builtin_bit_cast(uint32_t, v);
    }
    static __device__ __forceinline__ uint32_t from_f16x2(uint32_t h) { return h; }
};

// Field c (compile-time) of a native SQ unit.
template <int C>
__device__ __forceinline__ uint32_t sq_code(uint32_t w0, uint32_t w1, uint32_t w2) {
    constexpr int P = C >> 1, e = C & 1;
    if constexpr (P < 15) {
        uint32_t w = (P / 5 == 0) ? w0 : (P / 5 == 1) ? w1 : w2;
        return (w >> (1 + 3 * (P % 5) + 16 * e)) & 7u;
    } else {
        constexpr int b = 16 * e;
        return ((w0 >> b) & 1u) | (((w1 >> b) & 1u) << 1) | (((w2 >> b) & 1u) << 2);
    }
}
template <int P>
__device__ __forceinline__ uint32_t vq6_byteaddr(uint32_t w0, uint32_t w1, uint32_t w2) {
    if constexpr (P < 15) {
        uint32_t w = (P / 5 == 0) ? w0 : (P / 5 == 1) ? w1 : w2;
        return (w >> (6 * (P % 5))) & 0xFCu;
    } else {
        return ((w0 & 3u) << 2) | ((w1 & 3u) << 4) | ((w2 & 3u) << 6);
    }
}

// The two weights of pair P of a native SQ unit, dequantised as Sec. 2.2 Eq. "SQ" prescribes
// (q - z rounded, times s rounded).  The codes are not extracted: masked in place, a 3-bit code at
// mantissa bits b..b+2 of an fp16 half is the subnormal q * 2^(b-24); a mixed-precision FMA reads
// the half, multiplies by 2^(24-b) (exact) and subtracts z with the single rounding of q - z.  The
// codes at bits 10 and 13 of the halves come down to bits 1 and 4 with one shift by 9 per word.
template <int P>
__device__ __forceinline__ void sq_pair_deq(uint32_t w0, uint32_t w1, uint32_t w2, float s, float z, float& lo,
                                            float& hi) {
    uint32_t m;
    float c;
    if constexpr (P < 15) {
        constexpr int p = P % 5;
        const uint32_t w = (P / 5 == 0) ? w0 : (P / 5 == 1) ? w1 : w2;
        if constexpr (p == 0) { m = w & 0x000E000Eu; c = 8388608.f; }
        else if constexpr (p == 1) { m = w & 0x00700070u; c = 1048576.f; }
        else if constexpr (p == 2) { m = w & 0x03800380u; c = 131072.f; }
        else if constexpr (p == 3) { m = (w >> 9) & 0x000E000Eu; c = 8388608.f; }
        else { m = (w >> 9) & 0x00700070u; c = 1048576.f; }
    } else {
        // bit b of the pair's two codes sits at bits 0 and 16 of word b
        m = (w0 & 0x00010001u) | ((w1 & 0x00010001u) << 1) | ((w2 & 0x00010001u) << 2);
        c = 16777216.f;
    }
    const half2_t h = __builtin_bit_cast(half2_t, m);
    lo = __fmul_rn(fmaf((float)h.x, c, -z), s);
    hi = __fmul_rn(fmaf((float)h.y, c, -z), s);
}

// The SQ pair P as masked in-place codes (fp16 subnormals q * 2^(b-24)) and the power of two that
// undoes the position (see sq_pair_deq).
template <int P>
__device__ __forceinline__ uint32_t sq_pair_mask(uint32_t w0, uint32_t w1, uint32_t w2) {
    if constexpr (P < 15) {
        constexpr int p = P % 5;
        const uint32_t w = (P / 5 == 0) ? w0 : (P / 5 == 1) ? w1 : w2;
        if constexpr (p == 0) return w & 0x000E000Eu;
        else if constexpr (p == 1) return w & 0x00700070u;
        else if constexpr (p == 2) return w & 0x03800380u;
        else if constexpr (p == 3) return (w >> 9) & 0x000E000Eu;
        else return (w >> 9) & 0x00700070u;
    } else {
        return (w0 & 0x00010001u) | ((w1 & 0x00010001u) << 1) | ((w2 & 0x00010001u) << 2);
    }
}
template <int P> constexpr float sq_pair_unscale() {
    return P == 15 ? 16777216.f : (P % 5 == 0 || P % 5 == 3) ? 8388608.f : (P % 5 == 1 || P % 5 == 4) ? 1048576.f : 131072.f;
}

// Eight consecutive-k weights (step T4 of a unit) of one lane, as four packed pairs.
template <bool BF16, int T4>
__device__ __forceinline__ uint4_t sq_chunk(uint32_t w0, uint32_t w1, uint32_t w2, float s, float z) {
    uint4_t o;
    float a, b;
    sq_pair_deq<4 * T4 + 0>(w0, w1, w2, s, z, a, b); o.x = Elem<BF16>::pack(a, b);
    sq_pair_deq<4 * T4 + 1>(w0, w1, w2, s, z, a, b); o.y = Elem<BF16>::pack(a, b);
    sq_pair_deq<4 * T4 + 2>(w0, w1, w2, s, z, a, b); o.z = Elem<BF16>::pack(a, b);
    sq_pair_deq<4 * T4 + 3>(w0, w1, w2, s, z, a, b); o.w = Elem<BF16>::pack(a, b);
    return o;
}
template <int T4>
__device__ __forceinline__ uint4_t vq6_chunk(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t cb) {
    uint4_t o;
    o.x = __builtin_amdgcn_ds_bpermute(vq6_byteaddr<4 * T4 + 0>(w0, w1, w2), cb);
    o.y = __builtin_amdgcn_ds_bpermute(vq6_byteaddr<4 * T4 + 1>(w0, w1, w2), cb);
    o.z = __builtin_amdgcn_ds_bpermute(vq6_byteaddr<4 * T4 + 2>(w0, w1, w2), cb);
    o.w = __builtin_amdgcn_ds_bpermute(vq6_byteaddr<4 * T4 + 3>(w0, w1, w2), cb);
    return o;
}
__device__ __forceinline__ uint4_t vq8_chunk(uint32_t w, const uint32_t* cb) {
    uint4_t o = {cb[w & 255u], cb[(w >> 8) & 255u], cb[(w >> 16) & 255u], cb[w >> 24]};
    return o;
}

// LDS byte offset, inside a tile, of logical 16-byte chunk c (0..7) of row `row`.
__device__ __forceinline__ int tile_off(int row, int c) { return row * kRowBytes + ((c ^ (row & 7)) << 4); }

}  // namespace rwkvq

// What the matrix-core kernels share: operand types, the decoding of packed words into operands (Deq(W) of Sec. 2.2 rounded
// once to the type of x, or unrounded codes and entries), bf16 activations under a scale and the layout of an activation tile in LDS.
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

// ---- unrounded weights (the streaming kernels' contract) ------------------------------------------------------------
#define RWKVQ_MFMA(a, b, c) __builtin_amdgcn_mfma_f32_16x16x32_f16((a), (b), (c), 0, 0, 0)
template <bool BF16>
__device__ __forceinline__ float4_t mfma_bits(uint4_t x, uint4_t w, float4_t c) {
    if constexpr (BF16) return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, x), __builtin_bit_cast(bf16x8_t, w), c, 0, 0, 0);
    else return RWKVQ_MFMA(__builtin_bit_cast(half8_t, x), __builtin_bit_cast(half8_t, w), c);
}

// Two 3-bit codes as a pair of 8 + q, exact in either type: fp16 with the codes at mantissa bits 7 .. 9 (mask 0x03800380, magic
// 0x48004800), bf16 at bits 4 .. 6 (0x00700070, 0x41004100).  y += s (acc - (8 + z) X) per group, X from an MFMA against ones.
template <bool BF16, int P>
__device__ __forceinline__ uint32_t sq_pair_code(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t mask, uint32_t magic) {
    constexpr int at = BF16 ? 4 : 7;
    if constexpr (P < 15) {
        constexpr int p = P % 5, sh = at - 1 - 3 * p;
        uint32_t w = (P / 5 == 0) ? w0 : (P / 5 == 1) ? w1 : w2;
        uint32_t v = sh > 0 ? (w << (sh > 0 ? sh : 0)) : sh < 0 ? (w >> (sh < 0 ? -sh : 0)) : w;
        return (v & mask) | magic;
    } else {
        // bit b of the pair's two codes sits at bits 0 and 16 of word b
        uint32_t v = (w0 & 0x00010001u) | ((w1 & 0x00010001u) << 1) | ((w2 & 0x00010001u) << 2);
        return (v << at) | magic;
    }
}
// Its mask in a VGPR and magic in an SGPR: a VOP3 instruction of this ISA takes no literal and at most one scalar operand.
template <bool BF16>
__device__ __forceinline__ void sq_code_constants(uint32_t& mask, uint32_t& magic) {
    asm("v_mov_b32 %0, %1" : "=v"(mask) : "n"(BF16 ? 0x00700070 : 0x03800380));
    asm("s_mov_b32 %0, %1" : "=s"(magic) : "n"(BF16 ? 0x41004100 : 0x48004800));
}
template <bool BF16> constexpr uint32_t kSqOne = BF16 ? 0x3F803F80u : 0x3C003C00u;

template <bool BF16, int T>
__device__ __forceinline__ uint4_t sq_operand(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t mask, uint32_t magic) {
    return uint4_t{sq_pair_code<BF16, 4 * T + 0>(w0, w1, w2, mask, magic), sq_pair_code<BF16, 4 * T + 1>(w0, w1, w2, mask, magic),
                   sq_pair_code<BF16, 4 * T + 2>(w0, w1, w2, mask, magic), sq_pair_code<BF16, 4 * T + 3>(w0, w1, w2, mask, magic)};
}

// A codebook entry (two fp16) as the sum of two bf16 pairs (8 and 3 of the 11 bits, exact), which are multiplied in turn.
__device__ __forceinline__ uint2_t vq_split(uint32_t e) {
    const half2_t v = __builtin_bit_cast(half2_t, e);
    const uint32_t h = Elem<true>::from_f16x2(e);
    return uint2_t{h, Elem<true>::pack((float)v.x - __uint_as_float(h << 16), (float)v.y - __uint_as_float(h & 0xFFFF0000u))};
}

typedef unsigned short ushort2_t __attribute__((ext_vector_type(2)));

// Exponent n of the scale 2^n for a group whose largest bf16 magnitude has the bits `amax`: the
// largest lands in [2^15, 2^16).  An all-zero (or tiny) group takes the largest n whose inverse
// 2^-n is still a normal binary32 number.
__device__ __forceinline__ int bf16_scale_exponent(uint32_t amax) {
    const int e = (int)(amax >> 7);                 // biased exponent, 0..254 for finite values
    return 142 - (e > 16 ? e : 16);
}
// Two bf16 -> two fp16, each multiplied by 2^n first.  Exact where fp16 can hold the product.
__device__ __forceinline__ uint32_t bf16x2_to_f16x2(uint32_t v, int n) {
    const float lo = ldexpf(__builtin_bit_cast(float, v << 16), n);
    const float hi = ldexpf(__builtin_bit_cast(float, v & 0xFFFF0000u), n);
    return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(lo, hi));
}

// A 256-column tile of sixteen rows of x as the MFMA's A operands, straight from memory: lane (m, kg) = (lane % 16, lane / 16) holds,
// for column half u and k-step t, the eight consecutive activations 128 u + 32 t + 8 kg ... of row m in f[4 u + t].
struct XFrags { uint4_t f[8]; };
// COUNT bf16 fragments -> fp16: the exponent of the scale is that of the row's largest magnitude among them (the four lanes
// that hold a row agree through two exchanges).
template <int COUNT>
__device__ __forceinline__ int x_frags_exponent(const uint4_t (&f)[COUNT]) {
    uint32_t amax = 0;
    ushort2_t most = {0, 0};
#pragma unroll
    for (int i = 0; i < COUNT; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) most = __builtin_elementwise_max(most, __builtin_bit_cast(ushort2_t, f[i][j] & 0x7FFF7FFFu));
    amax = max((uint32_t)most.x, (uint32_t)most.y);
    auto both = __builtin_amdgcn_permlane16_swap(amax, amax, false, false);      // the other three lanes of the row
    amax = max((uint32_t)both[0], (uint32_t)both[1]);
    both = __builtin_amdgcn_permlane32_swap(amax, amax, false, false);
    return bf16_scale_exponent(max((uint32_t)both[0], (uint32_t)both[1]));
}
__device__ __forceinline__ uint4_t x_frag_to_f16(const uint4_t& f, int n) {
    return uint4_t{bf16x2_to_f16x2(f.x, n), bf16x2_to_f16x2(f.y, n), bf16x2_to_f16x2(f.z, n), bf16x2_to_f16x2(f.w, n)};
}

// Sums of bf16 activations as they are that leave binary32.  x goes to 3.4e38, a group's sum is up to 2^7 times as large and (8 + z)
// times that up to 2^16 times more (z is any fp16), where s times the difference may be any finite number; the same with entries, whose
// products may cancel; and an infinite entry is the sum of an infinity and a NaN.  Such a sum ends as an
// infinity or a NaN, whatever follows; the wavefront then takes its column tiles again for the sixteen rows of W and of x, with x
// brought into fp16 under exact power-of-two scales, and from there the elements that were not finite.  What is finite costs a test
// per element at the end of the wavefront's work: 1218 calls at 2 to 48 rows of x took 0.997 of the time before in the median.
// (The codes as 2^-12 (8 + q) kept a group's sums finite, not their products with 8 + z, and lost bits of activations below 2^-114.)
//
// Row tile `row_tile` of W (unpacked plainly: this is rare) times rows m0 .. m0 + 15 of x (those past M repeat row M - 1), column
// tiles t0, t0 + ts, ..; D layout of the MFMA: lane (n, mg) holds rows 4 mg .. 4 mg + 3 of x for row n of W.
template <class Mat>
__device__ __forceinline__ float4_t scaled_row_tile(const Mat& mt, int row_tile, int m0, int M, int t0, int ts, int lane) {
    const int KT = mt.K >> 8, m = m0 + (lane & 15) < M ? m0 + (lane & 15) : M - 1;
    const uint16_t* const xrow = (const uint16_t*)mt.x + (size_t)m * mt.K + 8 * (lane >> 4);
    const uint32_t one = kSqOne<false>;
    float4_t out = {0, 0, 0, 0};
    // 32 columns at a time: no more in registers than the loops before this have room for
#pragma unroll 1
    for (int T = t0; T < KT; T += ts) {
        int n = 142;                                                                        // the tile's scale: the least of the eight
#pragma unroll 1
        for (int i = 0; i < 8; ++i) {
            const uint4_t x[1] = {*(const uint4_t*)(xrow + 256 * T + 32 * i)};
            n = min(n, x_frags_exponent(x));
        }
        const uint32_t* const t = mt.codes + ((size_t)row_tile * KT + T) * (mt.fmt == FMT_VQ8 ? 512 : 384);
        const uint32_t* const a = t + 4 * lane;                                             // the lane's words: a[0] .. a[3], b[0], b[1]
        const uint32_t* const b = t + 256 + 2 * lane;
        const uint32_t* const book = (const uint32_t*)mt.aux + ((size_t)(row_tile >> 4) * KT + T) * (mt.fmt == FMT_VQ8 ? 256 : 64);
        float4_t part = {0, 0, 0, 0};
#pragma unroll 1
        for (int at = 0; at < 8; ++at) {
            const int u = at >> 2, k = at & 3;
            uint32_t op[4];
            if (mt.fmt == FMT_VQ8) {
                const uint32_t w = a[256 * u + k];
#pragma unroll
                for (int i = 0; i < 4; ++i) op[i] = book[(w >> (8 * i)) & 255u];
            } else {
                const uint32_t w[3] = {u == 0 ? a[0] : a[3], u == 0 ? a[1] : b[0], u == 0 ? a[2] : b[1]};
#pragma unroll
                for (int i = 0; i < 4; ++i) {                                               // as vq6_byteaddr and sq_pair_code
                    const int P = 4 * k + i;
                    const uint32_t word = P < 5 ? w[0] : P < 10 ? w[1] : w[2];
                    const uint32_t index = P == 15 ? (w[0] & 3u) | (w[1] & 3u) << 2 | (w[2] & 3u) << 4 : word >> (6 * (P % 5) + 2) & 63u;
                    const uint32_t codes = P == 15 ? ((w[0] & 0x00010001u) | (w[1] & 0x00010001u) << 1 | (w[2] & 0x00010001u) << 2) << 7
                                                   : word >> (3 * (P % 5)) << 6 & 0x03800380u;
                    op[i] = mt.fmt == FMT_SQ3 ? codes | 0x48004800u : book[index];
                }
            }
            const uint4_t f = x_frag_to_f16(*(const uint4_t*)(xrow + 256 * T + 32 * at), n);
            const float4_t zero = {0, 0, 0, 0};
            const float4_t sum = mfma_bits<false>(f, uint4_t{op[0], op[1], op[2], op[3]}, mt.fmt == FMT_SQ3 ? zero : part);
            if (mt.fmt == FMT_SQ3) {
                const float4_t X = mfma_bits<false>(f, uint4_t{one, one, one, one}, zero);
                const uint32_t szw = ((const uint32_t*)mt.aux)[(((size_t)row_tile * KT + T) * 16 + (lane & 15)) * 2 + u];
                const float s = f16_bits_to_f32((uint16_t)(szw & 0xFFFFu)), z8 = f16_bits_to_f32((uint16_t)(szw >> 16)) + 8.0f;
#pragma unroll
                for (int i = 0; i < 4; ++i) part[i] = fmaf(s, fmaf(-z8, X[i], sum[i]), part[i]);
            } else {
                part = sum;
            }
        }
        const float inverse = ldexpf(1.0f, -n);
#pragma unroll
        for (int i = 0; i < 4; ++i) out[i] = fmaf(part[i], __shfl(inverse, 4 * (lane >> 4) + i, 64), out[i]);
    }
    return out;
}
// Is any of a wavefront's sums not finite?
template <int COUNT>
__device__ __forceinline__ bool any_infinite(const float4_t (&out)[COUNT]) {
    float none = 0.0f;                             // 0, or NaN if one of them is not finite
#pragma unroll
    for (int j = 0; j < COUNT; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) none = fmaf(out[j][i], 0.0f, none);
    return __builtin_amdgcn_ballot_w64(none == 0.0f) != __builtin_amdgcn_ballot_w64(true);
}
__device__ __forceinline__ float4_t if_infinite(float4_t v, const float4_t& again) {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = fabsf(v[i]) < __builtin_inff() ? v[i] : again[i];
    return v;
}

}  // namespace rwkvq

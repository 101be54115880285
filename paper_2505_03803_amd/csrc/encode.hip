// The two encoders of Sec. 2.2: round-to-nearest scalar quantization (Eq. "SQ") and assignment of
// each weight pair to its nearest codebook entry (Eq. "VQ").  Dense weights in, canonical-layout
// codes / indices out (per-row little-endian bit strings, see include/rwkvq.h).  Every
// floating-point step is one binary32 operation rounded to nearest even, written with the
// intrinsics so that the compiler can neither fuse nor reorder them: the codes are integers and
// must come out the same as from any other implementation of these steps.
#include "common.h"

#include <type_traits>

#ifndef RWKVQ_SQ_ENCODE_PASSES
#define RWKVQ_SQ_ENCODE_PASSES 1   // stretches of 32 groups per workgroup of the SQ encoder
#endif

namespace rwkvq {

// Three-operand minimum / maximum and one butterfly step of a minimum / maximum across lanes
// (the data-parallel-primitive form of the instruction reads its first operand from the partner
// lane).  Written as instructions: the C library forms first canonicalise every operand, which
// doubles their cost, and keep the cross-lane move a separate instruction.  The two idle cycles
// in front of a cross-lane read are the ones the architecture asks for after a vector write of
// the register it reads.
__device__ __forceinline__ float min3f(float a, float b, float c) {
    float r;
    asm("v_min3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
__device__ __forceinline__ float max3f(float a, float b, float c) {
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
#define RWKVQ_LANE_STEP(op, v, ctrl) \
    asm volatile("s_nop 1\n\t" op " %0, %1, %1 " ctrl " row_mask:0xf bank_mask:0xf" : "=v"(v) : "v"(v))
// over the eight lanes of half a DPP row: quad permutes [1,0,3,2] and [2,3,0,1], then the mirror of the half row
__device__ __forceinline__ float half_row_min(float v) {
    RWKVQ_LANE_STEP("v_min_f32_dpp", v, "quad_perm:[1,0,3,2]");
    RWKVQ_LANE_STEP("v_min_f32_dpp", v, "quad_perm:[2,3,0,1]");
    RWKVQ_LANE_STEP("v_min_f32_dpp", v, "row_half_mirror");
    return v;
}
__device__ __forceinline__ float half_row_max(float v) {
    RWKVQ_LANE_STEP("v_max_f32_dpp", v, "quad_perm:[1,0,3,2]");
    RWKVQ_LANE_STEP("v_max_f32_dpp", v, "quad_perm:[2,3,0,1]");
    RWKVQ_LANE_STEP("v_max_f32_dpp", v, "row_half_mirror");
    return v;
}

// v / d for a divisor d whose correctly rounded reciprocal r is at hand: q0 = rn(v * r), then
// correction steps q' = rn(q + rn(v - d * q) * r), whose residual one fused multiply-add gives
// exactly.  Two steps yield the correctly rounded quotient whenever nothing over- or underflows
// on the way (one makes q faithful, the second rounds it correctly: Markstein's theorem); for a
// dividend that is a bf16 or fp16 value and a divisor that is an fp16 value one step does
// (checked on the host over every such pair with the dividend zero or in [2^-60, 2^60]:
// tests/host/quotient_check.c).
template <int STEPS>
__device__ __forceinline__ float quotient(float v, float d, float r) {
    float q = __fmul_rn(v, r);
#pragma unroll
    for (int i = 0; i < STEPS; ++i) q = __fmaf_rn(__fmaf_rn(-d, q, v), r, q);
    return q;
}

// Eight lanes per (row, group of 128 columns); a lane holds columns 8 l .. 8 l + 7 and
// 64 + 8 l .. 64 + 8 l + 7 of the group (two fully coalesced 16-byte loads for 16-bit weights),
// eight groups per wavefront and pass; a workgroup makes U passes over consecutive stretches of
// 32 groups, with the loads of all passes issued before the first is used.
//   s = (max - min) / 7 -> fp16;  z = -min / s -> fp16;  q = clamp(rne(w / s + z), 0, 7)
// with the stored (fp16) s and z; a constant group, or one whose fp16 scale would be zero, takes
// s = 1, z = -min.  All divisions are exact (correctly rounded binary32): the 16 + 1 by s share
// one reciprocal, refined from the hardware's approximation by one Newton step, which lands on
// the correctly rounded reciprocal of every fp16 value when the approximation is within four
// units in the last place (checked on the host).  A lane whose values leave the range the short
// sequence is proven for (a non-zero magnitude outside [2^-60, 2^60], a non-finite scale) takes
// the hardware division sequence instead.
// A lane's eight codes of one half are 24 bits of the group's 384-bit string, gathered in a
// binary32 (an integer below 2^24, so every step is exact): the four lanes of a quad hold
// 96 bits = three words, assembled with one quad permute.
template <int STEPS>
__device__ __forceinline__ void sq_encode_group(const float (&v)[16], int lane, bool live, long long unit,
                                                uint32_t* __restrict__ codes, uint16_t* __restrict__ scales,
                                                uint16_t* __restrict__ zeros) {
    const int sub = lane & 7;
    float lo = min3f(v[0], v[1], v[2]), hi = max3f(v[0], v[1], v[2]);
#pragma unroll
    for (int i = 3; i < 15; i += 2) { lo = min3f(lo, v[i], v[i + 1]); hi = max3f(hi, v[i], v[i + 1]); }
    lo = min3f(lo, v[15], v[15]);
    hi = max3f(hi, v[15], v[15]);
    lo = half_row_min(lo);
    hi = half_row_max(hi);
    const float range = __fsub_rn(hi, lo);
    float s32;
    if (range >= 0x1p-40f && range <= 0x1p100f) s32 = quotient<2>(range, 7.0f, 0x1.24924ap-3f);   // rn(1 / 7)
    else s32 = __fdiv_rn(range, 7.0f);
    uint16_t s16 = f32_to_f16_bits(s32);
    if (hi == lo || (s16 & 0x7FFFu) == 0) s16 = f32_to_f16_bits(1.0f);
    const float s = f16_bits_to_f32(s16);
    const bool s_finite = (s16 & 0x7C00u) != 0x7C00u;
    float r = __builtin_amdgcn_rcpf(s);
    r = __fmaf_rn(__fmaf_rn(-s, r, 1.0f), r, r);
    const float alo = fabsf(lo);
    float zf;
    if (lo == 0.0f) zf = -lo;                         // a zero of the right sign (the short sequence loses the sign of a zero)
    else if (s_finite && alo >= 0x1p-60f && alo <= 0x1p60f) zf = quotient<STEPS>(-lo, s, r);
    else zf = __fdiv_rn(-lo, s);
    const uint16_t z16 = f32_to_f16_bits(zf);
    const float z = f16_bits_to_f32(z16);
    int emin = 0;                                     // binary exponents (value = m 2^e, 1/2 <= m < 1; zero counts as 0)
#pragma unroll
    for (int i = 0; i < 16; i += 2)
        emin = min(emin, min(__builtin_amdgcn_frexp_expf(v[i]), __builtin_amdgcn_frexp_expf(v[i + 1])));
    const bool plain = !s_finite || emin < -59 || !(fmaxf(alo, fabsf(hi)) <= 0x1p60f);
    float quo[16];
    if (!plain) {
#pragma unroll
        for (int i = 0; i < 16; ++i) quo[i] = quotient<STEPS>(v[i], s, r);
    } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) quo[i] = __fdiv_rn(v[i], s);
    }
    uint32_t field[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        float acc = 0.0f;
#pragma unroll
        for (int i = 7; i >= 0; --i) {                // Horner in base 8: code i lands at bits 3 i .. 3 i + 2
            const float q = rintf(__builtin_amdgcn_fmed3f(__fadd_rn(quo[8 * h + i], z), 0.0f, 7.0f));
            acc = __fmaf_rn(acc, 8.0f, q);
        }
        field[h] = (uint32_t)acc;
    }
    // quad lanes 0..3 hold f0..f3: word0 = f0 | f1 << 24, word1 = f1 >> 8 | f2 << 16, word2 = f2 >> 16 | f3 << 8
    const int ql = lane & 3;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const uint32_t f = field[h];
        const uint32_t next = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)f, 0x39, 0xF, 0xF, true);   // quad_perm [1,2,3,0]
        const uint32_t word = ql == 0 ? (f | (next << 24)) : ql == 1 ? ((f >> 8) | (next << 16)) : ((f >> 16) | (next << 8));
        if (live && ql < 3) __builtin_nontemporal_store(word, codes + (size_t)unit * 12 + 6 * h + 3 * (sub >> 2) + ql);
    }
    if (live && sub == 0) { scales[unit] = s16; zeros[unit] = z16; }
}

template <int U, int WDT>
__global__ void __launch_bounds__(256) sq_encode_kernel(const void* __restrict__ w, int N, int K,
                                                        uint32_t* __restrict__ codes, uint16_t* __restrict__ scales,
                                                        uint16_t* __restrict__ zeros) {
    const int lane = threadIdx.x & 63, sub = lane & 7;
    const long long units = (long long)N * (K / kGroup);
    long long unit[U];                                // (row, group) indices
    bool live[U];
#pragma unroll
    for (int j = 0; j < U; ++j) {
        unit[j] = ((long long)blockIdx.x * U + j) * 32 + (threadIdx.x >> 6) * 8 + (lane >> 3);
        live[j] = unit[j] < units;
        if (!live[j]) unit[j] = units - 1;            // surplus rows of lanes redo the last group, store nothing
    }
    // groups are consecutive in a row-major matrix; the dense weights are read once
    if (WDT == DT_F32) {
        float4_t a[U][4];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const float* src = (const float*)w + (size_t)unit[j] * kGroup + 8 * sub;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                a[j][2 * h] = __builtin_nontemporal_load((const float4_t*)(src + 64 * h));
                a[j][2 * h + 1] = __builtin_nontemporal_load((const float4_t*)(src + 64 * h + 4));
            }
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
            float v[16];
#pragma unroll
            for (int i = 0; i < 4; ++i) { v[4 * i] = a[j][i].x; v[4 * i + 1] = a[j][i].y; v[4 * i + 2] = a[j][i].z; v[4 * i + 3] = a[j][i].w; }
            sq_encode_group<2>(v, lane, live[j], unit[j], codes, scales, zeros);
        }
    } else {
        uint4_t p[U][2];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const uint16_t* src = (const uint16_t*)w + (size_t)unit[j] * kGroup + 8 * sub;
            p[j][0] = __builtin_nontemporal_load((const uint4_t*)src);
            p[j][1] = __builtin_nontemporal_load((const uint4_t*)(src + 64));
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const uint32_t pw[8] = {p[j][0].x, p[j][0].y, p[j][0].z, p[j][0].w, p[j][1].x, p[j][1].y, p[j][1].z, p[j][1].w};
            float v[16];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                v[2 * i] = WDT == DT_F16 ? f16_bits_to_f32((uint16_t)(pw[i] & 0xFFFFu)) : bf16_bits_to_f32((uint16_t)(pw[i] & 0xFFFFu));
                v[2 * i + 1] = WDT == DT_F16 ? f16_bits_to_f32((uint16_t)(pw[i] >> 16)) : bf16_bits_to_f32((uint16_t)(pw[i] >> 16));
            }
            sq_encode_group<1>(v, lane, live[j], unit[j], codes, scales, zeros);
        }
    }
}

// Sixteen consecutive weights (eight pairs) starting at element e, widened to binary32, with
// 16-byte loads.
__device__ __forceinline__ void load_pairs8(const void* w, int wdt, size_t e, float (&v0)[8], float (&v1)[8]) {
    if (wdt == DT_F32) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float4_t a = *(const float4_t*)((const float*)w + e + 4 * i);
            v0[2 * i] = a.x; v1[2 * i] = a.y; v0[2 * i + 1] = a.z; v1[2 * i + 1] = a.w;
        }
    } else {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint4_t p = *(const uint4_t*)((const uint16_t*)w + e + 8 * i);
            const uint32_t pw[4] = {p.x, p.y, p.z, p.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint16_t lo = (uint16_t)(pw[j] & 0xFFFFu), hi = (uint16_t)(pw[j] >> 16);
                v0[4 * i + j] = wdt == DT_F16 ? f16_bits_to_f32(lo) : bf16_bits_to_f32(lo);
                v1[4 * i + j] = wdt == DT_F16 ? f16_bits_to_f32(hi) : bf16_bits_to_f32(hi);
            }
        }
    }
}

__device__ __forceinline__ float pair_distance(float v0, float v1, float c0, float c1) {
    const float t0 = __fsub_rn(v0, c0), t1 = __fsub_rn(v1, c1);
    return __fadd_rn(__fmul_rn(t0, t0), __fmul_rn(t1, t1));
}

// Index of the nearest of all E entries for each of P pairs (step 5 below): equal distances resolve to the lowest index, an
// infinite or NaN distance to every entry gives 0.  Eight entries' loads in front of eight entries' arithmetic, nothing moved between:
// 4096 x 4096 weights against 256 entries 225 -> 210 us, 64 entries 70 -> 66.
template <int P, int E>
__device__ __forceinline__ void nearest_of_all(const float2 (&entry)[E], const float* v0, const float* v1, uint32_t* arg) {
    float best[P];
#pragma unroll
    for (int p = 0; p < P; ++p) { best[p] = __builtin_inff(); arg[p] = 0u; }
#pragma unroll 2
    for (int e = 0; e < E; e += 4) {
        const float4_t a = *(const float4_t*)&entry[e], b = *(const float4_t*)&entry[e + 2];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const float least = min3f(min3f(pair_distance(v0[p], v1[p], a.x, a.y), pair_distance(v0[p], v1[p], a.z, a.w),
                                            pair_distance(v0[p], v1[p], b.x, b.y)),
                                      pair_distance(v0[p], v1[p], b.z, b.w), best[p]);
            if (least < best[p]) arg[p] = (uint32_t)e;             // strict: the first four that hold it
            best[p] = least;
        }
    }
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const uint32_t e = arg[p];
        arg[p] = 0u;
#pragma unroll
        for (int q = 3; q >= 0; --q) {
            const float2 c = entry[e + q];
            if (pair_distance(v0[p], v1[p], c.x, c.y) == best[p] && best[p] < __builtin_inff()) arg[p] = e + q;
        }
    }
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_move(uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true); }
__device__ __forceinline__ float wave_sum(float v) {                // quad_perm [1, 0, 3, 2], [2, 3, 0, 1], row_half_mirror, row_mirror
    v += __uint_as_float(dpp_move<0xB1>(__float_as_uint(v)));
    v += __uint_as_float(dpp_move<0x4E>(__float_as_uint(v)));
    v += __uint_as_float(dpp_move<0x141>(__float_as_uint(v)));
    v += __uint_as_float(dpp_move<0x140>(__float_as_uint(v)));
    auto both = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(both[0]) + __uint_as_float(both[1]);
    both = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(both[0]) + __uint_as_float(both[1]);
}
template <int CTRL>
__device__ __forceinline__ void nearest_first(float& best, uint32_t& arg) {    // the lower index of equal ones
    const float od = __uint_as_float(dpp_move<CTRL>(__float_as_uint(best)));
    const uint32_t oe = dpp_move<CTRL>(arg);
    if (od < best || (od == best && oe < arg)) { best = od; arg = oe; }
}
template <int CTRL>
__device__ __forceinline__ void nearer(float& best, int& arg) {      // of two lanes, as one of the exchanges above pairs them
    const float od = __uint_as_float(dpp_move<CTRL>(__float_as_uint(best)));
    const int oe = (int)dpp_move<CTRL>((uint32_t)arg);
    if (od < best) { best = od; arg = oe; }
}

// Nearest entries without comparing every pair with every entry.  A workgroup of 1024 threads takes a 256 x 256 block:
//   1. the plane is cut into 32 x 32 cells (256 entries: 64 x 64) over mean +- 3.25 standard deviations of the codebook's entries
//      (those outside are left out and the box is taken again, twice);
//   2. the entries that can be nearest to a point of a cell are listed: with r the entry nearest to the
//      centre, at distance |r|, and h the distance from the centre to the cell's farthest point, an entry farther than
//      |r| + 2 h from the centre is farther than r from every point of the cell, and so is one whose squared distance exceeds
//      r's at all four corners (the difference is linear over the cell).  The cell is taken 10 % and the limits 1e-5 of the
//      squared reach too large, far beyond the rounding of the binary32 distances (4 2^-24) and of the cell of a point, so the
//      entry that wins by the definition's rounded distances is always listed, and so is every entry that ties with it, but for
//      entries equal to one of a lower index: they never win, and copies of one entry would fill the lists;
//   3. a pair is compared with its cell's entries in index order (strict comparison: the lowest index wins a tie); unused
//      places of a list repeat its first entry, which never wins again;
//   4. pairs outside the cells, or in a cell with more than 16 entries (256: 8), are queued and compared with every entry: a few by
//      sixteen lanes for four of them, more by a thread each.  Those that find the queue full (a quarter of the block, with 256
//      entries an eighth: two workgroups share the LDS of a compute unit) are marked, and collected where the lists were, at once
//      where they fit (4096 x 4096, 256 entries, half of them zero, where some blocks queue a little more: a quarter of the block
//      after another 105 us, now 98);
//   5. blocks for which the cells do not pay (weights far wider than the codebook, crowded entries) compare every pair
//      with every entry: when a fifth (6 bits) or a third (8 bits) of 128 sampled pairs is outside the cells, before the lists
//      are made, or when a quarter of the first unit of every thread was queued, from there on (from the start, if half was).
//      Four entries at a time, the smallest of them against the best, which one it was found out at the end: 6 instructions
//      per pair and entry instead of 8.
// Bound: the chains of step 2 in the wavefronts of the middle, and the LDS look-ups of the 2 to 8 listed entries per pair (a wavefront
// runs to its longest list, in fours).
// Step 2 goes from 8 x 8 over 16 x 16 to 32 x 32 cells, sixteen lanes, four and one for a cell, a bit per entry: a cell tests only the
// entries of the cell around it, whose lists hold them all by the same argument.  With 256 entries a thread goes on to the quarters of
// its cell (32 entries at most): lists of sixteen places in 32 x 32 cells ran to all four fours, those of eight in 64 x 64 run to two, and
// 366 pairs of a block are queued instead of 543.  With 64 entries the quarters cost what they save (4096 x 4096 50 -> 46 us, 1024 x 1024
// 20 -> 25, 14336 x 4096 even).  Cycles of a workgroup alone on its compute unit, 256 entries, before -> now: lists 64000 -> 54000, a unit of
// eight pairs per thread 20000 -> 12000, the queue 21000 -> 17000.  A few queued pairs (step 4) are taken four at a time by sixteen lanes.
// Measured (bf16, near-normal weights, one in a thousand ten times as wide, one matrix repeated, us; every pair against every entry,
// with 32 x 32 cells that each looked through the entries near 8 x 8 of them, here): 4096 x 4096, 64 entries 77, 53, 50, 256 entries
// 279, 81, 64; 14336 x 4096, 64 entries 128 -> 125, 256 entries 887, 218, 171; 1024 x 1024, 64 entries 22 -> 20, 256 entries 83, 42, 39.
// Where there is little for the cells to find, 4096 x 4096 with 64 and 256 entries: weights 50 times as wide as the codebook 67 and 215,
// all entries equal 65 and 207, on nine places 30 and 44 (copies on the lists: 65 and 272), half of them zero 65 and 98 (75 and 184),
// half of them different ones within a thousandth of a deviation 65 and 110.  Registers: 64, for two workgroups on a compute unit (74:
// 14336 x 4096, 64 entries 126 -> 172).
template <int KBITS>
__global__ void __launch_bounds__(1024, 8) vq_assign_kernel(const void* __restrict__ w, int wdt, int N, int K,
                                                         const uint16_t* __restrict__ codebooks,
                                                         uint32_t* __restrict__ indices, int parts_log2) {
    constexpr int E = 1 << KBITS, kQueue = KBITS == 6 ? 8192 : 4096;
    constexpr bool kFine = KBITS == 8;                             // 64 x 64 cells of up to eight entries, else 32 x 32 of sixteen
    constexpr int G = kFine ? 64 : 32, kSlots = kFine ? 8 : 16;
    constexpr int kFewQueued = KBITS == 6 ? 256 : 768;             // a thread per pair: 2 and 8 us whatever their number, four at a time 2 us per 256
    __shared__ __attribute__((aligned(16))) float2 entry[E];
    __shared__ __attribute__((aligned(16))) uint8_t list[G * G][kSlots];
    __shared__ uint8_t listed[kFine ? 1 : G * G];
    __shared__ __attribute__((aligned(16))) uint8_t found[32768];
    __shared__ uint16_t queue[kQueue];
    __shared__ uint32_t over[1024];                                // pairs that the queue had no place for: a bit each, a byte per unit
    __shared__ int queued[2], outside;                             // by the first units, by the others
    __shared__ int crowds;                                         // (fine) cells of 16 x 16 that list a crowd, and which
    __shared__ uint8_t crowded[kFine ? 256 : 1];
    __shared__ float box[5];                                       // origin, cells per unit, h
    __shared__ __attribute__((aligned(8))) uint32_t distinct[E / 32];   // a bit per entry: none of a lower index is equal
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int block = blockIdx.x >> parts_log2, part = blockIdx.x & ((1 << parts_log2) - 1);
    const int bj = block % (K / kBlock), bi = block / (K / kBlock);
    const uint16_t* cb = codebooks + (size_t)block * E * 2;
    // the pairs of a workgroup's rows in units of eight: thread after thread, row after row; unit u is pairs 8 u .. 8 u + 7
    const int units = 4096 >> parts_log2;
    const size_t first_row = (size_t)bi * kBlock + (size_t)part * (kBlock >> parts_log2);
    const size_t base = first_row * K + (size_t)bj * kBlock;
    auto load_unit = [&](int u, float (&v0)[8], float (&v1)[8]) { load_pairs8(w, wdt, base + (size_t)(u >> 4) * K + 16 * (u & 15), v0, v1); };
    auto load_pair = [&](int id, float& vx, float& vy) {
        const size_t e = base + (size_t)(id >> 7) * K + 2 * (id & 127);
        if (wdt == DT_F32) {
            const float2 v = *(const float2*)((const float*)w + e);
            vx = v.x; vy = v.y;
        } else {
            const uint32_t v = *(const uint32_t*)((const uint16_t*)w + e);
            const uint16_t lo = (uint16_t)(v & 0xFFFFu), hi = (uint16_t)(v >> 16);
            vx = wdt == DT_F16 ? f16_bits_to_f32(lo) : bf16_bits_to_f32(lo);
            vy = wdt == DT_F16 ? f16_bits_to_f32(hi) : bf16_bits_to_f32(hi);
        }
    };
    float px = 0.f, py = 0.f;
    const bool sampled = tid < 128;                                // 128 pairs spread over the rows
    if (sampled) load_pair((tid * (units >> 4) & ~127) + (tid * 37 & 127), px, py);
    if (tid < E) entry[tid] = float2{f16_bits_to_f32(cb[2 * tid]), f16_bits_to_f32(cb[2 * tid + 1])};
    over[tid] = 0u;
    if (tid == 0) { queued[0] = 0; queued[1] = 0; outside = 0; crowds = 0; }
    // Beside the box: the lowest entry of each of 1024 hashes.  An entry equal to it never wins and is on no list.  (One that is equal to
    // another of its hash stays: it costs a place.)
    uint32_t* const lowest = (uint32_t*)found;
    const bool looks = tid >= 512 && tid < 512 + E;
    const uint32_t hash = looks ? (((const uint32_t*)cb)[tid - 512] * 0x9E3779B1u) >> 22 : 0u;
    lowest[tid] = E;
    __syncthreads();
    if (looks) atomicMin(&lowest[hash], (uint32_t)tid - 512u);
    if (wave == 0) {                                               // mean and deviation, twice more without the entries outside
        float m0 = entry[0].x, m1 = entry[0].y, r0 = __builtin_inff(), r1 = __builtin_inff();
#pragma unroll 1
        for (int pass = 0; pass < 3; ++pass) {
            float s[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int e = lane; e < E; e += 64) {
                const float2 c = entry[e];
                const float dx = c.x - m0, dy = c.y - m1;
                if (fabsf(dx) <= r0 && fabsf(dy) <= r1) { s[0] += dx; s[1] += dy; s[2] += dx * dx; s[3] += dy * dy; s[4] += 1.f; }
            }
#pragma unroll
            for (int i = 0; i < 5; ++i) s[i] = wave_sum(s[i]);
            if (s[4] < 1.f) break;
            const float a0 = s[0] / s[4], a1 = s[1] / s[4];
            m0 += a0; m1 += a1;
            // no cell narrower than 6e-6 of its place (the resolution of binary32 there)
            r0 = fmaxf(fmaxf(3.25f * sqrtf(fmaxf(s[2] / s[4] - a0 * a0, 0.f)), (kFine ? 2e-4f : 1e-4f) * fabsf(m0)), 1e-6f);
            r1 = fmaxf(fmaxf(3.25f * sqrtf(fmaxf(s[3] / s[4] - a1 * a1, 0.f)), (kFine ? 2e-4f : 1e-4f) * fabsf(m1)), 1e-6f);
        }
        if (lane == 0) {
            box[0] = m0 - r0; box[1] = m1 - r1; box[2] = 16.f / r0; box[3] = 16.f / r1;
            box[4] = 0.55f * (1.f / 16.f) * sqrtf(r0 * r0 + r1 * r1);
        }
    }
    __syncthreads();
    auto uniform = [](float v) { return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(v))); };   // a scalar register
    const float x0 = uniform(box[0]), y0 = uniform(box[1]), sx = uniform(box[2]), sy = uniform(box[3]);
    auto cell_of = [&](float vx, float vy) {                       // -1: outside
        const float fx = (vx - x0) * (sx * (G / 32)), fy = (vy - y0) * (sy * (G / 32));
        const bool in = fx >= 0.f && fx < (float)G && fy >= 0.f && fy < (float)G;
        return in ? (int)fy * G + (int)fx : -1;
    };
    auto store_found = [&](int u, const uint32_t (&arg)[8]) {
        *(uint2_t*)(found + 8 * u) = uint2_t{arg[0] | (arg[1] << 8) | (arg[2] << 16) | (arg[3] << 24),
                                           arg[4] | (arg[5] << 8) | (arg[6] << 16) | (arg[7] << 24)};
    };
    {
        const int n = __builtin_popcountll(__builtin_amdgcn_ballot_w64(sampled && cell_of(px, py) < 0));
        if (lane == 0 && n) atomicAdd(&outside, n);
    }
    if (looks) {
        const uint32_t at = (uint32_t)tid - 512u, e = lowest[hash];
        const float2 a = entry[at], b = entry[e];
        const unsigned long long m = __builtin_amdgcn_ballot_w64(!(e < at && a.x == b.x && a.y == b.y));
        if (lane == 0) *(unsigned long long*)&distinct[at >> 5] = m;
    }
    __syncthreads();
    int from = outside > (KBITS == 6 ? 24 : 40) ? 0 : 4096;         // units from here on: every pair with every entry
    int ahead = 0;                                                 // queued by the first units
    if (from) {
        // The lists, from the coarse to the fine: an entry that can be nearest to a point of a cell can be nearest to that point of the
        // cell around it.  A bit per entry; the bits of the two coarse grids lie where the results will.
        uint16_t* const coarse = (uint16_t*)found;                  // [8 x 8][E / 16]
        uint16_t* const middle = coarse + 64 * (E / 16);            // [16 x 16][E / 16], and as much again for the crowds
        // Fine: a cell of 16 x 16 that lists more than kCrowd entries would hold up the one lane per cell of the step after it, and is
        // listed by whole wavefronts behind it.  256 entries, a half of them within a thousandth of a deviation of one place: 4096 x 4096
        // 118 -> 110 us, 1024 x 1024 62 -> 54, a quarter of them 50 -> 46; near-normal ones even.  With 48 near-normal codebooks have such
        // cells (37.6 -> 38.9), with 110 the second stays at 60.  64 entries hold up less: nothing was gained.
        constexpr int kCrowd = 64;
        constexpr int kWords = E / 32;
        // at most this far from the centre of a cell of 32 / g x 32 / g: the limit, and what every unit of distance from r adds
        auto limits = [&](float g, float least, float& at_most, float& hx, float& hy) {
            const float reach = (sqrtf(least) + 2.f * g * box[4]) * 1.0001f;
            at_most = least + 1e-5f * (reach * reach);
            hx = 1.1f * g / sx; hy = 1.1f * g / sy;                 // twice 0.55 of a cell's sides
        };
        // of the entries base + (bits of m): the nearest
        auto nearest_of = [&](uint32_t m, int base, float cx, float cy, float& best, int& arg) {
#pragma unroll 1
            for (; m; m &= m - 1u) {                                 // two at a time
                const int e0 = base + __builtin_ctz(m);
                m &= m - 1u;
                const int e1 = m ? base + __builtin_ctz(m) : e0;
                const float2 o0 = entry[e0], o1 = entry[e1];
                const float d0 = pair_distance(cx, cy, o0.x, o0.y), d1 = pair_distance(cx, cy, o1.x, o1.y);
                if (d0 < best) { best = d0; arg = e0; }
                if (d1 < best) { best = d1; arg = e1; }
            }
        };
        auto within = [&](uint32_t m, int base, float cx, float cy, float2 r, float at_most, float hx, float hy) {
            uint32_t bits = 0u;
#pragma unroll 1
            for (; m; m &= m - 1u) {
                const int b0 = __builtin_ctz(m);
                m &= m - 1u;
                const int b1 = m ? __builtin_ctz(m) : b0;
                const float2 o0 = entry[base + b0], o1 = entry[base + b1];
                const float d0 = pair_distance(cx, cy, o0.x, o0.y), d1 = pair_distance(cx, cy, o1.x, o1.y);
                bits |= d0 <= fmaf(fabsf(r.x - o0.x), hx, fmaf(fabsf(r.y - o0.y), hy, at_most)) ? 1u << b0 : 0u;
                bits |= d1 <= fmaf(fabsf(r.x - o1.x), hx, fmaf(fabsf(r.y - o1.y), hy, at_most)) ? 1u << b1 : 0u;
            }
            return bits;
        };
        {   // 8 x 8 cells, sixteen lanes each
            const int part = tid & 15, at = tid >> 4;
            const float cx = x0 + (4.f * (float)(at & 7) + 2.f) / sx, cy = y0 + (4.f * (float)(at >> 3) + 2.f) / sy;
            float best = __builtin_inff(), at_most, hx, hy;
            int arg = part;
#pragma unroll 4
            for (int k = 0; k < E / 16; ++k) {
                const float2 o = entry[16 * k + part];
                const float d = pair_distance(cx, cy, o.x, o.y);
                if (d < best) { best = d; arg = 16 * k + part; }
            }
            nearer<0xB1>(best, arg); nearer<0x4E>(best, arg); nearer<0x141>(best, arg); nearer<0x140>(best, arg);
            limits(4.f, best, at_most, hx, hy);
            const float2 r = entry[arg];
            uint32_t mine = 0u;
#pragma unroll 4
            for (int k = 0; k < E / 16; ++k) {
                const float2 o = entry[16 * k + part];
                const float d = pair_distance(cx, cy, o.x, o.y);
                const unsigned long long m = __builtin_amdgcn_ballot_w64(d <= fmaf(fabsf(r.x - o.x), hx, fmaf(fabsf(r.y - o.y), hy, at_most)));
                if (part == k) mine = (uint32_t)(m >> (lane & 48)) & 0xFFFFu;
            }
            if (part < E / 16) coarse[at * (E / 16) + part] = (uint16_t)(mine & ((const uint16_t*)distinct)[part]);
        }
        __syncthreads();
        {   // 16 x 16 cells, four lanes each
            const int part = tid & 3, at = tid >> 2, gx = at & 15, gy = at >> 4;
            const float cx = x0 + (2.f * (float)gx + 1.f) / sx, cy = y0 + (2.f * (float)gy + 1.f) / sy;
            const uint16_t* const from_bits = coarse + (8 * (gy >> 1) + (gx >> 1)) * (E / 16) + part * (E / 64);
            uint16_t* const to_bits = middle + at * (E / 16) + part * (E / 64);
            constexpr int kOwn = E / 128 > 0 ? E / 128 : 1;          // words of a lane (64 entries: half a word)
            uint32_t own[kOwn];
#pragma unroll
            for (int q = 0; q < kOwn; ++q) own[q] = E >= 128 ? ((const uint32_t*)from_bits)[q] : from_bits[0];
            float best = __builtin_inff(), at_most, hx, hy;
            int arg = 0;
#pragma unroll
            for (int q = 0; q < kOwn; ++q) nearest_of(own[q], part * (E / 4) + 32 * q, cx, cy, best, arg);
            nearer<0xB1>(best, arg); nearer<0x4E>(best, arg);
            limits(2.f, best, at_most, hx, hy);
            const float2 r = entry[arg];
#pragma unroll
            for (int q = 0; q < kOwn; ++q) own[q] = within(own[q], part * (E / 4) + 32 * q, cx, cy, r, at_most, hx, hy);
            if constexpr (kFine) {
                int n = 0;
#pragma unroll
                for (int q = 0; q < kOwn; ++q) n += __builtin_popcount(own[q]);
                n += (int)dpp_move<0xB1>((uint32_t)n);
                n += (int)dpp_move<0x4E>((uint32_t)n);
                if (n > kCrowd) {
                    if (part == 0) crowded[atomicAdd(&crowds, 1)] = (uint8_t)at;
#pragma unroll
                    for (int q = 0; q < kOwn; ++q) { ((uint32_t*)(to_bits + 256 * (E / 16)))[q] = own[q]; own[q] = 0u; }
                }
            }
#pragma unroll
            for (int q = 0; q < kOwn; ++q) {
                if constexpr (E >= 128) ((uint32_t*)to_bits)[q] = own[q];
                else to_bits[0] = (uint16_t)own[q];
            }
        }
        __syncthreads();
        {   // 32 x 32 cells, one per thread, 8 x 8 per wavefront; the four wavefronts in the middle, where the entries are, on four SIMDs
            const int wy = wave >> 2, wx = (wave + (wy == 1 ? 1 : wy == 2 ? 3 : 0)) & 3;
            const int gx = 8 * wx + (lane & 7), gy = 8 * wy + (lane >> 3);
            const float cx = x0 + ((float)gx + 0.5f) / sx, cy = y0 + ((float)gy + 0.5f) / sy;
            const uint32_t* const from_bits = (const uint32_t*)(middle + (16 * (gy >> 1) + (gx >> 1)) * (E / 16));
            float best = __builtin_inff(), at_most, hx, hy;
            int arg = 0;
#pragma unroll
            for (int q = 0; q < kWords; ++q) nearest_of(from_bits[q], 32 * q, cx, cy, best, arg);
            limits(1.f, best, at_most, hx, hy);
            const float2 r = entry[arg];
            // The entries in order; a place is written until an entry keeps it.  Sixteen places of the cell itself, or, on the way to
            // finer cells, 32 in those of its four quarters.
            constexpr int kPlaces = kFine ? 32 : kSlots;
            uint8_t* const places = kFine ? list[2 * gy * G + 2 * gx] : list[gy * G + gx];
            auto place = [&](int i) { return places + (kFine && i >= 16 ? G * kSlots + i - 16 : i); };
            int n = 0;
#pragma unroll
            for (int q = 0; q < kWords; ++q)
#pragma unroll 1
                for (uint32_t m = from_bits[q]; m; m &= m - 1u) {
                    const int e0 = 32 * q + __builtin_ctz(m);
                    m &= m - 1u;
                    const bool two = m != 0u;
                    const int e1 = two ? 32 * q + __builtin_ctz(m) : e0;
                    const float2 o0 = entry[e0], o1 = entry[e1];
                    const float d0 = pair_distance(cx, cy, o0.x, o0.y), d1 = pair_distance(cx, cy, o1.x, o1.y);
                    if (n < kPlaces) *place(n) = (uint8_t)e0;
                    n += d0 <= fmaf(fabsf(r.x - o0.x), hx, fmaf(fabsf(r.y - o0.y), hy, at_most)) ? 1 : 0;
                    if (two && n < kPlaces) *place(n) = (uint8_t)e1;
                    n += two && d1 <= fmaf(fabsf(r.x - o1.x), hx, fmaf(fabsf(r.y - o1.y), hy, at_most)) ? 1 : 0;
                }
            const bool fits = n > 0 && n <= kPlaces;
            uint32_t word[kPlaces / 4];                              // unused places repeat the first entry
            word[0] = *(const uint32_t*)places;
            const uint32_t four = (word[0] & 255u) * 0x01010101u;
#pragma unroll
            for (int q = 0; q < kPlaces / 4; ++q) {
                const int used = min(max(n - 4 * q, 0), 4);
                const uint32_t mask = used == 4 ? 0xFFFFFFFFu : (1u << (8 * used)) - 1u;
                word[q] = (*(const uint32_t*)place(4 * q) & mask) | (four & ~mask);
            }
            if constexpr (!kFine) {
                listed[gy * G + gx] = (uint8_t)(fits ? n : 255);
                *(uint4_t*)places = uint4_t{word[0], word[1], word[2], word[3]};
            } else {
                // The quarters: twice over the list, four distances each time; a bit per place.
                const float qx[2] = {x0 + ((float)gx + 0.25f) / sx, x0 + ((float)gx + 0.75f) / sx};
                const float qy[2] = {y0 + ((float)gy + 0.25f) / sy, y0 + ((float)gy + 0.75f) / sy};
                const int entries = fits ? n : 0;
                float least[4], ax, ay;
                int near[4];
                uint32_t bits[4];
                auto each = [&](auto f) {
#pragma unroll
                    for (int q = 0; q < 8; ++q) {
                        if (__builtin_amdgcn_ballot_w64(entries > 4 * q) == 0) break;
#pragma unroll
                        for (int b = 0; b < 4; ++b) {
                            const int e = (int)((word[q] >> (8 * b)) & 255u);
                            const float2 o = entry[e];
                            const float t0 = __fsub_rn(qx[0], o.x), t1 = __fsub_rn(qx[1], o.x), u0 = __fsub_rn(qy[0], o.y), u1 = __fsub_rn(qy[1], o.y);
                            const float a0 = __fmul_rn(t0, t0), a1 = __fmul_rn(t1, t1), b0 = __fmul_rn(u0, u0), b1 = __fmul_rn(u1, u1);
                            const float d[4] = {__fadd_rn(a0, b0), __fadd_rn(a1, b0), __fadd_rn(a0, b1), __fadd_rn(a1, b1)};
#pragma unroll
                            for (int c = 0; c < 4; ++c) f(c, o, d[c], e, 4 * q + b);
                        }
                    }
                };
#pragma unroll
                for (int c = 0; c < 4; ++c) { least[c] = __builtin_inff(); near[c] = 0; bits[c] = 0u; }
                each([&](int c, const float2&, float d, int e, int) { if (d < least[c]) { least[c] = d; near[c] = e; } });
                float2 w[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    float most;
                    limits(0.5f, least[c], most, ax, ay);
                    least[c] = most;
                    w[c] = entry[near[c]];
                }
                each([&](int c, const float2& o, float d, int, int i) {
                    bits[c] |= d <= fmaf(fabsf(w[c].x - o.x), ax, fmaf(fabsf(w[c].y - o.y), ay, least[c])) ? 1u << i : 0u;
                });
                uint2_t to[4];
                const uint32_t real = entries == 32 ? 0xFFFFFFFFu : (1u << entries) - 1u;
#pragma unroll
                for (int c = 0; c < 4; ++c) {                        // a list that does not fit starts with 1 and 0
                    uint32_t m = bits[c] & real;
                    const int kept = __builtin_popcount(m);
                    uint32_t out[2] = {0u, 0u}, first = 0u;
                    if (kept > kSlots) m = 0u;
#pragma unroll
                    for (int j = 0; j < kSlots; ++j) {
                        if (__builtin_amdgcn_ballot_w64(m != 0u) == 0) {
                            if (j < 4) out[0] |= first * (0x01010101u << (8 * (j & 3)));
                            out[1] |= j < 4 ? first * 0x01010101u : first * (0x01010101u << (8 * (j & 3)));
                            break;
                        }
                        const uint32_t e = m ? *place(__builtin_ctz(m)) : first;
                        if (j == 0) first = e;
                        out[j >> 2] |= e << (8 * (j & 3));
                        m &= m - 1u;
                    }
                    to[c] = kept > kSlots || kept == 0 ? uint2_t{1u, 0u} : uint2_t{out[0], out[1]};
                }
                *(uint4_t*)places = uint4_t{to[0].x, to[0].y, to[1].x, to[1].y};
                *(uint4_t*)(places + G * kSlots) = uint4_t{to[2].x, to[2].y, to[3].x, to[3].y};
            }
        }
        __syncthreads();
        if constexpr (kFine)
            if (crowds) {
                // The sixteen cells within each: a wavefront for one after another, a lane for every 64th entry
                const int all = 16 * __builtin_amdgcn_readfirstlane(crowds);
#pragma unroll 1
                for (int j = wave; j < all; j += 16) {
                    const int at = __builtin_amdgcn_readfirstlane(crowded[j >> 4]);
                    const int gx = 4 * (at & 15) + (j & 3), gy = 4 * (at >> 4) + ((j >> 2) & 3);
                    const float cx = x0 + 0.5f * ((float)gx + 0.5f) / sx, cy = y0 + 0.5f * ((float)gy + 0.5f) / sy;
                    const uint32_t* const bits = (const uint32_t*)(middle + (256 + at) * (E / 16)) + (lane >> 5);
                    float d[E / 64], best = __builtin_inff(), at_most, hx, hy;
                    float2 o[E / 64];
                    int arg = 0;
#pragma unroll
                    for (int q = 0; q < E / 64; ++q) {
                        o[q] = entry[64 * q + lane];
                        d[q] = (bits[2 * q] >> (lane & 31)) & 1u ? pair_distance(cx, cy, o[q].x, o[q].y) : __builtin_nanf("");   // (never kept)
                        if (d[q] < best) { best = d[q]; arg = 64 * q + lane; }
                    }
                    nearer<0xB1>(best, arg); nearer<0x4E>(best, arg); nearer<0x141>(best, arg); nearer<0x140>(best, arg);
                    auto join = [&](auto both, auto which) {
                        const float d0 = __uint_as_float(both[0]), d1 = __uint_as_float(both[1]);
                        best = d1 < d0 ? d1 : d0; arg = (int)(d1 < d0 ? which[1] : which[0]);
                    };
                    uint32_t b = __float_as_uint(best), a = (uint32_t)arg;
                    join(__builtin_amdgcn_permlane16_swap(b, b, false, false), __builtin_amdgcn_permlane16_swap(a, a, false, false));
                    b = __float_as_uint(best); a = (uint32_t)arg;
                    join(__builtin_amdgcn_permlane32_swap(b, b, false, false), __builtin_amdgcn_permlane32_swap(a, a, false, false));
                    limits(0.5f, best, at_most, hx, hy);
                    const float2 r = entry[arg];
                    unsigned long long keeps[E / 64];
                    int n = 0, first = 0, before = 0;
#pragma unroll
                    for (int q = E / 64 - 1; q >= 0; --q) {
                        keeps[q] = __builtin_amdgcn_ballot_w64(d[q] <= fmaf(fabsf(r.x - o[q].x), hx, fmaf(fabsf(r.y - o[q].y), hy, at_most)));
                        n += __builtin_popcountll(keeps[q]);
                        if (keeps[q]) first = 64 * q + __builtin_ctzll(keeps[q]);
                    }
                    const bool fits = n > 0 && n <= kSlots;
                    uint8_t* const places = list[gy * G + gx];
                    if (lane < kSlots) places[lane] = (uint8_t)(fits ? first : lane == 0);   // a list that does not fit starts with 1 and 0
#pragma unroll
                    for (int q = 0; q < E / 64; ++q) {
                        const bool mine = fits && ((keeps[q] >> lane) & 1u);
                        if (mine) places[before + __builtin_popcountll(keeps[q] & ((1ull << lane) - 1u))] = (uint8_t)(64 * q + lane);
                        before += __builtin_popcountll(keeps[q]);
                    }
                }
                __syncthreads();
            }

#pragma unroll 1
        for (int u = tid; u < units; u += 1024) {
            if (u >= 1024 && u < 2048) {                           // the first units are through
                __syncthreads();
                ahead = queued[0];
                if (ahead > 2048) { from = ahead > 4096 ? 0 : 1024; break; }   // (of 8192)
            }
            float v0[8], v1[8];
            uint32_t arg[8];
            load_unit(u, v0, v1);
#pragma unroll
            for (int h = 0; h < 8; h += 4) {
                std::conditional_t<kFine, uint2_t, uint4_t> l[4];
                float best[4];
                int longest = 0;                                   // fine: are there entries in places 4 .. 7?
                bool again[4];
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    const int at = cell_of(v0[h + p], v1[h + p]), cell = max(at, 0);
                    if constexpr (kFine) {
                        l[p] = *(const uint2_t*)list[cell];
                        again[p] = at < 0 || (l[p].x & 255u) > ((l[p].x >> 8) & 255u);
                        longest |= again[p] || l[p].y == (l[p].x & 255u) * 0x01010101u ? 0 : 8;
                    } else {
                        const int cnt = listed[cell];
                        l[p] = *(const uint4_t*)list[cell];
                        again[p] = at < 0 || cnt == 255;
                        longest = max(longest, again[p] ? 0 : cnt);
                    }
                    best[p] = __builtin_inff();
                    arg[h + p] = 0u;
                }
#pragma unroll
                for (int q = 0; q < kSlots / 4; ++q) {             // four places at a time, up to the longest list of the wavefront
                    if ((!kFine || q > 0) && __builtin_amdgcn_ballot_w64(longest > 4 * q) == 0) break;
#pragma unroll
                    for (int b = 0; b < 4; ++b)
#pragma unroll
                        for (int p = 0; p < 4; ++p) {
                            const uint32_t e = (l[p][q] >> (8 * b)) & 255u;
                            const float2 ce = entry[e];
                            const float d = pair_distance(v0[h + p], v1[h + p], ce.x, ce.y);
                            if (d < best[p]) { best[p] = d; arg[h + p] = e; }
                        }
                }
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    if (again[p]) {
                        const int at = ahead + atomicAdd(&queued[u >= 1024], 1);
                        if (at < kQueue) queue[at] = (uint16_t)(8 * u + h + p);
                        else ((uint8_t*)over)[u] |= (uint8_t)(1u << (h + p));
                    }
                }
            }
            store_found(u, arg);
        }
        __syncthreads();
    }
    const int all = from ? __builtin_amdgcn_readfirstlane(queued[0] + queued[1]) : 0, todo = min(all, kQueue);
    if (from < units) {
#pragma unroll 1
        for (int u = from + tid; u < units; u += 1024) {
            float v0[8], v1[8];
            uint32_t arg[8];
            load_unit(u, v0, v1);
            nearest_of_all<8>(entry, v0, v1, arg);
            store_found(u, arg);
        }
    }
    auto each_by_itself = [&](const uint16_t* pairs, int n) {
        int i = tid;
        asm volatile("" : "+v"(i));                                // (nothing of it kept in registers over what comes before)
#pragma unroll 1
        for (; i < n; i += 1024) {
            const int id = pairs[i];
            float vx, vy;
            uint32_t arg;
            load_pair(id, vx, vy);
            nearest_of_all<1>(entry, &vx, &vy, &arg);
            found[id] = (uint8_t)arg;
        }
    };
    if (todo) {
        if (todo > kFewQueued) {                                   // a thread per queued pair
            each_by_itself(queue, todo);
        } else {
#pragma unroll 1
            for (int i0 = 0; i0 < todo; i0 += 256) {               // sixteen lanes per four queued pairs
                const int mine = i0 + 4 * (tid >> 4);
                if (mine >= todo) break;
                float vx[4], vy[4], bd[4];
                uint32_t be[4];
                int id[4];
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    id[p] = queue[min(mine + p, todo - 1)];
                    load_pair(id[p], vx[p], vy[p]);
                    bd[p] = __builtin_inff();
                    be[p] = 0xFFFFFFFFu;
                }
#pragma unroll 1
                for (int k = 0; k < E / 64; ++k) {                 // four entries at a time, as in nearest_of_all
                    float2 ce[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) ce[q] = entry[(tid & 15) + 16 * (4 * k + q)];
#pragma unroll
                    for (int p = 0; p < 4; ++p) {
                        const float least = min3f(min3f(pair_distance(vx[p], vy[p], ce[0].x, ce[0].y), pair_distance(vx[p], vy[p], ce[1].x, ce[1].y),
                                                        pair_distance(vx[p], vy[p], ce[2].x, ce[2].y)),
                                                  pair_distance(vx[p], vy[p], ce[3].x, ce[3].y), bd[p]);
                        if (least < bd[p]) be[p] = (uint32_t)k;
                        bd[p] = least;
                    }
                }
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    const int first = (tid & 15) + 64 * (bd[p] < __builtin_inff() ? (int)be[p] : 0);
                    be[p] = 0xFFFFFFFFu;
#pragma unroll
                    for (int q = 3; q >= 0; --q) {
                        const float2 c = entry[first + 16 * q];
                        if (pair_distance(vx[p], vy[p], c.x, c.y) == bd[p] && bd[p] < __builtin_inff()) be[p] = (uint32_t)(first + 16 * q);
                    }
                    nearest_first<0xB1>(bd[p], be[p]); nearest_first<0x4E>(bd[p], be[p]); nearest_first<0x141>(bd[p], be[p]); nearest_first<0x140>(bd[p], be[p]);
                    // (every distance infinite or NaN: entry 0; past the end the last pair again)
                    if ((tid & 15) == 0) found[id[p]] = (uint8_t)(be[p] == 0xFFFFFFFFu ? 0u : be[p]);
                }
            }
        }
        if (all > kQueue) {                                        // those that it had no place for: at once, or, where the room of the
            uint16_t* const more = (uint16_t*)list[0];             // lists does not hold them, a quarter of the block after another
            constexpr int kRoom = G * G * kSlots / 2;
            static_assert(kRoom >= 8192, "a quarter's pairs");
            const int step = all - kQueue <= kRoom ? 1024 : 256;
#pragma unroll 1
            for (int w0 = 0; w0 < units / 4; w0 += step) {
                __syncthreads();
                if (tid == 0) outside = 0;
                __syncthreads();
                int word = w0 + tid;
                asm volatile("" : "+v"(word));
                uint32_t m = tid < step ? over[word] : 0u;
                int at = m ? atomicAdd(&outside, __builtin_popcount(m)) : 0;
#pragma unroll 1
                for (; m; m &= m - 1u) more[at++] = (uint16_t)(32 * word + __builtin_ctz(m));
                __syncthreads();
                each_by_itself(more, outside);
            }
        }
    }
    __syncthreads();
    constexpr int wpr = KBITS == 6 ? 3 : 4;                        // output words per 16 pairs
    for (int u = tid; u < units / 2; u += 1024) {
        uint32_t* out = indices + (first_row + (u >> 3)) * (K / 2 * KBITS / 32) + (size_t)bj * (kBlock / 2 * KBITS / 32) + wpr * (u & 7);
        const uint4_t f = *(const uint4_t*)(found + 16 * u);
        if constexpr (KBITS == 8) {
            *(uint4_t*)out = f;
        } else {
            const uint32_t fw[4] = {f.x, f.y, f.z, f.w};
            uint32_t packed[4];                                    // four indices each: 24 bits
#pragma unroll
            for (int q = 0; q < 4; ++q)
                packed[q] = (fw[q] & 63u) | ((fw[q] >> 2) & 0xFC0u) | ((fw[q] >> 4) & 0x3F000u) | ((fw[q] >> 6) & 0xFC0000u);
            out[0] = packed[0] | (packed[1] << 24);
            out[1] = (packed[1] >> 8) | (packed[2] << 16);
            out[2] = (packed[2] >> 16) | (packed[3] << 8);
        }
    }
}

hipError_t launch_sq_encode(const void* w, int wdt, int N, int K, uint32_t* codes, uint16_t* scales,
                            uint16_t* zeros, hipStream_t s) {
    const long long units = (long long)N * (K / kGroup);
    constexpr int U = RWKVQ_SQ_ENCODE_PASSES;
    const dim3 grid((unsigned)((units + 32 * U - 1) / (32 * U)));
    if (wdt == DT_F32) hipLaunchKernelGGL((sq_encode_kernel<U, DT_F32>), grid, dim3(256), 0, s, w, N, K, codes, scales, zeros);
    else if (wdt == DT_F16) hipLaunchKernelGGL((sq_encode_kernel<U, DT_F16>), grid, dim3(256), 0, s, w, N, K, codes, scales, zeros);
    else hipLaunchKernelGGL((sq_encode_kernel<U, DT_BF16>), grid, dim3(256), 0, s, w, N, K, codes, scales, zeros);
    return hipGetLastError();
}

hipError_t launch_vq_assign(const void* w, int wdt, int N, int K, int kbits, const uint16_t* codebooks,
                            uint32_t* indices, hipStream_t s) {
    const unsigned blocks = (unsigned)((N / kBlock) * (K / kBlock));
    // a chip left idle by few blocks takes each in two or four parts, each with lists of its own (1024 x 1024, 64 entries:
    // whole blocks 42 us, quarters 22; 256 entries 83 and 50)
    int parts_log2 = 0;
    while (parts_log2 < 2 && (blocks << (parts_log2 + 1)) <= 256u) ++parts_log2;
    const dim3 grid(blocks << parts_log2);
    if (kbits == 6) hipLaunchKernelGGL(vq_assign_kernel<6>, grid, dim3(1024), 0, s, w, wdt, N, K, codebooks, indices, parts_log2);
    else hipLaunchKernelGGL(vq_assign_kernel<8>, grid, dim3(1024), 0, s, w, wdt, N, K, codebooks, indices, parts_log2);
    return hipGetLastError();
}

}  // namespace rwkvq

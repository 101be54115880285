// Streaming dequant-GEMV kernels for small batches (M <= 16), native layout, grouped launch.
//
// Computes y = x * Deq(W)^T (the W. products of App. A.1) for several matrices in one launch,
// each SQ or VQ as its flag says (Sec. 3.1, Eq. "optimization goal").  The work is bound by
// reading the packed weights once from HBM, so everything else is arranged around keeping
// 16-byte coalesced loads in flight while spending as few issue slots per weight as possible.
//
//   * decode_kernel<MT>: one wavefront owns one 16-row tile of one matrix and streams its
//     256-column tiles in order with DEPTH tiles in flight (tile_pipeline); four wavefronts form a
//     workgroup (64 rows).  Up to 256 matrices per launch, longest rows first; a workgroup finds
//     its matrix with ballots over the table in the kernel arguments.
//   * Batch 1 (MT = 1), all formats, on the vector ALU: lane (r, kg) owns row r's columns of column
//     group kg; the sixteen lanes of a row each load one activation pair, and every
//     v_dot2c_f32_f16 names the lane that holds its pair through the DPP control row_newbcast - no
//     LDS for the activations.  SQ codes are multiplied as they are: masked in place, a 3-bit code
//     at mantissa bits b..b+2 of an fp16 half is the subnormal q 2^(b-24); three accumulators (one
//     per bit position) are combined with exact powers of two per group, and
//     y += s (sum q x - z X) with X from four DPP adds.  VQ weights are gathered pair by pair from
//     the block's codebook in a wavefront-private LDS region.
//   * decode_splitk_kernel<S>: batch 1 for launches too small to fill the device (the stages of a
//     block): one workgroup of S wavefronts per row tile, the column tiles dealt round-robin, the
//     partial sums added in LDS in a fixed order.  With MixedDecodeArgs the token-shift mix of
//     Eq. "time mixing r/k/v" is applied while the activations are loaded; with PostMixArgs the
//     outputs also leave as the mixes of the stage that follows (store_post_mix).  The squared ReLU
//     and the gates of App. A.1 can be applied where an output is stored (store_post).
//   * decode_rkv_wkv_kernel: the three projections of time mixing and the wkv step of Eq. "time
//     mixing wkv" in one launch (a workgroup takes a row tile of r, k and v and steps its 16 channels).
//   * Batch 2..32 (MT = 4, 16, 32) on the matrix cores (v_mfma_f32_16x16x32_f16, activations = A
//     operand, weights = B operand): the activation tile of a column tile is fetched once per
//     workgroup into LDS (two buffers, one barrier per tile); SQ codes enter as 8 + q (one shift
//     and one and-or per pair), the group sums X come from one more MFMA against an all-ones
//     operand, y += s (acc - (8 + z) X); VQ pairs are LDS gathers.  A wavefront takes two row
//     tiles of W, and with MT = 32 two groups of 16 batch rows: every unpacked weight operand
//     feeds one MFMA per group.
//   * decode_stage_kernel: batch 2..16 for launches too small to fill the device: the wavefronts of a workgroup split the
//     columns, every one fetches its activations as operands and multiplies one to six row tiles by them.
//   * bf16 activations: multiplied as they are where the weights have an exact form in bf16 for little (SQ codes beyond batch 1, VQ
//     entries as two bf16 in decode_stage_kernel with few row tiles); elsewhere converted to fp16 on load, group by group under an
//     exact power-of-two scale (see "bf16 activations" below).
#include "matrix_core.h"
#include "../../include/rwkvq.h"
#include <algorithm>
#include <cmath>

namespace rwkvq {

// Batch 1: column tiles in flight beyond the one being consumed, and the wavefronts per SIMD the compiler must leave
// registers for.  One tile ahead keeps the grouped kernel at 64 registers, eight wavefronts per SIMD; two tiles ahead
// (79 registers, six per SIMD) put more bytes in flight per compute unit (72 against 48 KB) and were slower once the
// weight loads carried the non-temporal hint: 7B stack 5.79 -> 5.96 TB/s, 14B-class stack 5.65 -> 5.75 TB/s, the token
// step of the 7B blocks (split-K kernels, 65 registers instead of 79-106) 1.008 -> 0.935 ms, same box, alternating.
#ifndef RWKVQ_DECODE_MINBLOCKS
#define RWKVQ_DECODE_MINBLOCKS 8
#endif
#ifndef RWKVQ_DECODE_DEPTH
#define RWKVQ_DECODE_DEPTH 1
#endif
constexpr int kMaxGroupMats = 256;    // matrices per grouped launch (descriptor table in kernarg: a whole
                                      // 32-layer stack is one launch, one ramp-up and one tail)
constexpr int kXStride = 272;         // fp16 per staged activation row: 34 units of 16 bytes, so that the 16 lanes an LDS
                                      // cycle serves (rows m..m+7 of column groups kg, kg+1) fall into 16 distinct units
#ifndef RWKVQ_SPLIT_TARGET
#define RWKVQ_SPLIT_TARGET 2048
#endif
constexpr int kSplitTarget = RWKVQ_SPLIT_TARGET;   // wavefronts a batch-1 launch should have before it stops splitting K
#ifndef RWKVQ_DECODE_RT
#define RWKVQ_DECODE_RT 1
#endif
constexpr int kRT = RWKVQ_DECODE_RT;  // batch 1: 16-row tiles per wavefront
static_assert(kRT == 1, "the batch-1 tile loops hold one row tile per wavefront");
#ifndef RWKVQ_DECODE_BATCH_RT
#define RWKVQ_DECODE_BATCH_RT 2
#endif
#ifndef RWKVQ_BATCH_UB2
#define RWKVQ_BATCH_UB2 0            // batch 2..16: 1 = read the activation fragments of both column halves of a tile up front
#endif
#ifndef RWKVQ_BATCH_DEPTH
#define RWKVQ_BATCH_DEPTH 1          // batch 2..32: tiles in flight beyond the one being consumed
#endif
#ifndef RWKVQ_BATCH16_MINBLOCKS
#define RWKVQ_BATCH16_MINBLOCKS 4    // wavefronts per SIMD the compiler must leave registers for (batch 5..16)
#endif
#ifndef RWKVQ_BATCH4_MINBLOCKS
#define RWKVQ_BATCH4_MINBLOCKS 4
#endif
// Batch 2..16: row tiles per wavefront.  Every wavefront reads the whole activation tile from LDS as
// its A operands; with two row tiles those reads serve twice the weights (the batched path is bound
// by LDS traffic: M = 16 gained 12-16 % per format over one row tile).
constexpr int kBRT = RWKVQ_DECODE_BATCH_RT;
static_assert(kBRT == 1 || kBRT == 2 || kBRT == 4, "row tiles of a wavefront share a 256-row codebook block");
constexpr int rt_of(int MT) { return MT == 1 ? kRT : kBRT; }
#ifndef RWKVQ_BATCH_WAVES
#define RWKVQ_BATCH_WAVES 4
#endif
// Batch 2..32: wavefronts per workgroup (4 or 8).  They share the staged activation tile, so its reads from
// the L2 (M x 512 bytes per column tile and workgroup) are spread over that many rows of W.  Measured on the
// 14B-class shapes: eight wavefronts gain 1.5-3 % on single-format stacks at batch 16 and lose 2-8 % on the
// mixed stack at batch 4 and 32 (longer tails of the larger workgroups): four is the default.
constexpr int kBW = RWKVQ_BATCH_WAVES;
static_assert(kBW == 4 || kBW == 8, "sixteen or thirty-two threads stage a batch row");
constexpr int waves_of(int MT) { return MT == 1 ? 4 : kBW; }
// Batch 2..32: row passes of a workgroup per column tile (1 or 2, a template parameter of the kernel).  With two,
// the staged activation tile (and, for VQ, the tile's codebook) serves a second stretch of rows before the
// next tile is staged: half the activation reads from the L2, half the staging work and half the barriers
// per weight (configuration 5 at batch 16: 4.44 -> 4.79 TB/s).  The launcher takes two passes when the launch
// still has RWKVQ_OPT_STREAM_TWO_PASS_MIN_WGS workgroups that way (2048 unless set), and one otherwise: a single
// 4096 x 4096 matrix is 32 workgroups of 128 rows, and halving that count costs more than the staging saves
// (25 -> 40 us at 17..32 rows).
constexpr bool kTwoPassFits = 16 * kBW * kBRT * 2 <= 256;   // the rows of a workgroup share a 256-row codebook block
constexpr int wg_rows(int MT, int P = 1) { return 16 * waves_of(MT) * rt_of(MT) * (MT == 1 ? 1 : P); }   // rows of W per workgroup

struct DecodeMat {
    const uint32_t* codes;
    const uint16_t* aux;
    const void* x;
    void* y;
    int N, K, fmt;
    int post;                         // PostOp applied to the output before it is stored (batch 1)
    const void* gate;                 // POST_SIGMOID_GATE: [N] values of the output type
};
// A matrix whose input is mixed on the fly: x (of DecodeMat) is x_t.
struct MixedMat : DecodeMat {
    const uint16_t* xprev;            // x_{t-1}, same type and length as x
    const uint8_t* mix_idx;           // K / 2 indices of the mix weight
    const uint32_t* mix_cb;           // its codebook: mix_E entries of two fp16
    int mix_E, pad2;
};
constexpr int kMaxMixedMats = 64;
constexpr int kGrid2DMaxMats = 8;     // split-K kernels: launches of at most this many matrices are two-dimensional grids (matrix, row tile)
// A matrix whose output also leaves as the token-shift mixes of the stage that follows (up to four
// projections): out_p[n] = mu_p[n] y[n] + (1 - mu_p[n]) xprev[n].
struct PostMix { const uint8_t* idx; const uint32_t* cb; void* out; };
struct PostMixMat : DecodeMat {
    const void* xprev;                // the previous token's y, type of y
    PostMix mix[4];
    int n_mix, pad2;
};
struct PostMixArgs {
    static constexpr bool kMixed = false;
    static constexpr bool kPostMix = true;
    static constexpr int kMats = kMaxMixedMats;
    int wg_end[kMaxMixedMats];
    PostMixMat m[kMaxMixedMats];
    int M, xdt, ydt, pad;
};
struct MixedDecodeArgs {
    static constexpr bool kMixed = true;
    static constexpr bool kPostMix = false;
    static constexpr int kMats = kMaxMixedMats;
    int wg_end[kMaxMixedMats];
    MixedMat m[kMaxMixedMats];
    int M, xdt, ydt, pad;
};
template <int MATS> struct DecodeTable {
    static constexpr bool kMixed = false;
    static constexpr bool kPostMix = false;
    static constexpr int kMats = MATS;
    int wg_end[MATS];                 // first workgroup index after matrix i (INT_MAX when unused)
    DecodeMat m[MATS];
    int M, xdt, ydt, pad;
};
using DecodeArgs = DecodeTable<kMaxGroupMats>;         // 15 KB of kernel arguments
// The two-dimensional grids of few matrices: filling and handing over the table above is most of what the host does for a launch
// that lasts 3 us (a 1024 x 1024 matrix at batch 1, call after call: 8.4 us with it, 7.7 with this one).
using SmallDecodeArgs = DecodeTable<kGrid2DMaxMats>;

// Batch-1 output with the element-wise operator that follows the projection in the block (App. A.1)
// applied on the way out.  The value is first rounded to the output type, as a separate pass would
// have read it from memory, then max(y, 0)^2 (Eq. "channel mixing o", input of W'_v) or
// sigma(gate) * y (the gates of Eq. "time mixing o" / "channel mixing o") in binary32, then rounded
// for the store: the same bits as the projection followed by rwkvq_relu2 / rwkvq_sigmoid_gate.
// A value of the given type as its bits, and back: what the lanes that store a row tile ask memory for at the start of
// a split-K kernel (gate, previous token, mix indices) stays bits until the end, so that nothing in front of the
// multiply waits for it (converted at once, each load is a trip to memory that the wavefront sits out).
__device__ __forceinline__ uint32_t load_bits(const void* p, size_t i, int dt) {
    return dt == DT_F32 ? ((const uint32_t*)p)[i] : (uint32_t)((const uint16_t*)p)[i];
}
__device__ __forceinline__ float bits_to_f32(uint32_t b, int dt) {
    return dt == DT_F16 ? f16_bits_to_f32((uint16_t)b) : dt == DT_BF16 ? bf16_bits_to_f32((uint16_t)b) : __uint_as_float(b);
}
// gate_bits: the gate's bits if the caller fetched them ahead (have_gate), else it is loaded here
__device__ __forceinline__ float store_post(const DecodeMat& mt, size_t i, int ydt, float v, bool have_gate = false,
                                            uint32_t gate_bits = 0) {
    if (mt.post != POST_NONE) {
        if (ydt == DT_F16) v = f16_bits_to_f32(f32_to_f16_bits(v));
        else if (ydt == DT_BF16) v = bf16_bits_to_f32(f32_to_bf16_bits(v));
        if (mt.post == POST_RELU2) {
            const float m = fmaxf(v, 0.0f);
            v = m * m;
        } else {
            v = gate_f32(have_gate ? bits_to_f32(gate_bits, ydt) : load_as_f32(mt.gate, i, ydt), v);
        }
    }
    store_from_f32(mt.y, i, ydt, v);
    return v;
}

// The same, and the stored value again as the token-shift mixes of the stage that follows (Eq. "time
// mixing r/k/v", "channel mixing r/k"): the mix is element-wise, so it can be taken where the vector is
// produced, once, instead of by every workgroup of the stage that consumes it.  Arithmetic as the mix
// pass and the fused mix: the stored (rounded) y, binary32, one rounding per operation, rounded to the type.
// The previous token's value and the indices are fetched by post_mix_prefetch at the start of the kernel
// (their latency hides behind the GEMV); the codebook entries, which depend on the indices, here, in one
// batch of loads.
struct PostMixPre { uint32_t xp, ix[4], gate; };        // as bits (see load_bits)
__device__ __forceinline__ void post_mix_prefetch(PostMixPre& pre, const PostMixMat& mt, size_t i, int ydt) {
    if (mt.post == POST_SIGMOID_GATE) pre.gate = load_bits(mt.gate, i, ydt);
    if (mt.n_mix > 0) {
        pre.xp = load_bits(mt.xprev, i, ydt);
        // every load unconditional (a mix that is not there reads the first one's index): no branch, no wait between them;
        // the aligned word that holds the index byte (a byte load is widened on the spot, which waits for it; the index
        // arrays are 16-byte aligned and N / 2 is a multiple of 8); static indices: mt stays in registers
#pragma unroll
        for (int p = 0; p < 4; ++p) pre.ix[p] = ((const uint32_t*)(p < mt.n_mix ? mt.mix[p].idx : mt.mix[0].idx))[i >> 3];
    }
}
__device__ __forceinline__ void store_post_mix(const PostMixMat& mt, size_t i, int ydt, float v, const PostMixPre& pre) {
    v = store_post(mt, i, ydt, v, true, pre.gate);
    if (mt.n_mix > 0) {
        const float xt = ydt == DT_F16 ? f16_bits_to_f32(f32_to_f16_bits(v)) : bf16_bits_to_f32(f32_to_bf16_bits(v));
        const float xp = bits_to_f32(pre.xp, ydt);
        uint32_t e[4];
#pragma unroll
        for (int p = 0; p < 4; ++p) e[p] = p < mt.n_mix ? mt.mix[p].cb[(pre.ix[p] >> (8 * ((i >> 1) & 3))) & 255u] : 0u;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            if (p < mt.n_mix) {
                const float m = f16_bits_to_f32((uint16_t)((i & 1) ? e[p] >> 16 : e[p] & 0xFFFFu));
                const float o = __fadd_rn(__fmul_rn(m, xt), __fmul_rn(__fsub_rn(1.0f, m), xp));
                store_from_f32(mt.mix[p].out, i, ydt, o);
            }
        }
    }
}

__device__ __forceinline__ half8_t vq8_operand(uint32_t w, const uint32_t* cb) {
    uint4_t v = {cb[w & 255u], cb[(w >> 8) & 255u], cb[(w >> 16) & 255u], cb[w >> 24]};
    return __builtin_bit_cast(half8_t, v);
}

// ---- activation staging (per wavefront) ----------------------------------------------------
// LDS regions are private to one wavefront and the LDS unit serves one wavefront's requests in
// issue order, so no hardware barrier is needed between a lane's store and another lane's load;
// the wavefront-scope fences only stop the compiler from moving accesses across this point.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Batch 2..32: the activation tile [MT rows][256 columns] of a column tile is shared by the wavefronts of the
// workgroup.  kRowThreads threads fetch a row of it, kRowCols columns each (rows beyond M repeat row
// M - 1: every load is unconditional, see tile_pipeline) and later store them, converted to fp16,
// into one of two LDS buffers.
struct XShared { uint4_t a, b; };           // b: only with sixteen threads per row
constexpr int kRowThreads = 4 * kBW, kRowCols = 256 / kRowThreads;

__device__ __forceinline__ void x_load_wg(XShared& r, const uint16_t* x, int M, int K, int T, int tid, int g = 0) {
    const int row = 16 * g + tid / kRowThreads < M ? 16 * g + tid / kRowThreads : M - 1;
    const uint16_t* p = x + (size_t)row * K + 256 * T + kRowCols * (tid % kRowThreads);
    r.a = *(const uint4_t*)p;
    if constexpr (kRowCols == 16) r.b = *(const uint4_t*)(p + 8);
}

// ---- bf16 activations -----------------------------------------------------------------------
// Beyond batch 1 the codes of scalar-quantized matrices are as exact in bf16 as in fp16 (sq_pair_code), and nothing is converted: 36
// 5120 x 5120 and six 17920 x 5120 and 5120 x 17920 matrices in one call 161.8 -> 147.8 us at batch 2, 191.6 -> 176.0 at 16, 282 -> 243 at
// 32 (5.7 to 6.2, 4.8 to 5.2 and 3.3 to 3.8 TB/s), what fp16 activations take.  Codebook entries (fp16) take two bf16 each, twice the
// look-up words and MFMAs: in these calls 170 -> 203 us with 6-bit VQ, so VQ converts, but in launches with a workgroup per row tile or two
// (see StageTiles).  Batch 1 multiplies fp16 (v_dot2_f32_f16; SQ codes are fp16 subnormals in place).  Where it is
// converted: fp16 holds a bf16 value exactly only for magnitudes in [2^-17, 65536).  Activations that share an accumulator (batch 1: the 64 columns a
// row of sixteen lanes multiplies in a tile; batch > 1: the 256 columns of one batch row in a tile)
// are therefore first multiplied by the power of two that brings the largest magnitude among them to
// [2^15, 2^16), and their partial sum is multiplied by the inverse power before it joins the running
// output.  Both steps are exact, so every activation within 2^-32 of its group's largest enters the
// sum exactly, whatever the magnitudes are; a smaller one is cut off below 2^-39 of that largest (the
// conversion rounds toward zero, which only matters there), far below the resolution of the
// binary32 sum it joins.
// Larger of the two halves of max(|a|, |b|) taken per bf16 half: the magnitude bits of the largest of four values.
__device__ __forceinline__ uint32_t bf16x2_absmax(uint32_t a, uint32_t b) {
    const ushort2_t m = __builtin_elementwise_max(__builtin_bit_cast(ushort2_t, a & 0x7FFF7FFFu),
                                                  __builtin_bit_cast(ushort2_t, b & 0x7FFF7FFFu));
    const uint32_t w = __builtin_bit_cast(uint32_t, m);
    return max(w >> 16, w & 0xFFFFu);
}
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_max(uint32_t v) {   // lanes the control leaves out contribute zero
    const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
    return max(v, o);
}
// All sixteen lanes of a row get the row's maximum.
__device__ __forceinline__ uint32_t dpp_row_max(uint32_t v) {
    v = dpp_max<0xB1>(v);       // quad_perm [1, 0, 3, 2]
    v = dpp_max<0x4E>(v);       // quad_perm [2, 3, 0, 1]
    v = dpp_max<0x141>(v);      // row_half_mirror
    return dpp_max<0x140>(v);   // row_mirror
}
// bf16: the threads that hold one batch row's 256 columns are one or two DPP rows of sixteen lanes; they agree
// on the row's scale for this tile, convert, and the first of them leaves the inverse scale in xsc[row].
template <int MT, bool CONVERT>
__device__ __forceinline__ void x_store_wg(const XShared& r, half_t* xs, float* xsc, int tid, int g = 0) {
    const int row = 16 * g + tid / kRowThreads;
    uint4_t a = r.a, b = r.b;
    if constexpr (CONVERT) {
        const ushort2_t m01 = __builtin_elementwise_max(__builtin_bit_cast(ushort2_t, a.x & 0x7FFF7FFFu), __builtin_bit_cast(ushort2_t, a.y & 0x7FFF7FFFu));
        const ushort2_t m23 = __builtin_elementwise_max(__builtin_bit_cast(ushort2_t, a.z & 0x7FFF7FFFu), __builtin_bit_cast(ushort2_t, a.w & 0x7FFF7FFFu));
        ushort2_t mm = __builtin_elementwise_max(m01, m23);
        if constexpr (kRowCols == 16) {
            const ushort2_t m45 = __builtin_elementwise_max(__builtin_bit_cast(ushort2_t, b.x & 0x7FFF7FFFu), __builtin_bit_cast(ushort2_t, b.y & 0x7FFF7FFFu));
            const ushort2_t m67 = __builtin_elementwise_max(__builtin_bit_cast(ushort2_t, b.z & 0x7FFF7FFFu), __builtin_bit_cast(ushort2_t, b.w & 0x7FFF7FFFu));
            mm = __builtin_elementwise_max(mm, __builtin_elementwise_max(m45, m67));
        }
        const uint32_t w = __builtin_bit_cast(uint32_t, mm);
        uint32_t amax = dpp_row_max(max(w >> 16, w & 0xFFFFu));
        if constexpr (kRowThreads == 32) amax = max(amax, (uint32_t)__shfl_xor((int)amax, 16, 64));   // the row's other sixteen lanes
        const int n = bf16_scale_exponent(amax);
        a.x = bf16x2_to_f16x2(a.x, n); a.y = bf16x2_to_f16x2(a.y, n); a.z = bf16x2_to_f16x2(a.z, n); a.w = bf16x2_to_f16x2(a.w, n);
        if constexpr (kRowCols == 16) {
            b.x = bf16x2_to_f16x2(b.x, n); b.y = bf16x2_to_f16x2(b.y, n); b.z = bf16x2_to_f16x2(b.z, n); b.w = bf16x2_to_f16x2(b.w, n);
        }
        if (tid % kRowThreads == 0) xsc[row] = ldexpf(1.0f, -n);      // rows beyond MT repeat row M - 1: written, never used
    }
    if (row < MT) {
        half_t* d = xs + row * kXStride + kRowCols * (tid % kRowThreads);
        *(uint4_t*)d = a;
        if constexpr (kRowCols == 16) *(uint4_t*)(d + 8) = b;
    }
}

// Packed weights (and their scales) are read exactly once per launch: loaded with the non-temporal hint,
// so that the stream does not displace the activations (read by every workgroup of a matrix) from the L2.
// Measured on the 7B shapes, batch 1, SQ: 5.9 -> 6.3 TB/s.
template <class T>
__device__ __forceinline__ T stream_load(const T* p) { return __builtin_nontemporal_load(p); }

// v_dot2_f32_f16 on two packed fp16 pairs.
__device__ __forceinline__ float dot2(uint32_t w, uint32_t x, float acc) {   // two fp16 pairs, scalars in
    return __builtin_amdgcn_fdot2(__builtin_bit_cast(half2_t, w), __builtin_bit_cast(half2_t, x), acc, false);
}

// v + (v of the lane that the DPP control selects); lanes the control leaves out add zero.
template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ float dpp_add(float v) {
    const int o = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROW_MASK, 0xF, ROW_MASK == 0xF);
    return v + __builtin_bit_cast(float, o);
}


// ---- per-format tile loops ------------------------------------------------------------------

// Software pipeline over the column tiles T = 0 .. KT-1 with DEPTH tiles in flight from HBM
// *while* a tile is being consumed: there is one register set more than the depth, and the load
// of tile T + DEPTH is issued before tile T is computed (a wavefront that only reloaded a set
// after consuming it would have one tile fewer in flight for the whole of its compute phase,
// which is what bounds a latency-limited stream).  Every load is unconditional, so the compiler
// counts outstanding loads exactly and waits only for the tile about to be consumed: past the
// end of the row the loads fetch the last tile again (cache hits, never used).
template <int DEPTH, class Regs, class Load, class Compute>
__device__ __forceinline__ void tile_pipeline(int KT, Load load, Compute compute) {
    static_assert(DEPTH == 1 || DEPTH == 2 || DEPTH == 3, "pipeline depth");
    const int last = KT - 1;
    auto c = [&](int T) { return T < KT ? T : last; };
    if constexpr (DEPTH == 1) {                  // two register sets: the next tile in flight while one is consumed
        Regs q0, q1;
        auto issue1 = [&](Regs& r, int T) {
            load(r, c(T));
            __builtin_amdgcn_sched_barrier(0);
        };
        __builtin_amdgcn_sched_barrier(0);
        issue1(q0, 0);
        for (int T = 0; T < KT; T += 2) {
            issue1(q1, T + 1);
            compute(q0, T);
            issue1(q0, T + 2);
            if (T + 1 < KT) compute(q1, T + 1);
        }
        return;
    }
    Regs r0, r1, r2, r3;
    // The fences keep each tile's loads together and in program order, in the prologue too: the
    // wait the compiler derives for a tile then lets all younger tiles stay in flight.
    auto issue = [&](Regs& r, int T) {
        load(r, c(T));
        __builtin_amdgcn_sched_barrier(0);
    };
    __builtin_amdgcn_sched_barrier(0);
    issue(r0, 0);
    issue(r1, 1);
    if (DEPTH == 3) issue(r2, 2);
    for (int T = 0; T < KT; T += DEPTH + 1) {
        if (DEPTH == 2) {
            issue(r2, T + 2);
            compute(r0, T);
            issue(r0, T + 3);
            if (T + 1 < KT) compute(r1, T + 1);
            issue(r1, T + 4);
            if (T + 2 < KT) compute(r2, T + 2);
        } else {
            issue(r3, T + 3);
            compute(r0, T);
            issue(r0, T + 4);
            if (T + 1 < KT) compute(r1, T + 1);
            issue(r1, T + 5);
            if (T + 2 < KT) compute(r2, T + 2);
            issue(r2, T + 6);
            if (T + 3 < KT) compute(r3, T + 3);
        }
    }
}

// Batch 2..32 with two row passes per column tile: the units of the pipeline are (tile, pass) pairs, one in
// flight while one is consumed.  Pass 0 of a tile carries the activation tile (and the codebook) and stages
// them; pass 1 streams only weights and reads what pass 0 staged.
template <int J> struct PassTag { static constexpr int value = J; };
template <class Regs, class Load, class Compute>
__device__ __forceinline__ void tile_pipeline_two_pass(int KT, Load load, Compute compute) {
    Regs q0, q1;
    const int last = KT - 1;
    __builtin_amdgcn_sched_barrier(0);
    load(q0, 0, PassTag<0>{});
    __builtin_amdgcn_sched_barrier(0);
    for (int T = 0; T < KT; ++T) {
        load(q1, T, PassTag<1>{});
        __builtin_amdgcn_sched_barrier(0);
        compute(q0, T, PassTag<0>{});
        load(q0, T < last ? T + 1 : last, PassTag<0>{});
        __builtin_amdgcn_sched_barrier(0);
        compute(q1, T, PassTag<1>{});
    }
}
template <int DEPTH, int P, class Regs, class Load, class Compute>
__device__ __forceinline__ void batched_pipeline(int KT, Load load, Compute compute) {
    static_assert(P == 1 || P == 2, "row passes per column tile");
    if constexpr (P == 2) tile_pipeline_two_pass<Regs>(KT, load, compute);
    else tile_pipeline<DEPTH, Regs>(KT, [&](Regs& r, int T) { load(r, T, PassTag<0>{}); },
                                    [&](const Regs& r, int T) { compute(r, T, PassTag<0>{}); });
}

template <int P>
__device__ __forceinline__ uint32_t vq6_lds_addr(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t m, uint32_t base) {
    // LDS byte address of codebook entry P: (index * 4) | base, base aligned to 256 bytes
    if constexpr (P < 15) {
        constexpr int p = P % 5;
        uint32_t w = (P / 5 == 0) ? w0 : (P / 5 == 1) ? w1 : w2;
        return ((w >> (6 * p)) & m) | base;
    } else {
        return ((w0 & 3u) << 2) | ((w1 & 3u) << 4) | ((w2 & 3u) << 6) | base;
    }
}
__device__ __forceinline__ uint32_t lds_gather(uint32_t byte_addr) {
    return *(const __attribute__((address_space(3))) uint32_t*)(uintptr_t)byte_addr;
}
template <int T4>
__device__ __forceinline__ uint4_t vq6_gather4(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t m, uint32_t base) {
    uint4_t v = {lds_gather(vq6_lds_addr<4 * T4 + 0>(w0, w1, w2, m, base)), lds_gather(vq6_lds_addr<4 * T4 + 1>(w0, w1, w2, m, base)),
                 lds_gather(vq6_lds_addr<4 * T4 + 2>(w0, w1, w2, m, base)), lds_gather(vq6_lds_addr<4 * T4 + 3>(w0, w1, w2, m, base))};
    return v;
}

// bf16 activations as they are: the two bf16 pairs of a codebook entry (vq_split) stand side by side in LDS, eight bytes per entry.
struct VqPair { uint4_t high, low; };
__device__ __forceinline__ uint2_t lds_gather2(uint32_t byte_addr) {
    return *(const __attribute__((address_space(3))) uint2_t*)(uintptr_t)byte_addr;
}
template <int P>                                     // LDS byte address of entry P, eight bytes each; m = 0x1f8
__device__ __forceinline__ uint32_t vq6_lds_addr8(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t m, uint32_t base) {
    if constexpr (P < 15) {
        constexpr int sh = 6 * (P % 5) - 1;
        const uint32_t w = (P / 5 == 0) ? w0 : (P / 5 == 1) ? w1 : w2;
        return ((sh < 0 ? w << 1 : w >> (sh < 0 ? 0 : sh)) & m) | base;
    } else {
        return ((w0 & 3u) << 3) | ((w1 & 3u) << 5) | ((w2 & 3u) << 7) | base;
    }
}
__device__ __forceinline__ VqPair vq_pair(uint2_t a, uint2_t b, uint2_t c, uint2_t d) { return VqPair{uint4_t{a.x, b.x, c.x, d.x}, uint4_t{a.y, b.y, c.y, d.y}}; }
template <int T4>
__device__ __forceinline__ VqPair vq6_split4(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t m, uint32_t base) {
    return vq_pair(lds_gather2(vq6_lds_addr8<4 * T4 + 0>(w0, w1, w2, m, base)), lds_gather2(vq6_lds_addr8<4 * T4 + 1>(w0, w1, w2, m, base)),
                   lds_gather2(vq6_lds_addr8<4 * T4 + 2>(w0, w1, w2, m, base)), lds_gather2(vq6_lds_addr8<4 * T4 + 3>(w0, w1, w2, m, base)));
}
__device__ __forceinline__ VqPair vq8_split4(uint32_t w, const uint2_t* cb) {
    return vq_pair(cb[w & 255u], cb[(w >> 8) & 255u], cb[(w >> 16) & 255u], cb[w >> 24]);
}

// G = groups of 16 batch rows (1 for batch <= 16, 2 for batch 17..32)
constexpr int groups_of(int MT) { return MT <= 16 ? 1 : MT / 16; }
template <int G> struct SqRegs { uint4_t a[kBRT]; uint2_t b[kBRT]; uint2_t sz[kBRT]; XShared x[G]; };
template <int G> struct Vq6Regs { uint4_t a[kBRT]; uint2_t b[kBRT]; uint32_t cb; XShared x[G]; };
template <int G> struct Vq8Regs { uint4_t a[kBRT]; uint4_t b[kBRT]; uint4_t cb; XShared x[G]; };

// Everything a tile loop needs about its wavefront's position; R[i] are its row tiles (R[i] == R[0]
// for the tiles past the end of the matrix: worked on again, not stored).
struct WavePos {
    int R[4], M, lane, tid;
    int Rn[4];           // batch > 1, second row pass: its row tiles (Rn[i] == R[0] past the end of the matrix)
    bool xbf16;
    int t0, ts, nt;      // split-K (batch 1): this wavefront's column tiles are t0, t0 + ts, ... (nt of them)
    // fused token-shift mix (batch 1): the previous token's activations, the mix weight's indices
    // (one per column pair) and its codebook staged in LDS by this wavefront
    const uint16_t* xprev;
    const uint8_t* mix_idx;
    const uint32_t* mix_cb;
};

// Batch 2..16 on the matrix cores: activations = A operand (row m of the MFMA = batch row m, read
// from the shared LDS tile), weights = B operand.  `xs` points at the two activation buffers; the
// one workgroup barrier per tile both publishes tile T and guards the buffer tile T + 1 will
// overwrite (every wavefront has finished reading it once it has passed the barrier of tile T).
//
// SQ: the codes enter as 8 + q (one shift and one and-or per pair).  The group sums of the
// activations come from the matrix cores too: one more MFMA per k-step with an all-ones B operand
// leaves X_g[m] in the accumulator layout of the products, and y += s (acc - (8 + z) X_g).
template <int MT, int DEPTH, bool XB, int P>
__device__ __forceinline__ void run_sq(const DecodeMat& mt, const WavePos& wp, half_t* xs,
                                       float4_t (&out)[P][groups_of(MT)][kBRT]) {
    constexpr int G = groups_of(MT), UB = (G == 1 && RWKVQ_BATCH_UB2) ? 2 : 1;   // one group: the fragments of both column halves up front
    using Regs = SqRegs<G>;
    const int KT = mt.K >> 8, lane = wp.lane, M = wp.M;
    const uint32_t* codes[P][kBRT];
    const uint2_t* sz[P][kBRT];
#pragma unroll
    for (int j = 0; j < P; ++j)
#pragma unroll
        for (int rt = 0; rt < kBRT; ++rt) {
            const int R = j == 0 ? wp.R[rt] : wp.Rn[rt];
            codes[j][rt] = mt.codes + (size_t)R * KT * 384;
            sz[j][rt] = (const uint2_t*)mt.aux + (size_t)R * KT * 16;
        }
    int xoff[G];
#pragma unroll
    for (int g = 0; g < G; ++g) xoff[g] = (16 * g + (lane & 15) < M ? 16 * g + (lane & 15) : M - 1) * kXStride + 8 * (lane >> 4);
    uint32_t mask, magic;
    sq_code_constants<XB>(mask, magic);
    const uint4_t ones = {kSqOne<XB>, kSqOne<XB>, kSqOne<XB>, kSqOne<XB>};
    auto load = [&](Regs& r, int T, auto pass) {
        constexpr int J = decltype(pass)::value;
#pragma unroll
        for (int rt = 0; rt < kBRT; ++rt) {
            const uint32_t* t = codes[J][rt] + (size_t)T * 384;
            r.a[rt] = stream_load((const uint4_t*)(t + 4 * lane));
            r.b[rt] = stream_load((const uint2_t*)(t + 256 + 2 * lane));
            r.sz[rt] = stream_load(sz[J][rt] + (size_t)T * 16 + (lane & 15));
        }
        if constexpr (J == 0) {
#pragma unroll
            for (int g = 0; g < G; ++g) x_load_wg(r.x[g], (const uint16_t*)mt.x, M, mt.K, T, wp.tid, g);
        }
    };
    auto compute = [&](const Regs& r, int T, auto pass) {
        constexpr int J = decltype(pass)::value;
        half_t* buf = xs + (T & 1) * (MT * kXStride);
        if constexpr (J == 0) {
#pragma unroll
            for (int g = 0; g < G; ++g) x_store_wg<MT, false>(r.x[g], buf, nullptr, wp.tid, g);
            __syncthreads();
        }
#pragma unroll
        for (int ub = 0; ub < 2; ub += UB) {
            uint4_t xa[UB][G][4];
#pragma unroll
            for (int uu = 0; uu < UB; ++uu)
#pragma unroll
                for (int g = 0; g < G; ++g)
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        xa[uu][g][t] = *(const uint4_t*)(buf + xoff[g] + 128 * (ub + uu) + 32 * t);
#pragma unroll
            for (int uu = 0; uu < UB; ++uu) {
                const int u = ub + uu;
                float4_t X[G];                       // X_g[m] for the lane's batch rows
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    X[g] = float4_t{0, 0, 0, 0};
#pragma unroll
                    for (int t = 0; t < 4; ++t) X[g] = mfma_bits<XB>(xa[uu][g][t], ones, X[g]);
                }
#pragma unroll
                for (int rt = 0; rt < kBRT; ++rt) {
                    const uint32_t w0 = u == 0 ? r.a[rt].x : r.a[rt].w, w1 = u == 0 ? r.a[rt].y : r.b[rt].x,
                                   w2 = u == 0 ? r.a[rt].z : r.b[rt].y;
                    const uint4_t op0 = sq_operand<XB, 0>(w0, w1, w2, mask, magic), op1 = sq_operand<XB, 1>(w0, w1, w2, mask, magic),
                                  op2 = sq_operand<XB, 2>(w0, w1, w2, mask, magic), op3 = sq_operand<XB, 3>(w0, w1, w2, mask, magic);
                    const uint32_t szw = u == 0 ? r.sz[rt].x : r.sz[rt].y;
                    const float s = f16_bits_to_f32((uint16_t)(szw & 0xFFFFu));
                    const float z8 = f16_bits_to_f32((uint16_t)(szw >> 16)) + 8.0f;
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        float4_t acc = {0, 0, 0, 0};
                        acc = mfma_bits<XB>(xa[uu][g][0], op0, acc);
                        acc = mfma_bits<XB>(xa[uu][g][1], op1, acc);
                        acc = mfma_bits<XB>(xa[uu][g][2], op2, acc);
                        acc = mfma_bits<XB>(xa[uu][g][3], op3, acc);
#pragma unroll
                        for (int i = 0; i < 4; ++i) out[J][g][rt][i] = fmaf(s, fmaf(-z8, X[g][i], acc[i]), out[J][g][rt][i]);
                    }
                }
            }
        }
    };
    batched_pipeline<DEPTH, P, Regs>(KT, load, compute);
}

// 6-bit VQ: the codebook of a tile (64 entries, one per lane) goes through a wavefront-private LDS
// slot and every weight pair is one ds_read_b32 gather (cheaper on this part than ds_bpermute).
template <int MT, int DEPTH, bool XB, int P>
__device__ __forceinline__ void run_vq6(const DecodeMat& mt, const WavePos& wp, half_t* xs, float* xsc, uint32_t* cb_lds,
                                        float4_t (&out)[P][groups_of(MT)][kBRT]) {
    constexpr int G = groups_of(MT), UB = (G == 1 && RWKVQ_BATCH_UB2) ? 2 : 1;
    using Regs = Vq6Regs<G>;
    const int KT = mt.K >> 8, lane = wp.lane, M = wp.M;
    const uint32_t* codes[P][kBRT];
#pragma unroll
    for (int j = 0; j < P; ++j)
#pragma unroll
        for (int rt = 0; rt < kBRT; ++rt) codes[j][rt] = mt.codes + (size_t)(j == 0 ? wp.R[rt] : wp.Rn[rt]) * KT * 384;
    const uint32_t* cbs = (const uint32_t*)mt.aux + (size_t)(wp.R[0] >> 4) * KT * 64;
    int xoff[G];
#pragma unroll
    for (int g = 0; g < G; ++g) xoff[g] = (16 * g + (lane & 15) < M ? 16 * g + (lane & 15) : M - 1) * kXStride + 8 * (lane >> 4);
    const uint32_t base0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint32_t*)cb_lds;
    uint32_t m;
    asm("v_mov_b32 %0, 0xfc" : "=v"(m));
    auto load = [&](Regs& r, int T, auto pass) {
        constexpr int J = decltype(pass)::value;
#pragma unroll
        for (int rt = 0; rt < kBRT; ++rt) {
            const uint32_t* t = codes[J][rt] + (size_t)T * 384;
            r.a[rt] = stream_load((const uint4_t*)(t + 4 * lane));
            r.b[rt] = stream_load((const uint2_t*)(t + 256 + 2 * lane));
        }
        if constexpr (J == 0) {
            r.cb = (cbs + (size_t)T * 64)[lane];
#pragma unroll
            for (int g = 0; g < G; ++g) x_load_wg(r.x[g], (const uint16_t*)mt.x, M, mt.K, T, wp.tid, g);
        }
    };
    auto compute = [&](const Regs& r, int T, auto pass) {
        constexpr int J = decltype(pass)::value;
        half_t* buf = xs + (T & 1) * (MT * kXStride);
        float* scb = xsc + (T & 1) * (16 * G);
        if constexpr (J == 0) {
#pragma unroll
            for (int g = 0; g < G; ++g) x_store_wg<MT, XB>(r.x[g], buf, scb, wp.tid, g);
            cb_lds[(T & 1) * 256 + lane] = r.cb;     // two slots, 1 KB apart (the gather address ORs the index in)
            __syncthreads();
        }
        const uint32_t base = base0 + (T & 1) * 1024;
        // bf16: the tile's products are summed on their own and join the output through the rows' inverse scales
        float4_t part[G][kBRT];
        float4_t (&acc)[G][kBRT] = *(XB ? &part : &out[J]);
        if (XB) {
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int rt = 0; rt < kBRT; ++rt) part[g][rt] = float4_t{0, 0, 0, 0};
        }
#pragma unroll
        for (int ub = 0; ub < 2; ub += UB) {
            half8_t xa[UB][G][4];
#pragma unroll
            for (int uu = 0; uu < UB; ++uu)
#pragma unroll
                for (int g = 0; g < G; ++g)
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        xa[uu][g][t] = *(const half8_t*)(buf + xoff[g] + 128 * (ub + uu) + 32 * t);
#pragma unroll
            for (int uu = 0; uu < UB; ++uu) {
                const int u = ub + uu;
#pragma unroll
                for (int rt = 0; rt < kBRT; ++rt) {
                    const uint32_t w0 = u == 0 ? r.a[rt].x : r.a[rt].w, w1 = u == 0 ? r.a[rt].y : r.b[rt].x,
                                   w2 = u == 0 ? r.a[rt].z : r.b[rt].y;
                    const half8_t op0 = __builtin_bit_cast(half8_t, vq6_gather4<0>(w0, w1, w2, m, base)),
                                  op1 = __builtin_bit_cast(half8_t, vq6_gather4<1>(w0, w1, w2, m, base)),
                                  op2 = __builtin_bit_cast(half8_t, vq6_gather4<2>(w0, w1, w2, m, base)),
                                  op3 = __builtin_bit_cast(half8_t, vq6_gather4<3>(w0, w1, w2, m, base));
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        acc[g][rt] = RWKVQ_MFMA(xa[uu][g][0], op0, acc[g][rt]);
                        acc[g][rt] = RWKVQ_MFMA(xa[uu][g][1], op1, acc[g][rt]);
                        acc[g][rt] = RWKVQ_MFMA(xa[uu][g][2], op2, acc[g][rt]);
                        acc[g][rt] = RWKVQ_MFMA(xa[uu][g][3], op3, acc[g][rt]);
                    }
                }
            }
        }
        if (XB) {
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const float4_t sc = *(const float4_t*)(scb + 16 * g + 4 * (lane >> 4));
#pragma unroll
                for (int rt = 0; rt < kBRT; ++rt)
#pragma unroll
                    for (int i = 0; i < 4; ++i) out[J][g][rt][i] = fmaf(part[g][rt][i], sc[i], out[J][g][rt][i]);
            }
        }
    };
    batched_pipeline<DEPTH, P, Regs>(KT, load, compute);
}

// 8-bit VQ: the codebook of a tile (256 entries) goes through a wavefront-private LDS region; the
// workgroup barrier that publishes the activations also orders that store before the gathers.
template <int MT, int DEPTH, bool XB, int P>
__device__ __forceinline__ void run_vq8(const DecodeMat& mt, const WavePos& wp, half_t* xs, float* xsc, uint32_t* cb_lds,
                                        float4_t (&out)[P][groups_of(MT)][kBRT]) {
    constexpr int G = groups_of(MT);
    using Regs = Vq8Regs<G>;
    const int KT = mt.K >> 8, lane = wp.lane, M = wp.M;
    const uint32_t* codes[P][kBRT];
#pragma unroll
    for (int j = 0; j < P; ++j)
#pragma unroll
        for (int rt = 0; rt < kBRT; ++rt) codes[j][rt] = mt.codes + (size_t)(j == 0 ? wp.R[rt] : wp.Rn[rt]) * KT * 512;
    const uint4_t* cbs = (const uint4_t*)mt.aux + (size_t)(wp.R[0] >> 4) * KT * 64;
    int xoff[G];
#pragma unroll
    for (int g = 0; g < G; ++g) xoff[g] = (16 * g + (lane & 15) < M ? 16 * g + (lane & 15) : M - 1) * kXStride + 8 * (lane >> 4);
    auto load = [&](Regs& r, int T, auto pass) {
        constexpr int J = decltype(pass)::value;
#pragma unroll
        for (int rt = 0; rt < kBRT; ++rt) {
            const uint32_t* t = codes[J][rt] + (size_t)T * 512;
            r.a[rt] = stream_load((const uint4_t*)(t + 4 * lane));
            r.b[rt] = stream_load((const uint4_t*)(t + 256 + 4 * lane));
        }
        if constexpr (J == 0) {
            r.cb = (cbs + (size_t)T * 64)[lane];
#pragma unroll
            for (int g = 0; g < G; ++g) x_load_wg(r.x[g], (const uint16_t*)mt.x, M, mt.K, T, wp.tid, g);
        }
    };
    auto compute = [&](const Regs& r, int T, auto pass) {
        constexpr int J = decltype(pass)::value;
        half_t* buf = xs + (T & 1) * (MT * kXStride);
        float* scb = xsc + (T & 1) * (16 * G);
        uint32_t* cbuf = cb_lds + (T & 1) * 256;     // two codebook slots, like the activations
        if constexpr (J == 0) {
#pragma unroll
            for (int g = 0; g < G; ++g) x_store_wg<MT, XB>(r.x[g], buf, scb, wp.tid, g);
            *(uint4_t*)(cbuf + 4 * lane) = r.cb;
            __syncthreads();
        }
        float4_t part[G][kBRT];                      // bf16: as in run_vq6
        float4_t (&acc)[G][kBRT] = *(XB ? &part : &out[J]);
        if (XB) {
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int rt = 0; rt < kBRT; ++rt) part[g][rt] = float4_t{0, 0, 0, 0};
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            half8_t xa[G][4];
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    xa[g][t] = *(const half8_t*)(buf + xoff[g] + 128 * u + 32 * t);
#pragma unroll
            for (int rt = 0; rt < kBRT; ++rt) {
                const uint4_t w = u == 0 ? r.a[rt] : r.b[rt];
                const half8_t op0 = vq8_operand(w.x, cbuf), op1 = vq8_operand(w.y, cbuf), op2 = vq8_operand(w.z, cbuf),
                              op3 = vq8_operand(w.w, cbuf);
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    acc[g][rt] = RWKVQ_MFMA(xa[g][0], op0, acc[g][rt]);
                    acc[g][rt] = RWKVQ_MFMA(xa[g][1], op1, acc[g][rt]);
                    acc[g][rt] = RWKVQ_MFMA(xa[g][2], op2, acc[g][rt]);
                    acc[g][rt] = RWKVQ_MFMA(xa[g][3], op3, acc[g][rt]);
                }
            }
        }
        if (XB) {
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const float4_t sc = *(const float4_t*)(scb + 16 * g + 4 * (lane >> 4));
#pragma unroll
                for (int rt = 0; rt < kBRT; ++rt)
#pragma unroll
                    for (int i = 0; i < 4; ++i) out[J][g][rt][i] = fmaf(part[g][rt][i], sc[i], out[J][g][rt][i]);
            }
        }
    };
    batched_pipeline<DEPTH, P, Regs>(KT, load, compute);
}

// ------------------------------------------------------------------------------------------
// Batch 1 (GEMV proper).  Same streaming structure and native layout, but the contraction is
// done by the vector ALU (v_dot2c_f32_f16: two multiply-adds per lane, binary32 accumulate):
// with a single activation row fifteen sixteenths of every MFMA would be spent on padding, and
// the padded MFMA costs the same issue time as the dot products.  Lane (r, kg) accumulates the part
// of row r's dot product that falls on its own columns; the four kg lanes of a row are summed at
// the end.  The activations are not staged in LDS: lane (kg, i) loads pair i of the sixteen
// column pairs that column group kg multiplies in a unit, and each dot product names the lane of
// its row that holds its pair (DPP row broadcast).
//   SQ:  the codes are multiplied in place as fp16 subnormals; per group
//        y += s * (sum q x - z * Xp), Xp = the sum of the lane's own activations of the group.
//   VQ:  the codebook of the current block sits in a wavefront-private LDS region; each pair of
//        weights is one ds_read_b32 gather feeding one dot2.

// acc += w . x, where x is the fp16 pair that lane N of the 16-lane row holds in xp (DPP
// row_newbcast): the sixteen rows' lanes of a column group all multiply by the same activations,
// which therefore need neither LDS nor a copy per lane.
template <int N>
__device__ __forceinline__ float dot2_row_bcast(float acc, uint32_t xp, uint32_t w) {
    asm("v_dot2c_f32_f16_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(acc) : "v"(xp), "v"(w), "n"(N));
    return acc;
}
// The dot products above are opaque to the compiler's hazard checks.  On this ISA the result of
// a dot instruction may be read (or overwritten) by a different vector-ALU instruction only
// three wait states later; accumulating dot products of the same kind need none.  Call this
// between the last dot product into an accumulator and any other use of it.
#define RWKVQ_DOT_RESULT_FENCE(...) asm volatile("s_nop 2" : __VA_ARGS__)

template <int T>
__device__ __forceinline__ float dot8_row_bcast(float acc, uint32_t xp, const uint4_t b) {
    const uint32_t b0 = b.x, b1 = b.y, b2 = b.z, b3 = b.w;
    acc = dot2_row_bcast<4 * T + 0>(acc, xp, b0);
    acc = dot2_row_bcast<4 * T + 1>(acc, xp, b1);
    acc = dot2_row_bcast<4 * T + 2>(acc, xp, b2);
    acc = dot2_row_bcast<4 * T + 3>(acc, xp, b3);
    return acc;
}

// Activations of a tile for the row-broadcast dot products: lane (kg, i) holds, for unit u, the
// pair of columns 128 u + 32 (i / 4) + 8 kg + 2 (i % 4) + {0, 1}, i.e. pair i of the sixteen
// that the lanes of column group kg multiply in that unit, in MFMA-step order.
struct XPairs { uint32_t p[2]; };
__device__ __forceinline__ void xpairs_load(XPairs& r, const uint16_t* x, int T, int lane) {
    const int i = lane & 15, kg = lane >> 4;
    const uint16_t* xt = x + 256 * T + 32 * (i >> 2) + 8 * kg + 2 * (i & 3);
    r.p[0] = *(const uint32_t*)xt;
    r.p[1] = *(const uint32_t*)(xt + 128);
}

// Fused token-shift mix (Eq. "time mixing r/k/v"): the wavefront loads, beside its pairs of x_t, the
// same pairs of x_{t-1} and the two index bytes of the mix weight (one 2-vector of the weight covers
// exactly one column pair), and mixes before the dot products: fl(fl(m x_t) + fl(fl(1 - m) x_{t-1}))
// per element in binary32, rounded to the activation type - the values a separate mix pass would
// have stored.
__device__ __forceinline__ void mix_load(XPairs& xq, uint32_t& mi, const WavePos& wp, int T, int lane) {
    xpairs_load(xq, wp.xprev, T, lane);
    const int i = lane & 15, kg = lane >> 4;
    const uint8_t* p = wp.mix_idx + 128 * T + 16 * (i >> 2) + 4 * kg + (i & 3);
    mi = (uint32_t)p[0] | ((uint32_t)p[64] << 8);
}
__device__ __forceinline__ uint32_t mix_pair(uint32_t xt, uint32_t xp, uint32_t entry, bool bf16) {
    const half2_t mh = __builtin_bit_cast(half2_t, entry);
    const half_t ma = mh.x, mb = mh.y;
    const float m0 = (float)ma, m1 = (float)mb;
    float t0, t1, u0, u1;
    if (bf16) {
        t0 = __uint_as_float(xt << 16); t1 = __uint_as_float(xt & 0xFFFF0000u);
        u0 = __uint_as_float(xp << 16); u1 = __uint_as_float(xp & 0xFFFF0000u);
    } else {
        const half2_t th = __builtin_bit_cast(half2_t, xt), uh = __builtin_bit_cast(half2_t, xp);
        const half_t ta = th.x, tb = th.y, ua = uh.x, ub = uh.y;
        t0 = (float)ta; t1 = (float)tb; u0 = (float)ua; u1 = (float)ub;
    }
    const float o0 = __fadd_rn(__fmul_rn(m0, t0), __fmul_rn(__fsub_rn(1.0f, m0), u0));
    const float o1 = __fadd_rn(__fmul_rn(m1, t1), __fmul_rn(__fsub_rn(1.0f, m1), u1));
    if (bf16) return (uint32_t)f32_to_bf16_bits(o0) | ((uint32_t)f32_to_bf16_bits(o1) << 16);
    return (uint32_t)f32_to_f16_bits(o0) | ((uint32_t)f32_to_f16_bits(o1) << 16);
}
template <class Regs>
__device__ __forceinline__ void mix_apply(const Regs& r, const WavePos& wp, uint32_t& x0, uint32_t& x1) {
    x0 = mix_pair(r.x.p[0], r.xq.p[0], wp.mix_cb[r.mi & 255u], wp.xbf16);
    x1 = mix_pair(r.x.p[1], r.xq.p[1], wp.mix_cb[(r.mi >> 8) & 255u], wp.xbf16);
}

struct Vq6M1Regs { uint4_t a[kRT]; uint2_t b[kRT]; uint32_t cb; XPairs x, xq; uint32_t mi; };

template <int DEPTH, bool SPLIT, bool MIXED, bool XB>
__device__ __forceinline__ void run_vq6_m1(const DecodeMat& mt, const WavePos& wp, uint32_t* cb_lds, float (&out)[kRT]) {
    const int KT = mt.K >> 8, lane = wp.lane;
    const uint32_t* codes[2] = {mt.codes + (size_t)wp.R[0] * KT * 384, mt.codes + (size_t)wp.R[1] * KT * 384};
    const uint32_t* cbs = (const uint32_t*)mt.aux + (size_t)(wp.R[0] >> 4) * KT * 64;
    const uint32_t base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint32_t*)cb_lds;
    uint32_t m;
    asm("v_mov_b32 %0, 0xfc" : "=v"(m));
    float acc1 = 0.f;                      // second accumulation chain, folded in at the end
    auto load = [&](Vq6M1Regs& r, int T) {
        if (SPLIT) T = wp.t0 + T * wp.ts;
#pragma unroll
        for (int rt = 0; rt < kRT; ++rt) {
            const uint32_t* t = codes[rt] + (size_t)T * 384;
            r.a[rt] = stream_load((const uint4_t*)(t + 4 * lane));
            r.b[rt] = stream_load((const uint2_t*)(t + 256 + 2 * lane));
        }
        r.cb = (cbs + (size_t)T * 64)[lane];
        xpairs_load(r.x, (const uint16_t*)mt.x, T, lane);
        if (MIXED) mix_load(r.xq, r.mi, wp, T, lane);
    };
    auto compute = [&](const Vq6M1Regs& r, int) {
        wave_lds_sync();
        cb_lds[lane] = r.cb;
        wave_lds_sync();
        uint32_t x0 = r.x.p[0], x1 = r.x.p[1];
        if (MIXED) mix_apply(r, wp, x0, x1);
        int nx = 0;                                       // bf16: x0, x1 enter as 2^nx times the activations
        if (XB) {
            nx = bf16_scale_exponent(dpp_row_max(bf16x2_absmax(x0, x1)));
            x0 = bf16x2_to_f16x2(x0, nx); x1 = bf16x2_to_f16x2(x1, nx);
        }
        // a DPP read needs two wait states after a vector-ALU write of the register
        asm volatile("s_nop 1" : "+v"(x0), "+v"(x1));
        // All sixteen gathers of a unit are issued before its dot products, and the second
        // unit's before the first unit's dot products, so the LDS latency is paid once per tile.
        static_assert(kRT == 1, "one row tile per wavefront");
        uint4_t g[2][4];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const uint32_t w0 = u == 0 ? r.a[0].x : r.a[0].w, w1 = u == 0 ? r.a[0].y : r.b[0].x,
                           w2 = u == 0 ? r.a[0].z : r.b[0].y;
            g[u][0] = vq6_gather4<0>(w0, w1, w2, m, base);
            g[u][1] = vq6_gather4<1>(w0, w1, w2, m, base);
            g[u][2] = vq6_gather4<2>(w0, w1, w2, m, base);
            g[u][3] = vq6_gather4<3>(w0, w1, w2, m, base);
        }
        __builtin_amdgcn_sched_barrier(0);
        // two accumulation chains (one per unit), interleaved, so that a dot product never waits
        // for the one issued just before it
        if (XB) {
            // the tile's products on their own, then into the output through the inverse scale
            float p0 = 0.f, p1 = 0.f;
            p1 = dot8_row_bcast<0>(p1, x1, g[1][0]);
            p0 = dot8_row_bcast<0>(p0, x0, g[0][0]);
            p1 = dot8_row_bcast<1>(p1, x1, g[1][1]);
            p0 = dot8_row_bcast<1>(p0, x0, g[0][1]);
            p1 = dot8_row_bcast<2>(p1, x1, g[1][2]);
            p0 = dot8_row_bcast<2>(p0, x0, g[0][2]);
            p1 = dot8_row_bcast<3>(p1, x1, g[1][3]);
            p0 = dot8_row_bcast<3>(p0, x0, g[0][3]);
            RWKVQ_DOT_RESULT_FENCE("+v"(p0), "+v"(p1));
            out[0] += ldexpf(p0 + p1, -nx);
        } else {
            acc1 = dot8_row_bcast<0>(acc1, x1, g[1][0]);
            out[0] = dot8_row_bcast<0>(out[0], x0, g[0][0]);
            acc1 = dot8_row_bcast<1>(acc1, x1, g[1][1]);
            out[0] = dot8_row_bcast<1>(out[0], x0, g[0][1]);
            acc1 = dot8_row_bcast<2>(acc1, x1, g[1][2]);
            out[0] = dot8_row_bcast<2>(out[0], x0, g[0][2]);
            acc1 = dot8_row_bcast<3>(acc1, x1, g[1][3]);
            out[0] = dot8_row_bcast<3>(out[0], x0, g[0][3]);
        }
    };
    tile_pipeline<DEPTH, Vq6M1Regs>(SPLIT ? wp.nt : KT, load, compute);
    RWKVQ_DOT_RESULT_FENCE("+v"(out[0]), "+v"(acc1));
    out[0] += acc1;
}

// Batch-1 SQ on the vector ALU.  The codes are multiplied as they are, with no 8 + q pattern: a
// 3-bit code left at mantissa bits b..b+2 of an fp16 half is the subnormal q * 2^(b-24), which
// v_dot2c_f32_f16 multiplies exactly.  A pair of codes therefore costs one AND (codes at bits 1, 4
// or 7 of the halves) or a share of one shift by 9 that brings the codes at bits 10 and 13 down
// to bits 1 and 4.  Products of different bit positions go to different accumulators (acc[0..2] for
// bits 1, 4, 7), which are combined with exact powers of two once per group.
struct SqM1Regs { uint4_t a[kRT]; uint2_t b[kRT]; uint2_t sz[kRT]; XPairs x, xq; uint32_t mi; };

template <int P>
__device__ __forceinline__ void sq_dot_pair(float (&acc)[3], uint32_t xp, uint32_t w0, uint32_t w1, uint32_t w2,
                                            uint32_t s0, uint32_t s1, uint32_t s2) {
    // s0..s2 = w0..w2 >> 9
    if constexpr (P < 15) {
        constexpr int p = P % 5;
        const uint32_t w = (P / 5 == 0) ? w0 : (P / 5 == 1) ? w1 : w2;
        const uint32_t sh = (P / 5 == 0) ? s0 : (P / 5 == 1) ? s1 : s2;
        if constexpr (p == 0) acc[0] = dot2_row_bcast<P>(acc[0], xp, w & 0x000E000Eu);
        else if constexpr (p == 1) acc[1] = dot2_row_bcast<P>(acc[1], xp, w & 0x00700070u);
        else if constexpr (p == 2) acc[2] = dot2_row_bcast<P>(acc[2], xp, w & 0x03800380u);
        else if constexpr (p == 3) acc[0] = dot2_row_bcast<P>(acc[0], xp, sh & 0x000E000Eu);
        else acc[1] = dot2_row_bcast<P>(acc[1], xp, sh & 0x00700070u);
    } else {
        // bit b of the pair's two codes sits at bits 0 and 16 of word b; assembled at bits 1..3
        const uint32_t t = (((w2 & 0x00010001u) << 1) | (w1 & 0x00010001u)) << 1 | (w0 & 0x00010001u);
        acc[0] = dot2_row_bcast<15>(acc[0], xp, t << 1);
    }
}

template <int... P>
__device__ __forceinline__ void sq_dot_pairs(float (&acc)[3], uint32_t xp, uint32_t w0, uint32_t w1, uint32_t w2,
                                             uint32_t s0, uint32_t s1, uint32_t s2) {
    (sq_dot_pair<P>(acc, xp, w0, w1, w2, s0, s1, s2), ...);
}

template <int DEPTH, bool SPLIT, bool MIXED, bool XB>
__device__ __forceinline__ void run_sq_m1(const DecodeMat& mt, const WavePos& wp, float (&out)[kRT]) {
    static_assert(kRT == 1, "one row tile per wavefront");
    const int KT = mt.K >> 8, lane = wp.lane;
    const uint32_t* codes = mt.codes + (size_t)wp.R[0] * KT * 384;
    const uint2_t* sz = (const uint2_t*)mt.aux + (size_t)wp.R[0] * KT * 16;
    auto load = [&](SqM1Regs& r, int T) {
        if (SPLIT) T = wp.t0 + T * wp.ts;
        const uint32_t* t = codes + (size_t)T * 384;
        r.a[0] = stream_load((const uint4_t*)(t + 4 * lane));
        r.b[0] = stream_load((const uint2_t*)(t + 256 + 2 * lane));
        r.sz[0] = stream_load(sz + (size_t)T * 16 + (lane & 15));
        xpairs_load(r.x, (const uint16_t*)mt.x, T, lane);
        if (MIXED) mix_load(r.xq, r.mi, wp, T, lane);
    };
    auto compute = [&](const SqM1Regs& r, int) {
        uint32_t x0 = r.x.p[0], x1 = r.x.p[1];
        if (MIXED) mix_apply(r, wp, x0, x1);
        int nx = 0;                                       // bf16: x0, x1 enter as 2^nx times the activations
        if (XB) {
            nx = bf16_scale_exponent(dpp_row_max(bf16x2_absmax(x0, x1)));
            x0 = bf16x2_to_f16x2(x0, nx); x1 = bf16x2_to_f16x2(x1, nx);
        }
        asm volatile("s_nop 1" : "+v"(x0), "+v"(x1));     // vector-ALU write -> DPP read
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const uint32_t xp = u == 0 ? x0 : x1;
            const uint32_t w0 = u == 0 ? r.a[0].x : r.a[0].w, w1 = u == 0 ? r.a[0].y : r.b[0].x,
                           w2 = u == 0 ? r.a[0].z : r.b[0].y;
            // Xp = 2^-17 times the sum of the activations this lane's column group multiplies in the
            // unit: the sixteen lanes of the row hold one pair each
            float Xp = dot2(xp, 0x00800080u, 0.f);         // 2^-17 (x_lo + x_hi): fp16 0x0080 = 2^-17
            Xp = dpp_add<0xB1>(Xp);
            Xp = dpp_add<0x4E>(Xp);
            Xp = dpp_add<0x141>(Xp);
            Xp = dpp_add<0x140>(Xp);
            float acc[3] = {0.f, 0.f, 0.f};
            sq_dot_pairs<0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15>(acc, xp, w0, w1, w2, w0 >> 9, w1 >> 9, w2 >> 9);
            RWKVQ_DOT_RESULT_FENCE("+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]));
            // sum x q = 2^17 S with S = 64 acc0 + 8 acc1 + acc2; Xp carries the same 2^-17, and so
            // does the running output, which is scaled back once at the end
            const float S = fmaf(acc[0], 64.f, fmaf(acc[1], 8.f, acc[2]));
            const uint32_t szw = u == 0 ? r.sz[0].x : r.sz[0].y;
            const float s = f16_bits_to_f32((uint16_t)(szw & 0xFFFFu));
            const float z = f16_bits_to_f32((uint16_t)(szw >> 16));
            out[0] = fmaf(XB ? ldexpf(s, -nx) : s, fmaf(-z, Xp, S), out[0]);
        }
    };
    tile_pipeline<DEPTH, SqM1Regs>(SPLIT ? wp.nt : KT, load, compute);
    out[0] *= 131072.f;
}

struct Vq8M1Regs { uint4_t a[kRT]; uint4_t b[kRT]; uint4_t cb; XPairs x, xq; uint32_t mi; };

template <int DEPTH, bool SPLIT, bool MIXED, bool XB>
__device__ __forceinline__ void run_vq8_m1(const DecodeMat& mt, const WavePos& wp, uint32_t* cb_lds, float (&out)[kRT]) {
    static_assert(kRT == 1, "one row tile per wavefront");
    const int KT = mt.K >> 8, lane = wp.lane;
    const uint32_t* codes = mt.codes + (size_t)wp.R[0] * KT * 512;
    const uint4_t* cbs = (const uint4_t*)mt.aux + (size_t)(wp.R[0] >> 4) * KT * 64;
    float acc1 = 0.f;
    auto load = [&](Vq8M1Regs& r, int T) {
        if (SPLIT) T = wp.t0 + T * wp.ts;
        const uint32_t* t = codes + (size_t)T * 512;
        r.a[0] = stream_load((const uint4_t*)(t + 4 * lane));
        r.b[0] = stream_load((const uint4_t*)(t + 256 + 4 * lane));
        r.cb = (cbs + (size_t)T * 64)[lane];
        xpairs_load(r.x, (const uint16_t*)mt.x, T, lane);
        if (MIXED) mix_load(r.xq, r.mi, wp, T, lane);
    };
    auto compute = [&](const Vq8M1Regs& r, int) {
        wave_lds_sync();
        *(uint4_t*)(cb_lds + 4 * lane) = r.cb;
        wave_lds_sync();
        uint32_t x0 = r.x.p[0], x1 = r.x.p[1];
        if (MIXED) mix_apply(r, wp, x0, x1);
        int nx = 0;                                       // bf16: x0, x1 enter as 2^nx times the activations
        if (XB) {
            nx = bf16_scale_exponent(dpp_row_max(bf16x2_absmax(x0, x1)));
            x0 = bf16x2_to_f16x2(x0, nx); x1 = bf16x2_to_f16x2(x1, nx);
        }
        asm volatile("s_nop 1" : "+v"(x0), "+v"(x1));     // vector-ALU write -> DPP read
        uint4_t g[2][4];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const uint4_t w = u == 0 ? r.a[0] : r.b[0];
            g[u][0] = __builtin_bit_cast(uint4_t, vq8_operand(w.x, cb_lds));
            g[u][1] = __builtin_bit_cast(uint4_t, vq8_operand(w.y, cb_lds));
            g[u][2] = __builtin_bit_cast(uint4_t, vq8_operand(w.z, cb_lds));
            g[u][3] = __builtin_bit_cast(uint4_t, vq8_operand(w.w, cb_lds));
        }
        __builtin_amdgcn_sched_barrier(0);
        if (XB) {
            // the tile's products on their own, then into the output through the inverse scale
            float p0 = 0.f, p1 = 0.f;
            p1 = dot8_row_bcast<0>(p1, x1, g[1][0]);
            p0 = dot8_row_bcast<0>(p0, x0, g[0][0]);
            p1 = dot8_row_bcast<1>(p1, x1, g[1][1]);
            p0 = dot8_row_bcast<1>(p0, x0, g[0][1]);
            p1 = dot8_row_bcast<2>(p1, x1, g[1][2]);
            p0 = dot8_row_bcast<2>(p0, x0, g[0][2]);
            p1 = dot8_row_bcast<3>(p1, x1, g[1][3]);
            p0 = dot8_row_bcast<3>(p0, x0, g[0][3]);
            RWKVQ_DOT_RESULT_FENCE("+v"(p0), "+v"(p1));
            out[0] += ldexpf(p0 + p1, -nx);
        } else {
            acc1 = dot8_row_bcast<0>(acc1, x1, g[1][0]);
            out[0] = dot8_row_bcast<0>(out[0], x0, g[0][0]);
            acc1 = dot8_row_bcast<1>(acc1, x1, g[1][1]);
            out[0] = dot8_row_bcast<1>(out[0], x0, g[0][1]);
            acc1 = dot8_row_bcast<2>(acc1, x1, g[1][2]);
            out[0] = dot8_row_bcast<2>(out[0], x0, g[0][2]);
            acc1 = dot8_row_bcast<3>(acc1, x1, g[1][3]);
            out[0] = dot8_row_bcast<3>(out[0], x0, g[0][3]);
        }
    };
    tile_pipeline<DEPTH, Vq8M1Regs>(SPLIT ? wp.nt : KT, load, compute);
    RWKVQ_DOT_RESULT_FENCE("+v"(out[0]), "+v"(acc1));
    out[0] += acc1;
}

// The batch-1 tile loop of a matrix's format; XB = the activations are bf16.
template <int DEPTH, bool SPLIT, bool MIXED>
__device__ __forceinline__ void run_m1(const DecodeMat& mt, const WavePos& wp, uint32_t* cb_lds, float (&part)[kRT]) {
    if (wp.xbf16) {
        if (mt.fmt == FMT_SQ3) run_sq_m1<DEPTH, SPLIT, MIXED, true>(mt, wp, part);
        else if (mt.fmt == FMT_VQ6) run_vq6_m1<DEPTH, SPLIT, MIXED, true>(mt, wp, cb_lds, part);
        else run_vq8_m1<DEPTH, SPLIT, MIXED, true>(mt, wp, cb_lds, part);
    } else {
        if (mt.fmt == FMT_SQ3) run_sq_m1<DEPTH, SPLIT, MIXED, false>(mt, wp, part);
        else if (mt.fmt == FMT_VQ6) run_vq6_m1<DEPTH, SPLIT, MIXED, false>(mt, wp, cb_lds, part);
        else run_vq8_m1<DEPTH, SPLIT, MIXED, false>(mt, wp, cb_lds, part);
    }
}
// The same for batch 2..32.
template <int MT, int DEPTH, int P>
__device__ __forceinline__ void run_batched(const DecodeMat& mt, const WavePos& wp, half_t* xs, float* xsc, uint32_t* cb_lds,
                                            float4_t (&out)[P][groups_of(MT)][kBRT]) {
    if (wp.xbf16) {
        if (mt.fmt == FMT_SQ3) run_sq<MT, DEPTH, true, P>(mt, wp, xs, out);
        else if (mt.fmt == FMT_VQ6) run_vq6<MT, DEPTH, true, P>(mt, wp, xs, xsc, cb_lds, out);
        else run_vq8<MT, DEPTH, true, P>(mt, wp, xs, xsc, cb_lds, out);
    } else {
        if (mt.fmt == FMT_SQ3) run_sq<MT, DEPTH, false, P>(mt, wp, xs, out);
        else if (mt.fmt == FMT_VQ6) run_vq6<MT, DEPTH, false, P>(mt, wp, xs, xsc, cb_lds, out);
        else run_vq8<MT, DEPTH, false, P>(mt, wp, xs, xsc, cb_lds, out);
    }
}

// Workgroups per compute unit the compiler must leave registers for: the macros give wavefronts per SIMD.
constexpr int min_blocks(int MT) {
    if (MT == 1) return RWKVQ_DECODE_MINBLOCKS;
    const int per_simd = MT == 4 ? RWKVQ_BATCH4_MINBLOCKS : MT == 16 ? RWKVQ_BATCH16_MINBLOCKS : 2;
    return per_simd * 4 / kBW > 0 ? per_simd * 4 / kBW : 1;
}

// MT = number of activation rows carried (1, 4, 16 or 32 >= M).  MT = 1 runs every format on the
// vector ALU (run_*_m1); the others on the matrix cores, whose D layout is: lane holds batch rows
// 4*(lane/16) + i of output column lane%16.
template <int MT, int P = 1>
__global__ void __launch_bounds__(64 * waves_of(MT), min_blocks(MT)) decode_kernel(DecodeArgs a) {
    static_assert(MT > 1 || P == 1, "batch 1 has no staged activation tile to share");
    constexpr int DEPTH = MT == 1 ? RWKVQ_DECODE_DEPTH : RWKVQ_BATCH_DEPTH;
    // batch > 1: two activation tiles shared by the workgroup; codebook slots per wavefront
    __shared__ __attribute__((aligned(16))) half_t xs[MT == 1 ? 8 : 2 * MT * kXStride];
    __shared__ __attribute__((aligned(1024))) uint32_t cb_all[waves_of(MT)][MT == 1 ? 256 : 512];
    __shared__ __attribute__((aligned(16))) float xsc[MT == 1 ? 4 : 2 * 16 * groups_of(MT)];   // bf16: inverse scales per tile and batch row

    // Which matrix does this workgroup belong to?  Lane i compares against the end of matrix i
    // (one load per wavefront from the argument block); the count of matrices that end at or
    // before this workgroup is its matrix index.
    const int wg = blockIdx.x;
    static_assert(kMaxGroupMats % 64 == 0, "one table entry per lane and pass");
    int mi = 0;
#pragma unroll
    for (int j = 0; j < kMaxGroupMats; j += 64)
        mi += __builtin_popcountll(__builtin_amdgcn_ballot_w64(wg >= a.wg_end[j + (threadIdx.x & 63)]));
    const DecodeMat mt = a.m[mi];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int M = a.M;
    const bool xbf16 = a.xdt == DT_BF16;

    const int NR = mt.N >> 4;
    WavePos wp;
    constexpr int RT = rt_of(MT);
    wp.R[0] = RT * (waves_of(MT) * P * (wg - (mi ? a.wg_end[mi - 1] : 0)) + wave);
    const bool live = wp.R[0] < NR;                // rows beyond N (N not a multiple of the workgroup's rows)
    wp.M = M; wp.lane = lane; wp.tid = threadIdx.x; wp.xbf16 = xbf16;

    if constexpr (MT == 1) {
        if (!live) return;
        wp.R[1] = wp.R[2] = wp.R[3] = wp.R[0];
        float part[kRT];
#pragma unroll
        for (int rt = 0; rt < kRT; ++rt) part[rt] = 0.f;
        run_m1<DEPTH, false, false>(mt, wp, cb_all[wave], part);
#pragma unroll
        for (int rt = 0; rt < kRT; ++rt) {
            float v = part[rt];                    // sum the four column groups of each row
            v += __shfl_xor(v, 16, 64);
            v += __shfl_xor(v, 32, 64);
            if (lane < 16) store_post(mt, (size_t)16 * wp.R[rt] + lane, a.ydt, v);
        }
    } else {
        // every wavefront takes part in the shared activation tiles and their barriers; one
        // beyond the last row tile works on the last tile again and stores nothing
        if (!live) wp.R[0] = NR - 1;
#pragma unroll
        for (int rt = 1; rt < 4; ++rt) wp.R[rt] = (rt < RT && wp.R[0] + rt < NR) ? wp.R[0] + rt : wp.R[0];
        // second pass: the same positions one stretch of waves_of(MT) * RT row tiles further on
#pragma unroll
        for (int rt = 0; rt < 4; ++rt) {
            const int r2 = wp.R[0] + RT * waves_of(MT) + rt;
            wp.Rn[rt] = (live && rt < RT && r2 < NR) ? r2 : wp.R[0];
        }
        constexpr int G = groups_of(MT);
        float4_t out[P][G][RT];
#pragma unroll
        for (int j = 0; j < P; ++j)
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) out[j][g][rt] = float4_t{0, 0, 0, 0};
        run_batched<MT, DEPTH, P>(mt, wp, xs, xsc, cb_all[wave], out);
        if (!live) return;
        if (xbf16 && mt.fmt == FMT_SQ3 && __builtin_expect(any_infinite(reinterpret_cast<float4_t (&)[P * G * RT]>(out)), 0)) {
#pragma unroll 1
            for (int at = 0; at < P * G * RT; ++at) {              // (see scaled_row_tile)
                const int row_tile = wp.R[0] + RT * waves_of(MT) * (at / (G * RT)) + at % RT;
                const float4_t v = scaled_row_tile(mt, row_tile < NR ? row_tile : wp.R[0], 16 * (at / RT % G), M, 0, 1, lane);
#pragma unroll
                for (int j = 0; j < P * G * RT; ++j) {
                    float4_t& o = out[j / (G * RT)][j / RT % G][j % RT];
                    o = j == at ? if_infinite(o, v) : o;
                }
            }
        }
        // D layout of the MFMA: lane (n, mg) holds batch rows 4 mg .. 4 mg + 3 (of its group) of output column n
#pragma unroll
        for (int j = 0; j < P; ++j)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                const int R = j == 0 ? wp.R[rt] : wp.Rn[rt];
                if ((j > 0 || rt > 0) && R == wp.R[0]) continue;
                const int n = 16 * R + (lane & 15);
#pragma unroll
                for (int g = 0; g < G; ++g)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int m = 16 * g + 4 * (lane >> 4) + i;
                        if (m < M) store_from_f32(mt.y, (size_t)m * mt.N + n, a.ydt, out[j][g][rt][i]);
                    }
            }
    }
}

// Batch 1 when a launch holds too few row tiles to fill the device (a single projection, the
// matrices of one stage of a block): one workgroup per 16-row tile, its S wavefronts take the
// column tiles s, s + S, s + 2S, ... and their partial sums meet in LDS in a fixed order.  The
// grouped kernel above gives one wavefront a whole row tile, which keeps 4096 x 4096 on a quarter
// of the SIMDs.
template <int S, class Args, bool GRID2D>
__global__ void __launch_bounds__(64 * S) decode_splitk_kernel(Args a) {
    constexpr int DEPTH = RWKVQ_DECODE_DEPTH;
    constexpr bool MIXED = Args::kMixed;
    static_assert(kRT == 1, "one row tile per wavefront");
    __shared__ __attribute__((aligned(1024))) uint32_t cb_all[S][256];
    __shared__ uint32_t cb_mix[MIXED ? S : 1][256];
    __shared__ float red[S][16];
    // Which matrix, which row tile?  A launch of a few matrices (a stage of a block) is a two-dimensional grid,
    // blockIdx.y the matrix and blockIdx.x the row tile (workgroups past a shorter matrix's last tile leave at once):
    // the descriptor is then one load away.  The table of first-workgroup indices of the other form costs a load of
    // its own in front of it, and these launches last three or four trips to memory in all.
    int mi = 0, tile;
    if constexpr (GRID2D) {
        mi = blockIdx.y;
        tile = blockIdx.x;
    } else {
        const int wg = blockIdx.x;
#pragma unroll
        for (int j = 0; j < Args::kMats; j += 64)
            mi += __builtin_popcountll(__builtin_amdgcn_ballot_w64(wg >= a.wg_end[j + (threadIdx.x & 63)]));
        tile = wg - (mi ? a.wg_end[mi - 1] : 0);                                   // here wg_end counts row tiles
    }
    const int xdt = a.xdt, ydt = a.ydt;    // the end of the argument block: asked for together with the descriptor
    const auto mt = a.m[mi];
    asm volatile("" :: "s"(xdt), "s"(ydt), "s"(mt.N));
    if (GRID2D && tile >= ((mt.N + 15) >> 4)) return;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int KT = mt.K >> 8;
    WavePos wp;
    wp.R[0] = wp.R[1] = wp.R[2] = wp.R[3] = tile;
    wp.M = 1; wp.lane = lane; wp.tid = threadIdx.x; wp.xbf16 = xdt == DT_BF16;
    wp.t0 = wave; wp.ts = S; wp.nt = wave < KT ? (KT - wave + S - 1) / S : 0;
    if constexpr (MIXED) {
        for (int e = lane; e < mt.mix_E; e += 64) cb_mix[wave][e] = mt.mix_cb[e];
        wave_lds_sync();
        wp.xprev = mt.xprev; wp.mix_idx = mt.mix_idx; wp.mix_cb = cb_mix[wave];
    }
    PostMixPre pre{};
    if constexpr (Args::kPostMix) {
        if (wave == 0 && lane < 16) post_mix_prefetch(pre, mt, (size_t)16 * wp.R[0] + lane, ydt);
    } else {
        if (wave == 0 && lane < 16 && mt.post == POST_SIGMOID_GATE) pre.gate = load_bits(mt.gate, (size_t)16 * wp.R[0] + lane, ydt);
    }
    float part[kRT] = {0.f};
    if (wp.nt > 0) {
        run_m1<DEPTH, true, MIXED>(mt, wp, cb_all[wave], part);
    }
    float v = part[0];                             // sum the four column groups of each row
    v += __shfl_xor(v, 16, 64);
    v += __shfl_xor(v, 32, 64);
    if (lane < 16) red[wave][lane] = v;
    __syncthreads();
    if (wave == 0 && lane < 16) {
        float t = red[0][lane];
#pragma unroll
        for (int s = 1; s < S; ++s) t += red[s][lane];
        if constexpr (Args::kPostMix) store_post_mix(mt, (size_t)16 * wp.R[0] + lane, ydt, t, pre);
        else store_post(mt, (size_t)16 * wp.R[0] + lane, ydt, t, true, pre.gate);
    }
}

// ---- batch 2..16, small launches ------------------------------------------------------------
// What a row tile of a column tile is read into.
struct StageRegs {
    uint4_t a, b;                      // packed words; SQ: b = two words, scale and zero of both groups; VQ-6: b.z = codebook entry
    uint4_t cb;                        // VQ-8: four codebook entries
};
// Row tiles in flight.  The sets rotate with the row tiles of one column tile, or of two (MULTI).
constexpr int stage_sets(int R, bool multi) { return R == 6 ? 3 : multi && R == 1 ? 2 : R; }

template <bool DIRECT> constexpr int kStageSlot = DIRECT ? 512 : 256;   // words of a codebook slot
constexpr bool stage_as_is(int fmt, int R) { return fmt == FMT_SQ3 || R <= (fmt == FMT_VQ6 ? 2 : 1); }
template <int FMT, int R, bool MULTI, bool XB, bool AS_IS = stage_as_is(FMT, R)>
struct StageTiles {
    static constexpr int D = stage_sets(R, MULTI);
    static constexpr bool kOneBlock = 16 % R == 0;   // the row tiles share a codebook block
    // bf16 activations: as they are, or brought into fp16.  SQ codes are exact in either type.  VQ entries as two bf16 pairs take two
    // look-up words and two MFMAs where the conversion takes 235 instructions per column tile, for all row tiles: 6-bit VQ with up to two
    // of them, 8-bit with one (its look-ups of eight bytes meet in twice the banks).  Measured (us, converted -> as they are): 4096 x 4096
    // SQ at M = 2 5.8 -> 4.8, at 16 7.2 -> 6.7, 4096 x 14336 at 2 14.8 -> 11.4, 6-bit VQ 14.5 -> 11.7, 8-bit 15.4 -> 13.7; 17920 x 5120 and
    // 5120 x 5120 SQ (six row tiles) at 2 17.8 -> 12.8.  VQ of five row tiles at 2 10.7 -> 11.1, of two in 8 bits 5.4 -> 5.6 (converted);
    // with three and four column tiles the split of the codebook is not won back: 8192 x 768 6-bit VQ at 2 3.7 -> 4.0 (two row tiles:
    // converted there), 4096 x 1024 8-bit 3.6 -> 3.75, but 512 x 768 2.9 -> 2.8 (one: as they are).
    static constexpr bool kDirect = XB && AS_IS, kConvert = XB && !kDirect;
    static constexpr int kWords = FMT == FMT_VQ8 ? 512 : 384;
    const DecodeMat& mt;
    int R0, NR, KT, lane, xoff;
    float* xsc;
    uint32_t* cb_lds;
    uint32_t mask, magic, m6, base0;
    StageRegs w[D];
    XFrags xf[MULTI ? 2 : 1];

    __device__ __forceinline__ StageTiles(const DecodeMat& mt_, int R0_, int M, int lane_, float* xsc_, uint32_t* cb_)
        : mt(mt_), R0(R0_), NR(mt_.N >> 4), KT(mt_.K >> 8), lane(lane_), xsc(xsc_), cb_lds(cb_) {
        xoff = ((lane & 15) < M ? lane & 15 : M - 1) * mt.K + 8 * (lane >> 4);
        sq_code_constants<kDirect>(mask, magic);
        asm("v_mov_b32 %0, %1" : "=v"(m6) : "n"(kDirect ? 0x1f8 : 0xfc));
        base0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint32_t*)cb_lds;
    }
    // A column tile's activation fragments (XFrags, straight from memory: nothing is staged for the workgroup, no barrier), a row
    // tile's weights: together and in order (see tile_pipeline).  Past the
    // end (live = false) every lane asks for lane 0's bytes of a tile that was read already.
    __device__ __forceinline__ void load_x(XFrags& r, int T, bool live) {
        const uint16_t* p = (const uint16_t*)mt.x + 256 * T;
        const uint32_t at = live ? (uint32_t)xoff : 0u;
#pragma unroll
        for (int i = 0; i < 8; ++i) r.f[i] = *(const uint4_t*)(p + at + 128 * (i >> 2) + 32 * (i & 3));
        __builtin_amdgcn_sched_barrier(0);
    }
    __device__ __forceinline__ void load_w(StageRegs& r, int T, int rt, bool live) {
        const int row = R0 + rt < NR ? R0 + rt : NR - 1;                     // past the last row tile: that one again, not stored
        const uint32_t l = live ? (uint32_t)lane : 0u;
        const uint32_t* t = mt.codes + ((size_t)row * KT + T) * kWords;
        r.a = stream_load((const uint4_t*)t + l);
        if constexpr (FMT == FMT_VQ8) {
            r.b = stream_load((const uint4_t*)(t + 256) + l);
            if (!kOneBlock || rt == 0) r.cb = ((const uint4_t*)mt.aux + ((size_t)(row >> 4) * KT + T) * 64)[l];
        } else {
            const uint2_t two = stream_load((const uint2_t*)(t + 256) + l);
            r.b.x = two.x; r.b.y = two.y;
            if constexpr (FMT == FMT_SQ3) {
                const uint2_t sz = stream_load((const uint2_t*)mt.aux + ((size_t)row * KT + T) * 16 + (l & 15u));
                r.b.z = sz.x; r.b.w = sz.y;
            } else if (!kOneBlock || rt == 0) {
                r.b.z = ((const uint32_t*)mt.aux + ((size_t)(row >> 4) * KT + T) * 64)[l];
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    __device__ __forceinline__ void multiply(const StageRegs& r, const XFrags& x, int rt, const float4_t& sc, const float4_t (&X)[2], float4_t& out) {
        const uint32_t slot = (uint32_t)(kOneBlock ? 0 : rt & 1);
        uint32_t* const cbuf = cb_lds + kStageSlot<kDirect> * slot;
        if constexpr (FMT != FMT_SQ3) {
            if (!kOneBlock || rt == 0) {
                if constexpr (kDirect && FMT == FMT_VQ8) {
                    const uint2_t e0 = vq_split(r.cb.x), e1 = vq_split(r.cb.y), e2 = vq_split(r.cb.z), e3 = vq_split(r.cb.w);
                    *(uint4_t*)(cbuf + 8 * lane) = uint4_t{e0.x, e0.y, e1.x, e1.y};
                    *(uint4_t*)(cbuf + 8 * lane + 4) = uint4_t{e2.x, e2.y, e3.x, e3.y};
                } else if constexpr (kDirect) {
                    *(uint2_t*)(cbuf + 2 * lane) = vq_split(r.b.z);
                } else if constexpr (FMT == FMT_VQ8) {
                    *(uint4_t*)(cbuf + 4 * lane) = r.cb;
                } else {
                    cbuf[lane] = r.b.z;
                }
                wave_lds_sync();
            }
        }
        float4_t part = {0, 0, 0, 0};
        float4_t& acc = *(kConvert ? &part : &out);                          // (as in run_vq6)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const uint32_t w0 = u == 0 ? r.a.x : r.a.w, w1 = u == 0 ? r.a.y : r.b.x, w2 = u == 0 ? r.a.z : r.b.y;
            if constexpr (FMT == FMT_SQ3) {
                const uint4_t op[4] = {sq_operand<kDirect, 0>(w0, w1, w2, mask, magic), sq_operand<kDirect, 1>(w0, w1, w2, mask, magic),
                                       sq_operand<kDirect, 2>(w0, w1, w2, mask, magic), sq_operand<kDirect, 3>(w0, w1, w2, mask, magic)};
                const uint32_t szw = u == 0 ? r.b.z : r.b.w;
                const float s = f16_bits_to_f32((uint16_t)(szw & 0xFFFFu));
                const float z8 = f16_bits_to_f32((uint16_t)(szw >> 16)) + 8.0f;
                float4_t sum = {0, 0, 0, 0};
#pragma unroll
                for (int t = 0; t < 4; ++t) sum = mfma_bits<kDirect>(x.f[4 * u + t], op[t], sum);
#pragma unroll
                for (int i = 0; i < 4; ++i) out[i] = fmaf(s, fmaf(-z8, X[u][i], sum[i]), out[i]);
            } else if constexpr (kDirect) {
                const uint32_t base = base0 + 4 * kStageSlot<kDirect> * slot;
                const uint4_t q = u == 0 ? r.a : r.b;
                const uint2_t* const cb = (const uint2_t*)cbuf;
                VqPair op[4];
                if constexpr (FMT == FMT_VQ8) { op[0] = vq8_split4(q.x, cb); op[1] = vq8_split4(q.y, cb); op[2] = vq8_split4(q.z, cb); op[3] = vq8_split4(q.w, cb); }
                else {
                    op[0] = vq6_split4<0>(w0, w1, w2, m6, base); op[1] = vq6_split4<1>(w0, w1, w2, m6, base);
                    op[2] = vq6_split4<2>(w0, w1, w2, m6, base); op[3] = vq6_split4<3>(w0, w1, w2, m6, base);
                }
#pragma unroll
                for (int t = 0; t < 4; ++t) out = mfma_bits<true>(x.f[4 * u + t], op[t].low, mfma_bits<true>(x.f[4 * u + t], op[t].high, out));
            } else {
                const uint32_t base = base0 + 4 * kStageSlot<kDirect> * slot;
                const uint4_t q = u == 0 ? r.a : r.b;
                half8_t op[4];
                if constexpr (FMT == FMT_VQ8) { op[0] = vq8_operand(q.x, cbuf); op[1] = vq8_operand(q.y, cbuf); op[2] = vq8_operand(q.z, cbuf); op[3] = vq8_operand(q.w, cbuf); }
                else {
                    op[0] = __builtin_bit_cast(half8_t, vq6_gather4<0>(w0, w1, w2, m6, base));
                    op[1] = __builtin_bit_cast(half8_t, vq6_gather4<1>(w0, w1, w2, m6, base));
                    op[2] = __builtin_bit_cast(half8_t, vq6_gather4<2>(w0, w1, w2, m6, base));
                    op[3] = __builtin_bit_cast(half8_t, vq6_gather4<3>(w0, w1, w2, m6, base));
                }
#pragma unroll
                for (int t = 0; t < 4; ++t) acc = RWKVQ_MFMA(__builtin_bit_cast(half8_t, x.f[4 * u + t]), op[t], acc);
            }
        }
        if (kConvert)
#pragma unroll
            for (int i = 0; i < 4; ++i) out[i] = fmaf(part[i], sc[i], out[i]);
    }
    // Column tile T, whose fragments are in xf[J]; the weights of the row tiles D further on and the fragments of the column
    // tile after next are asked for as the registers become free.
    template <int J>
    __device__ __forceinline__ void column(int T, int S, int last, float4_t (&out)[R]) {
        XFrags& x = xf[J];
        float4_t sc = {1, 1, 1, 1};
        if (kConvert) {
            const int n = x_frags_exponent(x.f);
#pragma unroll
            for (int i = 0; i < 8; ++i) x.f[i] = x_frag_to_f16(x.f[i], n);
            if (lane < 16) xsc[lane] = ldexpf(1.0f, -n);
            wave_lds_sync();
            sc = *(const float4_t*)(xsc + 4 * (lane >> 4));
        }
        // group sums of the activations, for all row tiles
        const uint4_t ones = {kSqOne<kDirect>, kSqOne<kDirect>, kSqOne<kDirect>, kSqOne<kDirect>};
        float4_t X[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
        if constexpr (FMT == FMT_SQ3) {
#pragma unroll
            for (int i = 0; i < 8; ++i) X[i >> 2] = mfma_bits<kDirect>(x.f[i], ones, X[i >> 2]);
        }
#pragma unroll
        for (int rt = 0; rt < R; ++rt) {
            StageRegs& r = w[(J * R + rt) % D];
            multiply(r, x, rt, sc, X, out[rt]);
            if (MULTI && rt + 1 == R) load_x(x, T + 2 * S <= last ? T + 2 * S : last, T + 2 * S <= last);
            constexpr int ahead = D;
            const int turn = (rt + ahead) / R, to = (rt + ahead) % R;         // the row tile this set serves next
            if (turn == 0) load_w(r, T, to, true);
            else if (MULTI) load_w(r, T + turn * S <= last ? T + turn * S : last, to, T + turn * S <= last);
        }
    }
    // y[m][16 row tiles] over the column tiles t0, t0 + S, .. (nt of them; one if not MULTI), added to out.
    __device__ __forceinline__ void run(int t0, int S, int nt, float4_t (&out)[R]) {
        const int last = t0 + (nt - 1) * S;
        __builtin_amdgcn_sched_barrier(0);
        load_x(xf[0], t0, true);
#pragma unroll
        for (int i = 0; i < D; ++i) {
            if (MULTI && i == R) load_x(xf[MULTI], nt > 1 ? t0 + S : t0, nt > 1);
            if (i < R) load_w(w[i], t0, i, true);
            else load_w(w[i], nt > 1 ? t0 + S : t0, i - R, nt > 1);
        }
        if (MULTI && D <= R) load_x(xf[MULTI], nt > 1 ? t0 + S : t0, nt > 1);
        if constexpr (!MULTI) column<0>(t0, S, last, out);
        else
#pragma unroll 1
            for (int T = t0; T <= last; T += 2 * S) {
                column<0>(T, S, last, out);
                if (T + S <= last) column<1>(T + S, S, last, out);
            }
    }
};

// Batch 2..16 when a launch holds too few rows to fill the device with the kernel above (a single projection, the matrices of one
// stage of a block): a workgroup takes R row tiles of one matrix, its S wavefronts the column tiles s, s + S, ..., and the partial
// sums meet in LDS in a fixed order.  A wavefront fetches the activations of a column tile once, straight into the operand layout
// of the MFMA, and they serve R row tiles; nothing is staged for the workgroup, no barrier sits in the loop.
// What bounds it: start-up (about 4.5 us of a launch that moves nothing), then x: a compute unit reads all of x (131 KB at M = 16,
// K = 4096) in pieces of 64 bytes per batch row, half of a cache line at a time.  (Whole lines, two of the loads exchanging half of every
// DPP row in registers, were 0 to 11 % slower: the other half of a line is found in the L1, and the exchange costs.)  With 16
// wavefronts of one column tile each every byte of a workgroup is
// asked for at its start.  Measured (7B shapes, fp16 SQ, cold weights, us at M = 2 / 16), a workgroup per 32 rows of W with 4 or 8
// wavefronts (what this replaces) -> here: {r, k, v, g} 10.0 / 13.6 -> 7.8 / 9.8, o 6.1 / 8.9 -> 5.1 / 6.8, {k', r'} 12.6 / 19.1
// -> 8.8 / 11.1, v' 13.1 / 21.5 -> 11.5 / 18.2.
// most wavefronts of a workgroup: 128 registers each, or 168 where several column tiles are in flight.  Five and six row tiles spill up
// to seven of the 168; eight wavefronts of 256 spill none and were no better (us, batch 8, twelve -> eight: 20480 x 8192, fp16 SQ 18.7 ->
// 17.6 and bf16 VQ 22.3 -> 20.9, but 24576 x 4352 12.5 -> 13.4 and 13.8 -> 16.2: its 17 column tiles take three turns in place of two).
constexpr int stage_waves(bool multi, int R) { return multi && R > 1 ? 12 : 16; }
// MOST: wavefronts on a SIMD that the compiler may make room for, which costs registers and so loads in flight.  Left to itself (8) it
// makes room for four with two row tiles and several column tiles, for six with one column tile.  Rows of mixed lengths, whose long
// workgroups the launch waits for, run better with more loads in flight as long as nearly all of the launch stands on the device (`few` in
// launch_stage; us, left to itself -> held): {8192 x 2304, 2304 x 8192} SQ in fp16 at M = 14 16.7 -> 13.2, {4608 x 1280, 1280 x 4608} 6-bit
// VQ at 8 9.3 -> 7.9, layers of d = 2048 SQ at 2 13.7 -> 12.2, of 3072 (1008 workgroups of four) 8-bit VQ in fp16 at 16 31.8 -> 28.1, of 768 (one
// column tile) at 12 7.0 -> 6.2.  Not so beyond (a layer of d = 1280, 424 workgroups of six, at 3 in bf16 9.5 -> 11.5; of 3328, 1096 of four, 28.6
// -> 30.1, two of 1536, 1008 of four, at 5 13.9 -> 14.8, but five scalar-quantized matrices, 1050 of four, in fp16 at 11 24.4 -> 21.2) and
// not for rows of one length (5120 x 17920 8-bit VQ in bf16 at 8 23.8 -> 24.8, 40960 x 256 SQ at 2 4.0 -> 4.7).  More than 410 workgroups of five and
// more wavefronts, 415 to 500 of them: short ones run in the place that is left (`side_by_side`), unless the long ones decide, of many turns or
// far longer than the others (eight matrices of 2048 in SQ in fp16, turns of six, the longest 2.9 times the average, at 8 16.4 -> 13.5).
// Held, 169 such calls take 0.65 to 1.22 of the time left to itself; by the line 0.98 of held and 0.96 of left to itself in the mean, fp16 up
// to 14 % and bf16 up to 11 % from the better of the two.
constexpr int stage_most(bool multi, int R, bool mixed) { return !mixed ? 8 : multi && R == 2 ? 3 : !multi && R <= 3 ? 5 : 8; }
template <int MATS> struct StageArgs {
    static constexpr bool kGrid2D = MATS <= kGrid2DMaxMats;
    int wg_end[kGrid2D ? 1 : MATS];
    DecodeMat m[MATS];
    int M, xdt, ydt, S, waves, pad;
};
template <int R, bool MULTI, class Args, int MOST>
__global__ void __launch_bounds__(64 * stage_waves(MULTI, R)) __attribute__((amdgpu_waves_per_eu(stage_waves(MULTI, R) / 4, MOST)))
decode_stage_kernel(Args a) {
    extern __shared__ __attribute__((aligned(1024))) uint32_t stage_lds[];        // per wavefront: two codebook slots, later its R sums
    __shared__ __attribute__((aligned(16))) float xsc[16][16];
    int mi = 0, group;
    if constexpr (Args::kGrid2D) {
        mi = blockIdx.y;
        group = blockIdx.x;
    } else {
        const int wg = blockIdx.x;
#pragma unroll
        for (int j = 0; j < kMaxGroupMats; j += 64)
            mi += __builtin_popcountll(__builtin_amdgcn_ballot_w64(wg >= a.wg_end[j + (threadIdx.x & 63)]));
        group = wg - (mi ? a.wg_end[mi - 1] : 0);
    }
    const int M = a.M, xdt = a.xdt, ydt = a.ydt, S = a.S, waves = a.waves;   // the end of the argument block: asked for with the descriptor
    const DecodeMat mt = a.m[mi];
    asm volatile("" :: "s"(M), "s"(xdt), "s"(ydt), "s"(S), "s"(waves), "s"(mt.N));
    const int R0 = R * group;
    if (Args::kGrid2D && 16 * R0 >= mt.N) return;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int KT = mt.K >> 8;
    constexpr int kOwn = R > 2 ? 256 * R : 512;                    // words of LDS per wavefront
    uint32_t* mine = stage_lds + kOwn * wave;
    bool infinite = false;                                         // (bf16: see scaled_row_tile)
    float4_t out[R];
#pragma unroll
    for (int rt = 0; rt < R; ++rt) out[rt] = float4_t{0, 0, 0, 0};
    if (wave < KT && wave < S) {
        const int nt = (KT - wave + S - 1) / S;
        if (xdt == DT_BF16) {
            // (asked where it can be: behind all formats it costs the loads of the others, two layers of d = 5120 in 6-bit VQ at M = 6 73 -> 78 us)
            if (mt.fmt == FMT_SQ3) {
                StageTiles<FMT_SQ3, R, MULTI, true>(mt, R0, M, lane, xsc[wave], mine).run(wave, S, nt, out);
                infinite = any_infinite(out);
            } else if (mt.fmt == FMT_VQ6) {
                if constexpr (R == 2 && !MULTI) {
                    if (KT == 3 || KT == 4) StageTiles<FMT_VQ6, R, MULTI, true, false>(mt, R0, M, lane, xsc[wave], mine).run(wave, S, nt, out);
                    else { StageTiles<FMT_VQ6, R, MULTI, true>(mt, R0, M, lane, xsc[wave], mine).run(wave, S, nt, out); infinite = any_infinite(out); }
                } else {
                    StageTiles<FMT_VQ6, R, MULTI, true>(mt, R0, M, lane, xsc[wave], mine).run(wave, S, nt, out);
                    if (stage_as_is(FMT_VQ6, R)) infinite = any_infinite(out);
                }
            } else {
                StageTiles<FMT_VQ8, R, MULTI, true>(mt, R0, M, lane, xsc[wave], mine).run(wave, S, nt, out);
                if (stage_as_is(FMT_VQ8, R)) infinite = any_infinite(out);
            }
        } else {
            if (mt.fmt == FMT_SQ3) StageTiles<FMT_SQ3, R, MULTI, false>(mt, R0, M, lane, xsc[wave], mine).run(wave, S, nt, out);
            else if (mt.fmt == FMT_VQ6) StageTiles<FMT_VQ6, R, MULTI, false>(mt, R0, M, lane, xsc[wave], mine).run(wave, S, nt, out);
            else StageTiles<FMT_VQ8, R, MULTI, false>(mt, R0, M, lane, xsc[wave], mine).run(wave, S, nt, out);
        }
    }
    wave_lds_sync();                                               // (the codebook slots are read)
    if (wave < S) {
#pragma unroll
        for (int rt = 0; rt < R; ++rt) *(float4_t*)(mine + 256 * rt + 4 * lane) = out[rt];
    }
    if (__builtin_expect(infinite, 0)) {
        const int NR = mt.N >> 4;
#pragma unroll 1
        for (int rt = 0; rt < R; ++rt) {
            float4_t* const sum = (float4_t*)(mine + 256 * rt + 4 * lane);
            *sum = if_infinite(*sum, scaled_row_tile(mt, R0 + rt < NR ? R0 + rt : NR - 1, 0, M, wave, S, lane));
        }
    }
    __syncthreads();
    // D layout of the MFMA: lane (n, mg) holds batch rows 4 mg .. 4 mg + 3 of output column n
    const float* sums = (const float*)stage_lds;
    for (int i = threadIdx.x; i < 16 * R * M; i += 64 * waves) {
        const int m = i / (16 * R), n = i - 16 * R * m;
        const int at = 256 * (n >> 4) + 4 * (16 * (m >> 2) + (n & 15)) + (m & 3);
        float t = sums[at];
        for (int s = 1; s < S; ++s) t += sums[kOwn * s + at];
        if (16 * R0 + n < mt.N) store_from_f32(mt.y, (size_t)m * mt.N + 16 * R0 + n, ydt, t);
    }
}

// The same for 17 .. 48 rows of x (G = 2, 3 groups of sixteen), eight wavefronts of 256 registers.  The activations of a column tile
// would take all of them, so a tile goes in its two units of 128 columns: while the R row tiles are multiplied by the fragments of
// one, those of the next are in flight.  XB (bf16 activations, as they are): SQ only.  VQ would need two operands per weight and the
// registers for them, and is left to the kernels of midbatch.hip.  Without the conversion to fp16 that bf16 took before (us): {k', r'} of
// the 7B shapes SQ at M = 17 16.8 -> 14.0, at 32 19.7 -> 16.9, and 48 rows fit: 18432 x 4096 at 33 26.4 -> 19.4, at 48 27.7 -> 21.9.
template <int FMT, int R, int G, bool XB>
struct StageWide {
    static_assert(FMT == FMT_SQ3 || !XB, "one operand per weight");
    static constexpr int kWords = FMT == FMT_VQ8 ? 512 : 384;
    const DecodeMat& mt;
    int R0, NR, KT, lane, block0, more_blocks;
    uint32_t xoff[G];
    uint32_t* cb_lds;                  // [2][256]: codebooks of the first and of the last row tile's block
    uint32_t mask, magic, m6, base0;
    StageRegs w[R];                    // (a codebook in the first two only: R row tiles lie in at most two blocks)
    uint4_t xf[2][G][4];

    __device__ __forceinline__ StageWide(const DecodeMat& mt_, int R0_, int M, int lane_, uint32_t* cb_)
        : mt(mt_), R0(R0_), NR(mt_.N >> 4), KT(mt_.K >> 8), lane(lane_), cb_lds(cb_) {
#pragma unroll
        for (int g = 0; g < G; ++g) xoff[g] = (uint32_t)((16 * g + (lane & 15) < M ? 16 * g + (lane & 15) : M - 1) * mt.K + 8 * (lane >> 4));
        sq_code_constants<XB>(mask, magic);
        asm("v_mov_b32 %0, 0xfc" : "=v"(m6));
        block0 = R0 >> 4;
        more_blocks = ((R0 + R - 1 < NR ? R0 + R - 1 : NR - 1) >> 4) - block0;
        base0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint32_t*)cb_lds;
    }
    template <int U>
    __device__ __forceinline__ void load_x(int T, bool live) {
        const uint16_t* p = (const uint16_t*)mt.x + 256 * T + 128 * U;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const uint32_t at = live ? xoff[g] : 0u;
#pragma unroll
            for (int t = 0; t < 4; ++t) xf[U][g][t] = *(const uint4_t*)(p + at + 32 * t);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    __device__ __forceinline__ void load_w(StageRegs& r, int T, int rt, bool live) {
        const int row = R0 + rt < NR ? R0 + rt : NR - 1;
        const uint32_t l = live ? (uint32_t)lane : 0u;
        const uint32_t* t = mt.codes + ((size_t)row * KT + T) * kWords;
        r.a = stream_load((const uint4_t*)t + l);
        if constexpr (FMT == FMT_VQ8) {
            r.b = stream_load((const uint4_t*)(t + 256) + l);
            if (rt < 2) r.cb = ((const uint4_t*)mt.aux + ((size_t)(block0 + (rt ? more_blocks : 0)) * KT + T) * 64)[l];
        } else {
            const uint2_t two = stream_load((const uint2_t*)(t + 256) + l);
            r.b.x = two.x; r.b.y = two.y;
            if constexpr (FMT == FMT_SQ3) {
                const uint2_t sz = stream_load((const uint2_t*)mt.aux + ((size_t)row * KT + T) * 16 + (l & 15u));
                r.b.z = sz.x; r.b.w = sz.y;
            } else if (rt < 2) {
                r.b.z = ((const uint32_t*)mt.aux + ((size_t)(block0 + (rt ? more_blocks : 0)) * KT + T) * 64)[l];
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    // Columns 128 U .. of tile T for every row tile; the next tile's fragments of this unit follow, and behind the second unit
    // every row tile's next weights.
    template <int U>
    __device__ __forceinline__ void unit(int T, int Tn, bool more, float4_t (&out)[R][G]) {
        if (FMT != FMT_SQ3 && U == 0) {
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) {
                if constexpr (FMT == FMT_VQ8) *(uint4_t*)(cb_lds + 256 * rt + 4 * lane) = w[rt].cb;
                else cb_lds[256 * rt + lane] = w[rt].b.z;
            }
        }
        if (FMT != FMT_SQ3) wave_lds_sync();
        float4_t X[G];
        if constexpr (FMT == FMT_SQ3) {
            const uint4_t ones = {kSqOne<XB>, kSqOne<XB>, kSqOne<XB>, kSqOne<XB>};
#pragma unroll
            for (int g = 0; g < G; ++g) {
                X[g] = float4_t{0, 0, 0, 0};
#pragma unroll
                for (int t = 0; t < 4; ++t) X[g] = mfma_bits<XB>(xf[U][g][t], ones, X[g]);
            }
        }
#pragma unroll
        for (int rt = 0; rt < R; ++rt) {
            const StageRegs& r = w[rt];
            uint4_t op[4];
            const uint32_t slot = (R0 + rt) >> 4 != block0 ? (uint32_t)more_blocks : 0u;
            if constexpr (FMT == FMT_VQ8) {
                const uint4_t q = U == 0 ? r.a : r.b;
                const uint32_t* cbuf = cb_lds + 256 * slot;
                op[0] = __builtin_bit_cast(uint4_t, vq8_operand(q.x, cbuf)); op[1] = __builtin_bit_cast(uint4_t, vq8_operand(q.y, cbuf));
                op[2] = __builtin_bit_cast(uint4_t, vq8_operand(q.z, cbuf)); op[3] = __builtin_bit_cast(uint4_t, vq8_operand(q.w, cbuf));
            } else {
                const uint32_t w0 = U == 0 ? r.a.x : r.a.w, w1 = U == 0 ? r.a.y : r.b.x, w2 = U == 0 ? r.a.z : r.b.y;
                if constexpr (FMT == FMT_SQ3) {
                    op[0] = sq_operand<XB, 0>(w0, w1, w2, mask, magic); op[1] = sq_operand<XB, 1>(w0, w1, w2, mask, magic);
                    op[2] = sq_operand<XB, 2>(w0, w1, w2, mask, magic); op[3] = sq_operand<XB, 3>(w0, w1, w2, mask, magic);
                } else {
                    const uint32_t base = base0 + 1024 * slot;
                    op[0] = vq6_gather4<0>(w0, w1, w2, m6, base);
                    op[1] = vq6_gather4<1>(w0, w1, w2, m6, base);
                    op[2] = vq6_gather4<2>(w0, w1, w2, m6, base);
                    op[3] = vq6_gather4<3>(w0, w1, w2, m6, base);
                }
            }
            const uint32_t szw = U == 0 ? r.b.z : r.b.w;                      // (SQ)
            const float s = f16_bits_to_f32((uint16_t)(szw & 0xFFFFu)), z8 = f16_bits_to_f32((uint16_t)(szw >> 16)) + 8.0f;
#pragma unroll
            for (int g = 0; g < G; ++g) {
                float4_t sum = {0, 0, 0, 0};
                if (FMT != FMT_SQ3) sum = out[rt][g];
#pragma unroll
                for (int t = 0; t < 4; ++t) sum = mfma_bits<XB>(xf[U][g][t], op[t], sum);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if constexpr (FMT == FMT_SQ3) out[rt][g][i] = fmaf(s, fmaf(-z8, X[g][i], sum[i]), out[rt][g][i]);
                    else out[rt][g][i] = sum[i];
                }
            }
            if (U == 1) load_w(w[rt], Tn, rt, more);
            // (operands of one or two row tiles at a time: more would spill)
            else if (XB || (FMT != FMT_SQ3 && R == 6 && (rt & 1))) __builtin_amdgcn_sched_barrier(0);
        }
        load_x<U>(Tn, more);
    }
    __device__ __forceinline__ void run(int t0, int S, int nt, float4_t (&out)[R][G]) {
        const int last = t0 + (nt - 1) * S;
        __builtin_amdgcn_sched_barrier(0);
        load_x<0>(t0, true);
#pragma unroll
        for (int rt = 0; rt < R; ++rt) load_w(w[rt], t0, rt, true);
        load_x<1>(t0, true);
#pragma unroll 1
        for (int T = t0; T <= last; T += S) {
            const bool more = T + S <= last;
            unit<0>(T, more ? T + S : last, more, out);
            unit<1>(T, more ? T + S : last, more, out);
        }
    }
};

constexpr int kWideWaves = 8;
template <int R, int G, bool XB>
__global__ void __launch_bounds__(64 * kWideWaves) decode_stage_wide_kernel(StageArgs<kGrid2DMaxMats> a) {
    extern __shared__ __attribute__((aligned(1024))) uint32_t stage_lds[];        // per wavefront: R codebook slots, later its sums
    const int M = a.M, ydt = a.ydt, S = a.S;
    const DecodeMat mt = a.m[blockIdx.y];
    asm volatile("" :: "s"(M), "s"(ydt), "s"(S), "s"(mt.N));
    const int R0 = R * blockIdx.x;
    if (16 * R0 >= mt.N) return;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int KT = mt.K >> 8;
    constexpr int kOwn = 256 * R * G;                              // words of LDS per wavefront
    uint32_t* mine = stage_lds + kOwn * wave;
    float4_t out[R][G];
#pragma unroll
    for (int rt = 0; rt < R; ++rt)
#pragma unroll
        for (int g = 0; g < G; ++g) out[rt][g] = float4_t{0, 0, 0, 0};
    if (wave < KT) {
        const int nt = (KT - wave + S - 1) / S;
        if (XB || mt.fmt == FMT_SQ3) StageWide<FMT_SQ3, R, G, XB>(mt, R0, M, lane, mine).run(wave, S, nt, out);
        else if (mt.fmt == FMT_VQ6) StageWide<FMT_VQ6, R, G, false>(mt, R0, M, lane, mine).run(wave, S, nt, out);
        else StageWide<FMT_VQ8, R, G, false>(mt, R0, M, lane, mine).run(wave, S, nt, out);
    }
    wave_lds_sync();
#pragma unroll
    for (int rt = 0; rt < R; ++rt)
#pragma unroll
        for (int g = 0; g < G; ++g) *(float4_t*)(mine + 256 * (G * rt + g) + 4 * lane) = out[rt][g];
    if constexpr (XB)
        if (__builtin_expect(any_infinite(reinterpret_cast<float4_t (&)[R * G]>(out)), 0)) {   // (see scaled_row_tile)
            const int NR = mt.N >> 4;
#pragma unroll 1
            for (int at = 0; at < R * G; ++at) {
                float4_t* const sum = (float4_t*)(mine + 256 * at + 4 * lane);
                const int row_tile = R0 + at / G;
                *sum = if_infinite(*sum, scaled_row_tile(mt, row_tile < NR ? row_tile : NR - 1, 16 * (at % G), M, wave, S, lane));
            }
        }
    __syncthreads();
    const float* sums = (const float*)stage_lds;
    for (int i = threadIdx.x; i < 16 * R * M; i += 64 * S) {
        const int m = i / (16 * R), n = i - 16 * R * m;
        const int at = 256 * (G * (n >> 4) + (m >> 4)) + 4 * (16 * ((m & 15) >> 2) + (n & 15)) + (m & 3);
        float t = sums[at];
        for (int s = 1; s < S; ++s) t += sums[kOwn * s + at];
        if (16 * R0 + n < mt.N) store_from_f32(mt.y, (size_t)m * mt.N + 16 * R0 + n, ydt, t);
    }
}

// Time mixing's r, k, v and the wkv step in one launch.  The recurrence is per channel, and channel c
// needs r[c], k[c], v[c]: output row c of three matrices.  A workgroup of 12 wavefronts takes row tile R
// of all three (four wavefronts per matrix, the column tiles dealt as in the split-K kernel with S = 4,
// the same order of summation), and the 16 lanes that hold the tile's sums step the recurrence for
// channels 16 R .. 16 R + 15 and store sigma(r) wkv, the vector W_o multiplies: no launch and no pass
// over memory between the projections and the recurrence, and every channel's state is touched by
// exactly one lane.  Arithmetic and bits as rwkvq_linear_dispatch on the three matrices followed by
// rwkvq_wkv (the projections are rounded to the output type before they enter the recurrence, as
// they would be read back).
struct WkvFuseArgs {
    DecodeMat m[3];
    const float* w; const float* u; float* state; void* out;
    int d, xdt, ydt, pad;
};
__global__ void __launch_bounds__(768) decode_rkv_wkv_kernel(WkvFuseArgs a) {
    constexpr int DEPTH = RWKVQ_DECODE_DEPTH, S = 4;
    __shared__ __attribute__((aligned(1024))) uint32_t cb_all[3 * S][256];
    __shared__ float red[3 * S][16];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int mi = wave >> 2, s = wave & 3;
    const DecodeMat mt = mi == 0 ? a.m[0] : mi == 1 ? a.m[1] : a.m[2];
    const int xdt = a.xdt;
    // the descriptor, the types and the recurrence's pointers sit in four cache lines of the argument block: all asked
    // for before the first wait (one after the other each is a trip of its own at the start of a kernel that lasts 8 us)
    asm volatile("" :: "s"(mt.codes), "s"(mt.K), "s"(xdt), "s"(a.state), "s"(a.d));
    const int KT = mt.K >> 8;
    WavePos wp;
    wp.R[0] = wp.R[1] = wp.R[2] = wp.R[3] = blockIdx.x;
    wp.M = 1; wp.lane = lane; wp.tid = threadIdx.x; wp.xbf16 = xdt == DT_BF16;
    wp.t0 = s; wp.ts = S; wp.nt = s < KT ? (KT - s + S - 1) / S : 0;
    wp.xprev = nullptr; wp.mix_idx = nullptr; wp.mix_cb = nullptr;
    // the recurrence's operands for this tile's channels: fetched now, used after the GEMV
    const size_t c = (size_t)16 * blockIdx.x + (lane & 15);
    float sa = 0.f, sb = 0.f, sp = 0.f, wc = 0.f, uc = 0.f;
    if (wave == 0 && lane < 16) {
        sa = a.state[c]; sb = a.state[(size_t)a.d + c]; sp = a.state[2 * (size_t)a.d + c];
        wc = a.w[c]; uc = a.u[c];
    }
    float part[kRT] = {0.f};
    if (wp.nt > 0) {
        run_m1<DEPTH, true, false>(mt, wp, cb_all[wave], part);
    }
    float v = part[0];                             // sum the four column groups of each row
    v += __shfl_xor(v, 16, 64);
    v += __shfl_xor(v, 32, 64);
    if (lane < 16) red[wave][lane] = v;
    __syncthreads();
    if (wave == 0 && lane < 16) {
        float y[3];
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            float t = red[S * m][lane];
#pragma unroll
            for (int j = 1; j < S; ++j) t += red[S * m + j][lane];
            store_from_f32(m == 0 ? a.m[0].y : m == 1 ? a.m[1].y : a.m[2].y, c, a.ydt, t);
            y[m] = a.ydt == DT_F16 ? f16_bits_to_f32(f32_to_f16_bits(t)) : bf16_bits_to_f32(f32_to_bf16_bits(t));
        }
        store_from_f32(a.out, c, a.ydt, gate_f32(y[0], wkv_out(sa, sb, sp, uc, y[1], y[2])));
        wkv_advance(sa, sb, sp, wc, y[1], y[2]);
        a.state[c] = sa; a.state[(size_t)a.d + c] = sb; a.state[2 * (size_t)a.d + c] = sp;
    }
}

hipError_t launch_decode_rkv_wkv(const MatDev* rkv, const WkvDev& wkv, int x_dtype, int y_dtype, hipStream_t s) {
    WkvFuseArgs a;
    for (int i = 0; i < 3; ++i)
        a.m[i] = DecodeMat{rkv[i].codes, rkv[i].aux, rkv[i].x, rkv[i].y, rkv[i].N, rkv[i].K, rkv[i].fmt, POST_NONE, nullptr};
    a.w = wkv.w; a.u = wkv.u; a.state = wkv.state; a.out = wkv.out;
    a.d = rkv[0].N; a.xdt = x_dtype; a.ydt = y_dtype; a.pad = 0;
    hipLaunchKernelGGL(decode_rkv_wkv_kernel, dim3(rkv[0].N / 16), dim3(768), 0, s, a);
    return hipGetLastError();
}

// Smallest S of 4, 8, 16 that brings `tiles` row tiles to kSplitTarget wavefronts.
static int pick_split(int tiles) { return tiles * 4 >= kSplitTarget ? 4 : tiles * 8 >= kSplitTarget ? 8 : 16; }

// n_mats <= kGrid2DMaxMats: grid (longest matrix's row tiles, matrices); else one row of `wgs` workgroups and the table.  The tables of
// eight and of 256 matrices are for one of the two each (launch_decode).
template <class Args>
static hipError_t launch_splitk(int split, int wgs, Args& a, int n_mats, hipStream_t s) {
    a.pad = 0;
    if constexpr (Args::kMats < kMaxGroupMats)
        if (Args::kMats == kGrid2DMaxMats || (n_mats <= kGrid2DMaxMats && option(RWKVQ_OPT_SPLIT_GRID_2D) == 1)) {
            int longest = 0;
            for (int i = 0; i < n_mats; ++i) longest = std::max(longest, a.wg_end[i] - (i ? a.wg_end[i - 1] : 0));
            const dim3 grid(longest, n_mats);
            if (split == 4) hipLaunchKernelGGL((decode_splitk_kernel<4, Args, true>), grid, dim3(256), 0, s, a);
            else if (split == 8) hipLaunchKernelGGL((decode_splitk_kernel<8, Args, true>), grid, dim3(512), 0, s, a);
            else hipLaunchKernelGGL((decode_splitk_kernel<16, Args, true>), grid, dim3(1024), 0, s, a);
            return hipGetLastError();
        }
    if constexpr (Args::kMats > kGrid2DMaxMats) {
        const dim3 grid(wgs);
        if (split == 4) hipLaunchKernelGGL((decode_splitk_kernel<4, Args, false>), grid, dim3(256), 0, s, a);
        else if (split == 8) hipLaunchKernelGGL((decode_splitk_kernel<8, Args, false>), grid, dim3(512), 0, s, a);
        else hipLaunchKernelGGL((decode_splitk_kernel<16, Args, false>), grid, dim3(1024), 0, s, a);
        return hipGetLastError();
    }
    return hipErrorInvalidValue;
}

// Batch 1 with the token-shift mix fused into the activation load: always the split-K kernel
// (these are the stages of a block; 64 matrices per launch).
hipError_t launch_decode_mixed(const MatDev* mats, const MixDev* mixes, int n_mats, int x_dtype, int y_dtype,
                               hipStream_t s, const PostDev* posts) {
    for (int base = 0; base < n_mats; base += kMaxMixedMats) {
        MixedDecodeArgs a;
        const int cnt = n_mats - base < kMaxMixedMats ? n_mats - base : kMaxMixedMats;
        int tiles = 0;
        for (int i = 0; i < cnt; ++i) tiles += (mats[base + i].N + 15) / 16;
        int wgs = 0;
        for (int i = 0; i < kMaxMixedMats; ++i) {
            if (i < cnt) {
                const MatDev& m = mats[base + i];
                const MixDev& x = mixes[base + i];
                wgs += (m.N + 15) / 16;
                MixedMat mm;
                mm.codes = m.codes; mm.aux = m.aux; mm.x = m.x; mm.y = m.y; mm.N = m.N; mm.K = m.K; mm.fmt = m.fmt;
                mm.post = posts ? posts[base + i].op : POST_NONE; mm.gate = posts ? posts[base + i].gate : nullptr;
                mm.xprev = (const uint16_t*)x.x_prev; mm.mix_idx = x.idx; mm.mix_cb = (const uint32_t*)x.cb; mm.mix_E = x.E; mm.pad2 = 0;
                a.m[i] = mm;
                a.wg_end[i] = wgs;
            } else {
                a.m[i] = MixedMat{};
                a.wg_end[i] = 0x7FFFFFFF;
            }
        }
        a.M = 1; a.xdt = x_dtype; a.ydt = y_dtype; a.pad = 0;
        hipError_t e = launch_splitk(pick_split(tiles), wgs, a, cnt, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Batch 1 with the outputs also leaving as the mixes of the next stage: the split-K kernel (these are
// single projections of a block).
hipError_t launch_decode_postmix(const MatDev* mats, const PostDev* posts, const PostMixDev* pm, int n_mats,
                                 int x_dtype, int y_dtype, hipStream_t s) {
    for (int base = 0; base < n_mats; base += kMaxMixedMats) {
        PostMixArgs a;
        const int cnt = n_mats - base < kMaxMixedMats ? n_mats - base : kMaxMixedMats;
        int tiles = 0;
        for (int i = 0; i < cnt; ++i) tiles += (mats[base + i].N + 15) / 16;
        int wgs = 0;
        for (int i = 0; i < kMaxMixedMats; ++i) {
            PostMixMat mm{};
            if (i < cnt) {
                const MatDev& m = mats[base + i];
                const PostMixDev& x = pm[base + i];
                wgs += (m.N + 15) / 16;
                mm.codes = m.codes; mm.aux = m.aux; mm.x = m.x; mm.y = m.y; mm.N = m.N; mm.K = m.K; mm.fmt = m.fmt;
                mm.post = posts[base + i].op; mm.gate = posts[base + i].gate;
                mm.xprev = x.x_prev; mm.n_mix = x.n_mix; mm.pad2 = 0;
                for (int p = 0; p < 4; ++p)
                    mm.mix[p] = p < x.n_mix ? PostMix{x.idx[p], (const uint32_t*)x.cb[p], x.out[p]} : PostMix{nullptr, nullptr, nullptr};
                a.wg_end[i] = wgs;
            } else {
                a.wg_end[i] = 0x7FFFFFFF;
            }
            a.m[i] = mm;
        }
        a.M = 1; a.xdt = x_dtype; a.ydt = y_dtype; a.pad = 0;
        hipError_t e = launch_splitk(pick_split(tiles), wgs, a, cnt, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <int R, bool MULTI, bool MIXED, class Args>
static hipError_t launch_stage_kernel(const Args& a, dim3 grid, hipStream_t s) {
    constexpr int MOST = stage_most(MULTI, R, MIXED);
    const int lds = a.S * (R > 2 ? R : 2) * 1024;
    if (lds > 60 * 1024) {
        static std::atomic<unsigned long long> raised{0ull};
        const hipError_t e = raise_lds((const void*)decode_stage_kernel<R, MULTI, Args, MOST>, 16 * R * 1024, raised);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((decode_stage_kernel<R, MULTI, Args, MOST>), grid, dim3(64 * a.waves), lds, s, a);
    return hipGetLastError();
}
// Launches of more matrices than the two-dimensional grid takes (the table) know one, two and four row tiles per workgroup.
constexpr int stage_rows(bool grid2d, int r) { return grid2d ? r : r == 3 ? 4 : r > 4 ? 0 : r; }
enum StageKind { STAGE_SHORT, STAGE_ROUND, STAGE_MIXED, STAGE_ROUNDS, STAGE_MIXED_ROUNDS };
struct StageShape {
    int R, S, turns, waves;            // row tiles of a workgroup; wavefronts that split the columns, tiles that one takes; wavefronts in all
    StageKind kind;
    int columns;                       // of the longest row
    double row_tiles;
    double spread;                     // the longest row over the average one: beyond 1.6 rows of mixed lengths
};
// Row tiles R and wavefronts S of a workgroup, swept over R = 1 .. 6 and S = 3 .. 16 at M = 2 to 16 in every format and both types of
// x (us: fp16 where no type is named, cold weights).  `spread` is the longest row over the average one.
//   * rows of at most 512 columns: a workgroup is over so soon that small ones, several to a compute unit, are best: 14336 x 256 SQ at
//     M = 8 4.3 with R = 4 and a workgroup per compute unit, 3.6 with R = 1; 24 of 2048 x 512 6.0 with R = 4, 7.6 with R = 1;
//   * one round: the fewest row tiles that make at most 256 workgroups, each with a compute unit to itself and, up to sixteen, a
//     wavefront per column tile: every byte is asked for at the start ({r, k, v, g} of the 7B shapes in SQ at M = 16 9.9, in four
//     wavefronts 11.2; {k', r'} 11.1 and 12.9).  17 to 19 columns in turns of at most eight wavefronts, of twelve from three row tiles on and with two in
//     bf16.  Longer rows: fp16, and SQ in bf16, by fewer as M grows, whose lines of x the others evict (4096 x 14336 SQ at M = 8 in fp16 14.0
//     by eight, 13.3 by six, in bf16 14.0 and 13.2; at M = 16 in bf16 18.6 by eight, 18.0 by five); bf16 with VQ, whose conversion or second
//     operands every wavefront repeats, by eight or twelve, a multiple of the SIMDs (5120 x 17920 6-bit VQ at M = 2 19.6 by seven, 17.5 by
//     twelve), twelve where a tile of x is short, or with one row tile by ten up to M = 8 and by six beyond (4096 x 14336 6-bit VQ at M = 2
//     11.9 by twelve, 11.7 by ten; at M = 16 19.8 by eight, 18.2 by six).  In fp16 on 690 calls within 1.1 % of the best S in the mean.  With
//     up to two row tiles that is for calls of more than eight matrices and for those that staged_cheaper leaves here;
//   * one round, mixed lengths: a workgroup of the longest rows would end long after the others: two row tiles instead of three to
//     six, or one (a layer of d = 2048 in 8-bit VQ at M = 2 20.2 with R = 6, now 13.4; {8192 x 256, 256 x 8192} in SQ at M = 8 12.2 and 9.4);
//   * several rounds, of one length or of mixed ones: small workgroups overlap ({k', r', v'} of the 14B-class shapes in 8-bit VQ at M = 4
//     46.0 with R = 4, now 29.1; a 7B layer 38.6 and 31.9).
// A wavefront takes R M / 4 steps for the sums at the end by itself: four at least take part, eight in one round of R >= 3.
static StageShape stage_shape(const MatDev* mats, const int* order, int n_mats, int M, int x_dtype) {
    const bool grid2d = n_mats <= kGrid2DMaxMats;
    int columns = 0, fits = 0;
    bool vq = false;
    double row_tiles = 0.0, tiles = 0.0, vq8 = 0.0;
    for (int i = 0; i < n_mats; ++i) {
        const MatDev& m = mats[order[i]];
        columns = std::max(columns, m.K >> 8);
        row_tiles += m.N >> 4; tiles += (double)(m.N >> 4) * (m.K >> 8);
        vq = vq || m.fmt != FMT_SQ3;
        if (m.fmt == FMT_VQ8) vq8 += m.N >> 4;
    }
    for (int r = 1; r <= 6 && !fits; ++r) {
        if (stage_rows(grid2d, r) != r) continue;
        long long n = 0;
        for (int i = 0; i < n_mats; ++i) n += (mats[order[i]].N + 16 * r - 1) / (16 * r);
        if (n <= 256) fits = r;
    }
    const double spread = columns * row_tiles / tiles;
    StageShape p;
    p.columns = columns; p.row_tiles = row_tiles; p.spread = spread;
    int most;
    if (columns <= 2) {
        p.kind = STAGE_SHORT;
        p.R = row_tiles <= 1024.0 ? 1 : row_tiles <= 2560.0 ? 2 : 4; most = 2;
    } else if (fits && (spread <= 1.6 || fits <= (columns <= 16 ? 3 : 2))) {
        p.kind = STAGE_ROUND;
        p.R = fits; most = columns <= 16 ? 16 : fits == 1 || (fits == 2 && x_dtype != DT_BF16) ? 8 : 12;
    } else if (fits) {
        p.kind = STAGE_MIXED;
        p.R = spread > 8.0 ? 1 : 2; most = columns <= 16 ? 16 : row_tiles <= 1000.0 ? 8 : 4;
    } else if (spread <= 1.6) {
        p.kind = STAGE_ROUNDS;
        p.R = row_tiles <= 1600.0 ? 2 : 4; most = columns <= 8 ? 8 : 4;
    } else {
        p.kind = STAGE_MIXED_ROUNDS;
        p.R = row_tiles <= 2200.0 || (!grid2d && row_tiles <= 2700.0 && 2.0 * vq8 > row_tiles) ? 2 : grid2d ? 3 : 4;
        most = spread > 8.0 ? 6 : 4;
    }
    p.turns = (columns + most - 1) / most;
    p.S = (columns + p.turns - 1) / p.turns;
    if (p.kind == STAGE_ROUND && columns >= 20) {
        if (x_dtype == DT_BF16 && vq) p.S = fits == 1 ? (M <= 8 ? 10 : 6) : M <= 8 && columns > 20 ? 12 : 8;
        else p.S = fits == 6 || ((fits == 2 || fits == 3) && M <= 4) ? 8 : M <= 12 || fits == 1 ? 6 : 5;
        p.turns = (columns + p.S - 1) / p.S;
    }
    p.waves = std::max(p.S, fits >= 3 && p.R == fits ? 8 : 4);
    return p;
}

// Batch 2..16: is the column split (decode_stage_kernel) the faster of the two?  Measured on 8248 launches of 1 to 256 matrices, K = 256
// to 17920, up to 21504 row tiles, M = 2 to 16, every format, both types of x (us: columns / rows).  In a launch of one round it always is
// (4672 of them; 4096 x 4096 SQ at M = 8 5.5 / 14.7, 1024 x 1024 3.1 / 5.6).  Beyond, decode_kernel fills the device too, and its
// workgroups share what they read of x:
//   * rows of at most 512 columns: up to 4200 row tiles, 1536 beyond M = 8, where the end of a workgroup weighs more (256 of 256 x 512 SQ
//     at M = 4 5.2 / 5.9, at 16 7.5 / 6.2): 15 of 2024 take a kernel that is more than 4 % slower, the worst 11 %;
//   * several rounds of one length: up to 3200 row tiles, and M = 12 up to 2048 columns (24 of 2048 x 1024 SQ at M = 8 7.4 / 8.8), M = 4
//     beyond (44 of 512 x 2560: SQ at M = 8 11.8 / 10.7, 8-bit VQ at 2 11.8 / 12.8): 94 of 816, the worst 23 %;
//   * several rounds of mixed lengths (whole layers): an estimate of both durations: 15 of 736, the worst 14 %.
// RWKVQ_OPT_STREAM_SPLIT_MAX_WORK moves the lines in proportion (1: never split, 1000000: always, and always by this kernel).
static bool stage_cheaper(const MatDev* mats, const int* order, int n_mats, int M, int x_dtype, const StageShape& p) {
    const int max_work = option(RWKVQ_OPT_STREAM_SPLIT_MAX_WORK);
    if (max_work <= 1 || max_work >= 1000000) return max_work > 1;
    const double by = (double)max_work / kStreamSplitMaxWork;
    // (stacks: every workgroup's own read of x grows with them)
    if (p.row_tiles * (16 + M) > 4.0 * kStreamSplitMaxWork * by) return false;
    switch (p.kind) {
        case STAGE_ROUND: case STAGE_MIXED: return true;
        case STAGE_SHORT: return p.row_tiles <= (M <= 8 ? 4200.0 : 1536.0) * by;
        case STAGE_ROUNDS: return p.row_tiles <= 3200.0 * by && M <= (p.columns <= 8 ? 12 : 4);
        default: break;
    }
    const bool bf16 = x_dtype == DT_BF16;
    double rows = 0.0, chain = 0.0, split = 0.0;
    for (int i = 0; i < n_mats; ++i) {
        const MatDev& m = mats[order[i]];
        const double tiles = 1e-3 * (m.N >> 4) * (m.K >> 8);
        const int f = m.fmt == FMT_SQ3 ? 0 : m.fmt == FMT_VQ6 ? 1 : 2;
        static const double kSplit[3] = {0.269, 0.269, 0.342}, kRows[3] = {0.257, 0.270, 0.378}, kChain[3] = {0.69, 0.80, 0.91};
        split += tiles * (kSplit[f] + 0.0062 * M + (bf16 ? 0.0525 : 0.0));
        rows += tiles * kRows[f];
        chain = std::max(chain, (m.K >> 8) * (kChain[f] + (bf16 ? 0.25 : 0.0)));
    }
    split += 4.46 + 0.195 * M + (0.73 + 0.002 * M) * 1e-3 * p.row_tiles + 0.072 * p.columns + (bf16 ? 0.76 : 0.0);
    rows = rows * (1.0 + 0.016 * M) * (bf16 ? 1.053 : 1.0) + 0.318e-3 * p.row_tiles;
    return split <= (3.0 + 0.021 * M + std::pow(std::pow(rows, 2.3) + std::pow(chain, 2.3), 1.0 / 2.3)) * by;
}

// A launch of one round with up to two row tiles per workgroup: the kernel of midbatch.hip that copies activations into LDS by itself, 64
// columns in four steps ahead, instead of decode_stage_kernel, whose wavefronts have one or two column tiles of operands in flight?
// It starts later (a launch of 4096 x 1024 takes 5 to 25 % longer) and wins as rows get longer and x wider.  Measured (us, there -> here)
// on 120 matrices' shapes and formats at eight values of M, fp16 and bf16: 4096 x 14336 SQ at M = 2 11.5 -> 10.7, at 8 13.3 -> 11.5, at 16 18.3 ->
// 13.3, 6-bit VQ in fp16 at 8 13.4 -> 11.8, at 16 17.9 -> 13.4, in bf16 at 4 12.5 -> 13.5, at 8 14.4 -> 13.7; 2048 x 5120 SQ at 16 9.0 -> 5.4;
// 4096 x 4096 SQ at 8 5.5 -> 5.5, at 16 6.7 -> 5.9, 8-bit VQ at 16 7.1 -> 7.4; two row tiles: 5120 x 17920 SQ at 4 16.8 -> 16.6, at 16 24.0
// -> 19.1, 8-bit VQ in fp16 at 12 21.6 -> 21.1; 8192 x 4096 at 16 4 to 11 % longer.  Nine columns are a second turn here for one of eight
// K groups: 4096 x 2304 SQ at 10 4.4 -> 4.6, at 12 even, 6-bit VQ at 14 4.8 -> 5.1, in bf16 5.2 -> 5.6.  Of 4290 calls (N = 512 to 8192, nine to
// 70 columns, M = 2 to 16, both types of x) that come here none is more than 4 % slower; what stays there up to M = 6 with more than 28 columns
// of VQ would be faster here in fp16 (512 x 14336 6-bit at 6 11.8 -> 10.0), not in bf16.
// RWKVQ_OPT_STREAM_SPLIT_MAX_WORK = 1000000 never comes here.
static bool staged_cheaper(const MatDev* mats, const int* order, int n_mats, int M, const StageShape& p) {
    if (p.kind != STAGE_ROUND || p.R > 2 || n_mats > kGrid2DMaxMats || option(RWKVQ_OPT_STREAM_SPLIT_MAX_WORK) >= 1000000) return false;
    int f = FMT_SQ3;
    for (int i = 0; i < n_mats; ++i) f = std::max(f, mats[order[i]].fmt);
    if (p.R == 2) return p.columns > 16 && M >= (f == FMT_SQ3 ? 6 : f == FMT_VQ6 ? 14 : 15);
    if (p.columns > 16) return f == FMT_SQ3 || p.columns <= 28 || M > 6;
    return p.columns == 9 ? f == FMT_SQ3 && M >= 12 : p.columns > 9 && f != FMT_VQ8 && M >= (f == FMT_SQ3 ? 10 : 14);
}

template <int MATS>
static hipError_t launch_stage(const MatDev* mats, const int* order, int n_mats, int M, int x_dtype, int y_dtype, const StageShape& p, hipStream_t s) {
    StageArgs<MATS> a;
    int wgs = 0, longest = 0;
    for (int i = 0; i < MATS; ++i) {
        a.m[i] = DecodeMat{nullptr, nullptr, nullptr, nullptr, 0, 0, 0, POST_NONE, nullptr};
        if (i < n_mats) {
            const MatDev& m = mats[order[i]];
            const int n = (m.N + 16 * p.R - 1) / (16 * p.R);
            a.m[i] = DecodeMat{m.codes, m.aux, m.x, m.y, m.N, m.K, m.fmt, POST_NONE, nullptr};
            wgs += n; longest = std::max(longest, n);
        }
        if constexpr (!StageArgs<MATS>::kGrid2D) a.wg_end[i] = i < n_mats ? wgs : 0x7FFFFFFF;
    }
    a.M = M; a.xdt = x_dtype; a.ydt = y_dtype; a.S = p.S; a.waves = p.waves; a.pad = 0;
    const dim3 grid = StageArgs<MATS>::kGrid2D ? dim3(longest, n_mats) : dim3(wgs);
    const int on_simd = (p.waves + 3) / 4;                          // wavefronts of a workgroup
    const bool bf16 = x_dtype == DT_BF16;
    const bool side_by_side = bf16 ? p.spread <= 2.6 || p.turns <= 3 : p.turns <= 3 ? p.spread <= 2.4 : p.turns <= 5 && p.spread <= 2.0;
    const bool few = p.spread > 1.6 && (p.turns <= 1 ? (wgs + 255) / 256 * on_simd <= 4
                                        : on_simd == 1 ? wgs <= (bf16 ? 768 : 1100) : wgs <= 410 || !side_by_side);
#define RWKVQ_STAGE(R_) case R_: if constexpr (stage_rows(StageArgs<MATS>::kGrid2D, R_) == R_) \
        return p.turns <= 1 ? (few ? launch_stage_kernel<R_, false, true>(a, grid, s) : launch_stage_kernel<R_, false, false>(a, grid, s)) \
                            : (few ? launch_stage_kernel<R_, true, true>(a, grid, s) : launch_stage_kernel<R_, true, false>(a, grid, s)); break;
    switch (p.R) {
        RWKVQ_STAGE(1) RWKVQ_STAGE(2) RWKVQ_STAGE(3) RWKVQ_STAGE(4) RWKVQ_STAGE(5) RWKVQ_STAGE(6)
    }
#undef RWKVQ_STAGE
    return hipErrorInvalidValue;
}

template <int R, int G, bool XB>
static hipError_t launch_wide_kernel(const StageArgs<kGrid2DMaxMats>& a, dim3 grid, hipStream_t s) {
    static std::atomic<unsigned long long> raised{0ull};
    const hipError_t e = raise_lds((const void*)decode_stage_wide_kernel<R, G, XB>, kWideWaves * R * G * 1024, raised);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((decode_stage_wide_kernel<R, G, XB>), grid, dim3(64 * a.S), a.S * R * G * 1024, s, a);
    return hipGetLastError();
}
// Row tiles of a workgroup (5 or 6; 0: the kernels of midbatch.hip) at 17 <= M <= 48.  Those take 64 rows of W in a workgroup that has
// a compute unit to itself; from 257 of them on they need a second round, which one round of 80 or 96 rows saves.  Smaller calls stay
// there: every workgroup reads all of x (4096 x 4096 at M = 32 10.9 us here, 9.3 there; 4096 x 14336 29.7 and 21.3).
// What the round costs beside its columns grows with M and the row tiles (16 R M sums of up to eight partial ones through LDS), so rows
// of few columns stay there as M grows.  RWKVQ_OPT_STREAM_SPLIT_MAX_WORK = 1000000 takes every call that fits.
// Measured (us, there -> here) at K = 256 to 7168, N = 16640 to 24576, M = 17 to 48 in every format: the calls that the line below lets
// through take 0.55 to 1.02 of the time there.  16640 x 256 SQ at M = 24 9.4 -> 9.7, at 48 10.9 -> 15.4 (not taken); {k', r'} of the 7B
// shapes fp16 SQ at M = 17 23.5 -> 15.2, 32 24.9 -> 17.3, 48 27.9 -> 22.0; of 14B-class shapes (six row tiles) fp16 SQ at 32
// 29.3 -> 23.0, 6-bit VQ 28.4 -> 22.7; bf16 SQ 18432 x 2048 at 33 18.5 -> 13.7, at 48 19.3 -> 15.5.
// The round ends with its longest rows, there shorter ones of a second round run beside them: beyond 32 rows of x, where a column costs
// most, an estimate of both (us, here / there, at M = 48: {14336 x 4096, 4096 x K} SQ 22 / 27 at K = 4096, 29 / 27 at 6144, 54 / 36 at
// 14336; {9216 x 2048, 9216 x K} 16 / 19 at 2048, 22 / 19 at 4096; at 33 24 / 27 and 19 / 19 in the second of each).  Of 216 calls of
// 24 kinds at 33, 40 and 48 rows none takes a kernel that is more than 4 % slower.
static int wide_row_tiles(const MatDev* mats, int n_mats, int M, int x_dtype) {
    const bool bf16 = x_dtype == DT_BF16;
    if (n_mats > kGrid2DMaxMats || M <= 16 || M > 48) return 0;
    double row_tiles = 0.0, tiles = 0.0;
    LaunchLoad there;
    for (int i = 0; i < n_mats; ++i) {
        if (bf16 && mats[i].fmt != FMT_SQ3) return 0;              // (see StageWide)
        there.add((mats[i].N + 63) / 64, mats[i].K);
        row_tiles += mats[i].N / 16;
        tiles += (double)(mats[i].N / 16) * (mats[i].K / 256);
    }
    auto workgroups = [&](int r) { long long n = 0; for (int i = 0; i < n_mats; ++i) n += (mats[i].N + 16 * r - 1) / (16 * r); return n; };
    const int R = workgroups(4) <= 256 ? 0 : workgroups(5) <= 256 ? 5 : M <= 32 && workgroups(6) <= 256 ? 6 : 0;
    if (R == 0 || option(RWKVQ_OPT_STREAM_SPLIT_MAX_WORK) >= 1000000) return R;
    const double columns = tiles / row_tiles;                      // of the average row
    const double most = R == 6 ? 12.0 + 5.0 * columns : 16.0 + 8.0 * columns;
    if (M > 32 && 7.0 + 0.0667 * M + (0.268 + 0.0107 * M) * there.longest > 11.0 + 0.47 * there.columns(0.5)) return 0;
    return M <= most ? R : 0;
}
bool wide_cheaper(const MatDev* mats, int n_mats, int M, int x_dtype) { return wide_row_tiles(mats, n_mats, M, x_dtype) > 0; }
hipError_t launch_wide(const MatDev* mats, int n_mats, int M, int x_dtype, int y_dtype, hipStream_t s) {
    StageArgs<kGrid2DMaxMats> a;
    const int R = wide_row_tiles(mats, n_mats, M, x_dtype);
    int columns = 0, longest = 0;
    for (int i = 0; i < kGrid2DMaxMats; ++i) {
        a.m[i] = DecodeMat{nullptr, nullptr, nullptr, nullptr, 0, 0, 0, POST_NONE, nullptr};
        if (i >= n_mats) continue;
        const MatDev& m = mats[i];
        a.m[i] = DecodeMat{m.codes, m.aux, m.x, m.y, m.N, m.K, m.fmt, POST_NONE, nullptr};
        columns = std::max(columns, m.K >> 8); longest = std::max(longest, (m.N + 16 * R - 1) / (16 * R));
    }
    const int turns = (columns + kWideWaves - 1) / kWideWaves;
    a.M = M; a.xdt = x_dtype; a.ydt = y_dtype; a.S = (columns + turns - 1) / turns;
    const dim3 grid(longest, n_mats);
    const bool bf16 = x_dtype == DT_BF16;
    if (M > 32) return bf16 ? launch_wide_kernel<5, 3, true>(a, grid, s) : launch_wide_kernel<5, 3, false>(a, grid, s);
    if (R == 5) return bf16 ? launch_wide_kernel<5, 2, true>(a, grid, s) : launch_wide_kernel<5, 2, false>(a, grid, s);
    return bf16 ? launch_wide_kernel<6, 2, true>(a, grid, s) : launch_wide_kernel<6, 2, false>(a, grid, s);
}

hipError_t launch_decode(const MatDev* mats, int n_mats, int M, int x_dtype, int y_dtype, hipStream_t s,
                         const PostDev* posts) {
    for (int base = 0; base < n_mats; base += kMaxGroupMats) {
        int cnt = n_mats - base < kMaxGroupMats ? n_mats - base : kMaxGroupMats;
        // Workgroups are handed out in index order and a workgroup's running time grows with K:
        // the matrices of a launch go longest rows first, so that the launch does not end on a
        // few long workgroups (the outputs are independent, the order is free).
        int order[kMaxGroupMats];
        for (int i = 0; i < cnt; ++i) order[i] = base + i;
        std::stable_sort(order, order + cnt, [&](int p, int q) { return mats[p].K > mats[q].K; });
        // Batch 1 with fewer row tiles than two per SIMD: split the columns over S wavefronts of a
        // workgroup (one workgroup per row tile), S the smallest of 4, 8, 16 that reaches that count
        // (measured on the stages of a 7B block: 2048 beats 1024 and 4096 by 3-8 %, 16384 loses 40 %).
        int tiles = 0;
        for (int i = 0; i < cnt; ++i) tiles += (mats[order[i]].N + 15) / 16;
        int split = 0;
        if (M == 1 && tiles < kSplitTarget) split = pick_split(tiles);
        auto fill = [&](auto& a, auto rows_of) {               // the matrices in order; workgroups of rows_of rows
            int wgs = 0;
            for (int i = 0; i < cnt; ++i) {
                const MatDev& m = mats[order[i]];
                wgs += (m.N + rows_of - 1) / rows_of;
                a.m[i] = DecodeMat{m.codes, m.aux, m.x, m.y, m.N, m.K, m.fmt, posts ? posts[order[i]].op : POST_NONE,
                                   posts ? posts[order[i]].gate : nullptr};
                a.wg_end[i] = wgs;
            }
            for (int i = cnt; i < a.kMats; ++i) {
                a.m[i] = DecodeMat{nullptr, nullptr, nullptr, nullptr, 0, 0, 0, POST_NONE, nullptr};
                a.wg_end[i] = 0x7FFFFFFF;
            }
            a.M = M; a.xdt = x_dtype; a.ydt = y_dtype; a.pad = 0;
            return wgs;
        };
        if (split && cnt <= kGrid2DMaxMats && option(RWKVQ_OPT_SPLIT_GRID_2D) == 1) {
            SmallDecodeArgs a;
            const int wgs = fill(a, 16);
            const hipError_t e = launch_splitk(split, wgs, a, cnt, s);
            if (e != hipSuccess) return e;
            continue;
        }
        // batch 2..16 with few rows in the launch: the wavefronts of a workgroup split the columns
        if (M > 1 && M <= 16) {
            const StageShape p = stage_shape(mats, order, cnt, M, x_dtype);
            if (stage_cheaper(mats, order, cnt, M, x_dtype, p)) {
                const hipError_t e = staged_cheaper(mats, order, cnt, M, p) ? launch_mid(mats + base, cnt, M, x_dtype, y_dtype, true, s)
                                   : cnt <= kGrid2DMaxMats ? launch_stage<kGrid2DMaxMats>(mats, order, cnt, M, x_dtype, y_dtype, p, s)
                                                           : launch_stage<kMaxGroupMats>(mats, order, cnt, M, x_dtype, y_dtype, p, s);
                if (e != hipSuccess) return e;
                continue;
            }
        }
        // batch > 1: two row passes per workgroup if the launch keeps enough workgroups that way
        int passes = 1;
        if (M > 1) {
            long long wgs2 = 0;
            for (int i = 0; i < cnt; ++i) wgs2 += (mats[order[i]].N + wg_rows(M, 2) - 1) / wg_rows(M, 2);
            if (kTwoPassFits && wgs2 >= option(RWKVQ_OPT_STREAM_TWO_PASS_MIN_WGS)) passes = 2;
        }
        DecodeArgs a;
        const int wgs = fill(a, split ? 16 : wg_rows(M, passes));
        const dim3 grid(wgs), wide(64 * kBW);
        if (split) { hipError_t e = launch_splitk(split, wgs, a, cnt, s); if (e != hipSuccess) return e; }
        else if (M == 1) hipLaunchKernelGGL(decode_kernel<1>, grid, dim3(256), 0, s, a);
        else if (M <= 4 && passes == 1) hipLaunchKernelGGL((decode_kernel<4, 1>), grid, wide, 0, s, a);
        else if (M <= 4) hipLaunchKernelGGL((decode_kernel<4, 2>), grid, wide, 0, s, a);
        else if (M <= 16 && passes == 1) hipLaunchKernelGGL((decode_kernel<16, 1>), grid, wide, 0, s, a);
        else if (M <= 16) hipLaunchKernelGGL((decode_kernel<16, 2>), grid, wide, 0, s, a);
        else if (passes == 1) hipLaunchKernelGGL((decode_kernel<32, 1>), grid, wide, 0, s, a);
        else hipLaunchKernelGGL((decode_kernel<32, 2>), grid, wide, 0, s, a);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace rwkvq

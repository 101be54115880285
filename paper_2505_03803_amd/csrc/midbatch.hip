// Matrix-core path for 17 to about a thousand rows of x (prompts, chunks of them; EXACT: also 2 to 16 in small launches of long
// rows): y[M][N] = x[M][K] * Deq(W)^T with the feed of prefill.hip (Deq(W) rounded once to the type of x, binary32 accumulate)
// in another cut.  prefill.hip gives a workgroup 128 or 256 rows of x and 256 of W and all of K; with a few hundred rows of x a
// projection is then 16 to 48 workgroups on 256 compute units, each a chain of K / 64 steps.  Here
//   * a workgroup of eight wavefronts takes 16 MF rows of x (MF = 4, 6, 8) and 16 NF NW rows of W (NF = 4; NW = 1, 2): a 4096 x
//     4096 matrix at 333 rows is 192 workgroups (MF = 4, NW = 2);
//   * the wavefronts split K as well: KW = 8 / NW groups take the 256-column tiles kg, kg + KW, ..., so the chain is KW times
//     shorter; their partial sums meet in LDS at the end, in group order;
//   * W never goes through LDS: a lane's packed words hold exactly its operand of v_mfma_f32_16x16x32 (native layout), so
//     the wavefront that multiplies a row tile unpacks it in registers, one half step ahead, a share behind every row of MFMAs;
//   * activations: copied global -> LDS by the load unit (chunk ^ (row & 7) swizzle as in prefill.hip) into a ring per
//     K group, 2 to 4 tiles of 64 columns, shared by the group's NW wavefronts; one barrier per step (none for NW = 1);
//   * formats share a launch (prefill.hip: one launch per format).
// What bounds it: a wavefront's own chain.  Two wavefronts on a SIMD (registers, LDS) issue unpack, fragment reads and MFMAs in
// order and wait 28 to 42 % of the time; no unit is full (counters at 333 rows: matrix cores 37 to 42 % busy, vector ALU a third
// of the rate that two wavefronts sustain, LDS 15 to 50 %).  The unpack costs the same for 64 rows of x as for 128: a step of
// MF = 4 takes 1.2 us, of MF = 8 1.5 us, of which the MFMAs are 0.45 and 0.9.
// Measured (bf16, SQ and 6-bit VQ, us; prefill.hip -> here): 4096 x 4096 at M = 333 82 -> 27.5, at M = 1024 82 -> 40.5;
// 4096 x 14336 at M = 333 265 -> 78, at M = 1024 269 -> 120; four 4096 x 4096 at M = 333 170 -> 66, at M = 1024 178 -> 140.
// EXACT instances (17 <= M <= 128, and launches of long rows from M = 2 on, where the streaming kernels' contract holds: weights
// unrounded, fp16 or bf16 x multiplied as it is): NW = 1, 16 to 64 rows of x per workgroup, so a call that took ceil(M / 32) passes
// over W takes one (M <= 64).  SQ: codes as 8 + q with the scale and zero point applied to the group's sums; VQ: the fp16 entries,
// for bf16 x as the sum of two bf16.
// A workgroup takes 32 rows of W (NF = 2) where that gives at most one per compute unit, and 64 otherwise; 16 (NF = 1) where 32 would
// leave half of the compute units without one: each then multiplies half as many rows by the x that it reads either way (36 bytes per
// clock and compute unit, what bounds long rows beyond 32 rows of x).  Of 336 calls of one matrix of 1024 to 4096 rows none got more than
// 1 % slower; us, 32 rows -> 16: 4096 x 4096 fp16 SQ at M = 17 8.5 -> 7.6, at 48 10.1 -> 9.0, at 64 12.3 -> 11.5; 4096 x 14336 6-bit VQ at 17
// 19.4 -> 16.9, at 48 26.3 -> 25.8; 1024 x 14336 SQ at 128 31.7 -> 29.2; 2048 x 2048 8-bit VQ at 48 6.8 -> 5.8.
// Measured (fp16, us; streaming kernels -> here): {r, k, v, g} of 4096 x 4096 at M = 32 21.3 -> 12.6, 48 34.8 -> 15.4, 64
// 41 -> 17.6, 128 83 -> 31; bf16, 8-bit VQ: 4096 x 4096 at M = 17 10.1 -> 8.4 (64 rows: 11.7), 4096 x 14336 at 17 26.1 -> 18.2
// (27.6), at 64 75 -> 26 (35); SQ: 61 -> 20 at 48 (28); {r, k, v, g} are 512 workgroups of 32 rows and slower in them (SQ, M = 48
// 16.0, 64 rows 12.9).
// Tried and slower or equal: wavefronts of 32 instead of 64 rows of W with sixteen per workgroup (the fragment reads from
// LDS double: - 8 % at M = 64, + 20 % at M = 1024), fragment reads three and four rows ahead (equal), an MFMA / vector
// instruction interleave fixed with scheduling groups (equal at MF = 4, spills at MF = 8).
#include "matrix_core.h"
#include "mid_tiles.h"
#include "../../include/rwkvq.h"

#include <algorithm>
#include <type_traits>

namespace rwkvq {

constexpr int kMidWaves = 8;
constexpr int kMidBook = 1024;                 // bytes of a converted 8-bit-index codebook
constexpr int kMidMaxMats = 64;

struct MidMat {
    const uint32_t* codes;
    const uint16_t* aux;
    const void* x;
    void* y;
    int N, K, fmt, pad;
};
struct MidArgs {
    int wg_end[kMidMaxMats];
    MidMat m[kMidMaxMats];
    int M, ydt, m_tiles, pad;
};

// Per kernel instance: activation tiles in the ring of a K group, register sets of packed words (two: the next tile's words
// are asked for a whole tile ahead; MF = 8 has no registers for that and asks half a step ahead), bytes of LDS.
constexpr int mid_sets(int MF, bool EXACT) { return MF <= (EXACT ? 3 : 6) ? 2 : 1; }
constexpr int mid_stage(int MF) { return 16 * MF * kRowBytes; }
constexpr int mid_book(bool EXACT) { return EXACT ? 2 * kMidBook : kMidBook; }       // EXACT, bf16: two words per entry
constexpr int mid_stages(int MF, int NW, bool EXACT) { return std::min(4, (EXACT ? 128 : 144) * 1024 / (kMidWaves / NW * mid_stage(MF))); }
constexpr int mid_ring(int MF, int NW, bool EXACT) { return kMidWaves / NW * mid_stages(MF, NW, EXACT) * mid_stage(MF); }
constexpr int mid_red() { return kMidWaves * 4 * 4 * 1024; }           // partial sums of four subtile rows of every wavefront
constexpr int mid_lds(int MF, int NW, bool EXACT) {
    return std::max(mid_ring(MF, NW, EXACT) + kMidWaves * mid_sets(MF, EXACT) * mid_book(EXACT), mid_red());
}

// Buffer loads: a descriptor and the moving offset in scalar registers, one 32-bit offset per lane (global loads came out
// as 64-bit lane addresses, an addition and two registers each).  The hardware's check against `bytes` leaves the scalar offset
// out, so every offset below lies inside the matrix by itself.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t mid_buffer(const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, (int)bytes, 0x00020000);
}
// All but the newest N vector-memory operations and all LDS operations have finished (gfx9 encoding).
template <int N>
__device__ __forceinline__ void mid_wait() {
    static_assert(N >= 0 && N < 64, "six bits");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0070);
}
// Packed words of one 256-column tile for the wavefront's row tiles.
template <int FMT, int NF> struct MidRegs;
template <int NF> struct MidRegs<FMT_SQ3, NF> { uint4_t a[NF]; uint2_t b[NF]; uint2_t sz[NF]; };   // sz: (scale, zero) x 2 units
template <int NF> struct MidRegs<FMT_VQ6, NF> { uint4_t a[NF]; uint2_t b[NF]; uint32_t cb; };
template <int NF> struct MidRegs<FMT_VQ8, NF> { uint4_t a[NF]; uint4_t b[NF]; uint4_t cb8; };

// SQ pair P of a unit.  The definition rounds q - z and then the product with s (sq_pair_deq).  q s and z s are exact in
// binary32 (3 and 11 bits times 11 bits), so q s - z s with one rounding is the same value whenever q - z is exact, which
// it is for z = 0 and |z| >= 2^-11 (the bits of q - z then span at most 24 places): one multiply-add per weight instead of
// a multiply-add and a multiplication (- 10 % of the kernel's time).  ROUND: a group of the tile has a smaller zero point.
template <bool BF16, bool ROUND, int P>
__device__ __forceinline__ uint32_t mid_sq_pair(uint32_t w0, uint32_t w1, uint32_t w2, float s, float z) {
    if constexpr (ROUND) {
        float lo, hi;
        sq_pair_deq<P>(w0, w1, w2, s, z, lo, hi);
        if constexpr (!BF16) {                 // as below
            uint32_t o;
            asm("v_cvt_pk_f16_f32 %0, %1, %2" : "=v"(o) : "v"(lo), "v"(hi));
            return o;
        }
        return Elem<BF16>::pack(lo, hi);
    } else {
        const half2_t h = __builtin_bit_cast(half2_t, sq_pair_mask<P>(w0, w1, w2));
        const float sc = s * sq_pair_unscale<P>(), zs = z * s;
        float lo = fmaf((float)h.x, sc, -zs), hi = fmaf((float)h.y, sc, -zs);
        // fp16: left to itself the compiler merges the multiply-add with the conversion into one instruction that rounds
        // once; the definition rounds to binary32 first
        if constexpr (!BF16) {
            uint32_t o;
            asm("v_cvt_pk_f16_f32 %0, %1, %2" : "=v"(o) : "v"(lo), "v"(hi));
            return o;
        }
        return Elem<BF16>::pack(lo, hi);
    }
}
// Does any group of the workgroup's rows of W have a zero point in (0, 2^-11) or (-2^-11, 0)?
// The scales and zero points (8 % of W's bytes) are read here once more than by the loop, each wavefront its eighth; a test
// per tile in the loop held both forms of the unpack in registers and spilled.
__device__ __forceinline__ bool mid_small_zero(const void* sz, int bytes, int tid, uint32_t* lds) {
    const __amdgpu_buffer_rsrc_t buf = mid_buffer(sz, (uint32_t)bytes);
    uint32_t least = 0xFFFFFFFFu;              // of |z| - 1 (fp16 bits, high half): a zero wraps to the top
    auto z = [](uint32_t v) { return (v & 0x7FFF0000u) - 0x00010000u; };
    for (int at = 16 * tid; at < bytes; at += 8 * 16 * 64 * kMidWaves) {
        uint4_t v[8];                          // eight loads in flight: a 4096-column workgroup's 16 KB need two
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = __builtin_amdgcn_raw_buffer_load_b128(buf, std::min(at + k * 16 * 64 * kMidWaves, bytes - 16), 0, 0);
#pragma unroll
        for (int k = 0; k < 8; ++k)
            least = min(min(least, min(z(v[k].x), z(v[k].y))), min(z(v[k].z), z(v[k].w)));
    }
    const bool any = __builtin_amdgcn_ballot_w64(least < 0x0FFF0000u) != 0;      // fp16 0x1000 = 2^-11
    if ((tid & 63) == 0) lds[tid >> 6] = any;
    __syncthreads();
    uint32_t all = 0;
#pragma unroll
    for (int w = 0; w < kMidWaves; ++w) all |= lds[w];
    __syncthreads();                           // the ring takes the place of the flags
    return __builtin_amdgcn_readfirstlane(all) != 0;
}

// EXACT (weights enter unrounded, as in the streaming kernels): pair p of step H as 8 + q
template <bool BF16, int H, int NF>
__device__ __forceinline__ uint32_t mid_code_pair(const MidRegs<FMT_SQ3, NF>& r, int i, int p, uint32_t mask, uint32_t magic) {
    constexpr int u = H >> 2, t = H & 3;
    const uint32_t w0 = u == 0 ? r.a[i].x : r.a[i].w, w1 = u == 0 ? r.a[i].y : r.b[i].x, w2 = u == 0 ? r.a[i].z : r.b[i].y;
    return p == 0 ? sq_pair_code<BF16, 4 * t>(w0, w1, w2, mask, magic) : p == 1 ? sq_pair_code<BF16, 4 * t + 1>(w0, w1, w2, mask, magic)
         : p == 2 ? sq_pair_code<BF16, 4 * t + 2>(w0, w1, w2, mask, magic) : sq_pair_code<BF16, 4 * t + 3>(w0, w1, w2, mask, magic);
}
// Index of weight pair p of step H, row tile i.
template <int FMT, int H, int NF>
__device__ __forceinline__ uint32_t mid_index(const MidRegs<FMT, NF>& r, int i, int p) {
    constexpr int u = H >> 2, t = H & 3;
    if constexpr (FMT == FMT_VQ8) {
        const uint4_t q = u == 0 ? r.a[i] : r.b[i];
        return ((t == 0 ? q.x : t == 1 ? q.y : t == 2 ? q.z : q.w) >> (8 * p)) & 255u;
    } else {
        const uint32_t w0 = u == 0 ? r.a[i].x : r.a[i].w, w1 = u == 0 ? r.a[i].y : r.b[i].x, w2 = u == 0 ? r.a[i].z : r.b[i].y;
        return (p == 0 ? vq6_byteaddr<4 * t>(w0, w1, w2) : p == 1 ? vq6_byteaddr<4 * t + 1>(w0, w1, w2)
              : p == 2 ? vq6_byteaddr<4 * t + 2>(w0, w1, w2) : vq6_byteaddr<4 * t + 3>(w0, w1, w2)) >> 2;
    }
}

// Weight pair p (0..3) of 32-column step H (0..7) of the 256-column tile, row tile i: two weights as they are multiplied.
template <bool BF16, int FMT, bool ROUND, int H, int NF>
__device__ __forceinline__ uint32_t mid_pair(const MidRegs<FMT, NF>& r, int i, int p, const uint32_t* book) {
    constexpr int u = H >> 2, t = H & 3;
    if constexpr (FMT == FMT_VQ8) {
        const uint4_t q = u == 0 ? r.a[i] : r.b[i];
        const uint32_t w = t == 0 ? q.x : t == 1 ? q.y : t == 2 ? q.z : q.w;
        return book[(w >> (8 * p)) & 255u];
    } else {
        const uint32_t w0 = u == 0 ? r.a[i].x : r.a[i].w, w1 = u == 0 ? r.a[i].y : r.b[i].x, w2 = u == 0 ? r.a[i].z : r.b[i].y;
        if constexpr (FMT == FMT_SQ3) {
            const uint32_t szw = u == 0 ? r.sz[i].x : r.sz[i].y;
            const float s = f16_bits_to_f32((uint16_t)(szw & 0xFFFFu)), z = f16_bits_to_f32((uint16_t)(szw >> 16));
            return p == 0 ? mid_sq_pair<BF16, ROUND, 4 * t>(w0, w1, w2, s, z) : p == 1 ? mid_sq_pair<BF16, ROUND, 4 * t + 1>(w0, w1, w2, s, z)
                 : p == 2 ? mid_sq_pair<BF16, ROUND, 4 * t + 2>(w0, w1, w2, s, z) : mid_sq_pair<BF16, ROUND, 4 * t + 3>(w0, w1, w2, s, z);
        } else {
            const uint32_t at = p == 0 ? vq6_byteaddr<4 * t>(w0, w1, w2) : p == 1 ? vq6_byteaddr<4 * t + 1>(w0, w1, w2)
                              : p == 2 ? vq6_byteaddr<4 * t + 2>(w0, w1, w2) : vq6_byteaddr<4 * t + 3>(w0, w1, w2);
            return *(const uint32_t*)((const char*)book + at);         // from LDS (ds_bpermute instead: + 15 % at MF = 8)
        }
    }
}
// Pairs n0 .. n1-1 of the 4 NF (row tile, pair) that a half step takes.
template <bool BF16, int FMT, bool ROUND, int H, int NF>
__device__ __forceinline__ void mid_pairs(uint32_t (&b)[NF][4], const MidRegs<FMT, NF>& r, int n0, int n1, const uint32_t* book) {
#pragma unroll
    for (int n = n0; n < n1; ++n) b[n >> 2][n & 3] = mid_pair<BF16, FMT, ROUND, H>(r, n >> 2, n & 3, book);
}

template <bool BF16, int FMT, bool ROUND, int MF, int NW, bool EXACT, int NF>
__device__ __forceinline__ void mid_loop(const MidArgs& a, const MidMat& mt, char* lds, int m0, int n0, int wave, int lane,
                                         float4_t (&acc)[MF][NF]) {
    constexpr int KW = kMidWaves / NW, ST = mid_stages(MF, NW, EXACT), SETS = mid_sets(MF, EXACT), AHEAD = ST - 1, kStage = mid_stage(MF);
    constexpr int tw = FMT == FMT_VQ8 ? 512 : 384, kBook = FMT == FMT_VQ8 ? 1024 : 256;
    constexpr bool SQ = FMT == FMT_SQ3;
    static_assert(ST >= 2 && ST <= 4, "one activation tile is copied while one is multiplied");
    const int nw = wave % NW, kg = wave / NW;
    const int K = mt.K, KT = K >> 8, R0 = (n0 >> 4) + NF * nw;
    const int nt = kg < KT ? (KT - kg + KW - 1) / KW : 0, rounds = (KT + KW - 1) / KW;   // column tiles of this group, of the longest
    char* const ring = lds + kg * ST * kStage;
    uint32_t* const books = (uint32_t*)(lds + mid_ring(MF, NW, EXACT)) + wave * (SETS * mid_book(EXACT) / 4);

    // the group's wavefronts copy its activation tile together: copy i of this one brings rows 8 (NW i + nw) .. + 7 (rows
    // past M repeat row M - 1)
    constexpr int kCopies = 2 * MF / NW;
    uint32_t xoff[kCopies];
#pragma unroll
    for (int i = 0; i < kCopies; ++i) {
        const int row = 8 * (NW * i + nw) + (lane >> 3), c = (lane & 7) ^ (row & 7);
        const int rr = m0 + row < a.M ? row : a.M - 1 - m0;
        xoff[i] = (uint32_t)rr * (uint32_t)K * 2u + 16u * c;
    }
    const char* const xrows = (const char*)mt.x + (size_t)m0 * K * 2;
    const uint32_t xbytes = (uint32_t)std::min(a.M - m0, 16 * MF) * (uint32_t)K * 2u;
    // EXACT: N is any multiple of 16; row tiles past the end repeat the last one and are not stored
    const int tiles = EXACT ? mid_row_tiles(mt.N, R0, NF) : NF;
    const uint32_t wbytes = (uint32_t)(tiles * KT * tw * 4), abytes = SQ ? (uint32_t)(tiles * KT * 128) : (uint32_t)(KT * kBook);
    const char* const words = (const char*)(mt.codes + (size_t)R0 * KT * tw);
    const char* const aux = SQ ? (const char*)mt.aux + (size_t)R0 * KT * 128 : (const char*)mt.aux + (size_t)(R0 >> 4) * KT * kBook;
    const int last = 4 * nt - 1;
    // Past the end of a group's sequence a load is still counted by the waits, but a buffer of no bytes makes it no request (the last
    // step's 48 KB of x and the last tile's words again, as before, were a ninth and a third of what 4096 columns ask for).
    auto copy = [&](int step, int stage) {     // step = 4 j + KQ of this group's sequence
        const __amdgpu_buffer_rsrc_t xbuf = mid_buffer(xrows, step <= last ? xbytes : 0u);
        step = step < last ? step : last;
        const int at = 512 * (kg + KW * (step >> 2)) + kRowBytes * (step & 3);
        char* dst = ring + stage * kStage;
#pragma unroll
        for (int i = 0; i < kCopies; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(xbuf, (__attribute__((address_space(3))) void*)(dst + (NW * i + nw) * 1024), 16,
                                                     xoff[i], at, 0, 0);
    };
    auto load = [&](MidRegs<FMT, NF>& r, int j) {
        const __amdgpu_buffer_rsrc_t wbuf = mid_buffer(words, j < nt ? wbytes : 0u), abuf = mid_buffer(aux, j < nt ? abytes : 0u);
        const int T = kg + KW * (j < nt ? j : nt - 1);
        const int at = 16 * lane;
#pragma unroll
        for (int i = 0; i < NF; ++i) {
            const int row_tile = EXACT ? mid_row_tile(i, tiles) : i;
            const int tile = mid_tile_offset(row_tile, T, KT, 4 * tw);
            r.a[i] = __builtin_amdgcn_raw_buffer_load_b128(wbuf, at, tile, 0);
            if constexpr (FMT == FMT_VQ8) r.b[i] = __builtin_amdgcn_raw_buffer_load_b128(wbuf, at + 1024, tile, 0);
            else r.b[i] = __builtin_amdgcn_raw_buffer_load_b64(wbuf, (at >> 1) + 1024, tile, 0);
            if constexpr (SQ) r.sz[i] = __builtin_amdgcn_raw_buffer_load_b64(abuf, 8 * (lane & 15), mid_tile_offset(row_tile, T, KT, 128), 0);
        }
        if constexpr (FMT == FMT_VQ6) r.cb = __builtin_amdgcn_raw_buffer_load_b32(abuf, at >> 2, T * kBook, 0);
        if constexpr (FMT == FMT_VQ8) r.cb8 = __builtin_amdgcn_raw_buffer_load_b128(abuf, at, T * kBook, 0);
    };
    auto keep = [](const MidRegs<FMT, NF>& r) {
#pragma unroll
        for (int i = 0; i < NF; ++i) {
            asm volatile("" :: "v"(r.a[i]), "v"(r.b[i]));
            if constexpr (SQ) asm volatile("" :: "v"(r.sz[i]));
        }
        if constexpr (FMT == FMT_VQ6) asm volatile("" :: "v"(r.cb));
        if constexpr (FMT == FMT_VQ8) asm volatile("" :: "v"(r.cb8));
    };
    constexpr int kLoads = SQ ? 3 * NF : 2 * NF + 1;
    constexpr bool SPLIT = EXACT && BF16 && !SQ;   // fp16 entries as the sum of two bf16 (8 + 3 of the 11 bits, exact), multiplied in turn
    auto stage_book = [&](const MidRegs<FMT, NF>& r, uint32_t* to) {   // VQ: the tile's codebook as it is multiplied
        if constexpr (FMT == FMT_VQ6) {
            if constexpr (SPLIT) *(uint2_t*)(to + 2 * lane) = vq_split(r.cb);
            else to[lane] = Elem<BF16>::from_f16x2(r.cb);
        }
        if constexpr (FMT == FMT_VQ8) {
            const uint32_t c[4] = {r.cb8.x, r.cb8.y, r.cb8.z, r.cb8.w};
            if constexpr (SPLIT) {
                const uint2_t e0 = vq_split(c[0]), e1 = vq_split(c[1]), e2 = vq_split(c[2]), e3 = vq_split(c[3]);
                *(uint4_t*)(to + 8 * lane) = uint4_t{e0.x, e0.y, e1.x, e1.y};
                *(uint4_t*)(to + 8 * lane + 4) = uint4_t{e2.x, e2.y, e3.x, e3.y};
            } else {
                *(uint4_t*)(to + 4 * lane) = uint4_t{Elem<BF16>::from_f16x2(c[0]), Elem<BF16>::from_f16x2(c[1]), Elem<BF16>::from_f16x2(c[2]), Elem<BF16>::from_f16x2(c[3])};
            }
        }
    };
    uint32_t mask, magic;                      // EXACT SQ: in registers (the and-or takes no literals)
    sq_code_constants<BF16>(mask, magic);

    const int row = lane & 15, q = lane >> 4;
    uint32_t b[2][NF][4], bl[SPLIT ? 2 : 1][NF][4];            // operands of the two halves (32 columns) of a step; SPLIT: low parts
    // pairs n0 .. n1 - 1 of step H into b[h]
    auto pairs = [&](auto step, int h, const MidRegs<FMT, NF>& r, int n0, int n1, const uint32_t* book) {
        constexpr int H = decltype(step)::value;
        if constexpr (EXACT && SQ) {
#pragma unroll
            for (int n = n0; n < n1; ++n) b[h][n >> 2][n & 3] = mid_code_pair<BF16, H>(r, n >> 2, n & 3, mask, magic);
        } else if constexpr (SPLIT) {
#pragma unroll
            for (int n = n0; n < n1; ++n) {
                const uint2_t e = *(const uint2_t*)(book + 2 * mid_index<FMT, H>(r, n >> 2, n & 3));
                b[h][n >> 2][n & 3] = e.x;
                bl[h][n >> 2][n & 3] = e.y;
            }
        } else {
            mid_pairs<BF16, FMT, ROUND, H>(b[h], r, n0, n1, book);
        }
    };
    float4_t part[EXACT && SQ ? MF : 1][NF], X[EXACT && SQ ? MF : 1];   // EXACT SQ: the group's products and activation sums
    MidRegs<FMT, NF> r0, r1;
    int stage = 0;                             // ring slot of the current step

    // Step KQ of tile j.  HEAD: wait for its activations, ask for those AHEAD steps on and, at the first step, for the next
    // tile's words.  BODY: the MFMAs, between them the operands of the half step that follows.
    auto head = [&](auto tag, int j) {
        constexpr int KQ = decltype(tag)::value;
        // asked for after this step's activations: the copies of AHEAD - 1 steps and, with two register sets, the words
        // that the first step of the tile asks for
        constexpr int kSince = (AHEAD - 1) * kCopies + (SETS == 2 && KQ >= 1 && KQ <= AHEAD ? kLoads : 0);
        mid_wait<kSince>();
        if constexpr (NW > 1) RWKVQ_BARRIER(); // the group's copies have landed and its reads of the slot below are over
        copy(4 * j + KQ + AHEAD, stage >= 1 ? stage - 1 : ST - 1);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (SETS == 2 && KQ == 0) { load(r1, j + 1); __builtin_amdgcn_sched_barrier(0); }
    };
    auto operand = [](const uint32_t (&v)[4]) { return uint4_t{v[0], v[1], v[2], v[3]}; };
    auto body = [&](auto tag, int j) {
        constexpr int KQ = decltype(tag)::value;
        const char* xt = ring + stage * kStage;
        stage = stage + 1 < ST ? stage + 1 : 0;
        const char* const p[2] = {xt + tile_off(row, q), xt + tile_off(row, 4 + q)};
        // the first operands of a tile: with two register sets they are made during the last half step of the tile before
        uint32_t* const book = books + (SETS == 2 ? (j & 1) * (mid_book(EXACT) / 4) : 0);
        uint32_t* const next = books + (SETS == 2 ? (~j & 1) * (mid_book(EXACT) / 4) : 0);
        if constexpr (SETS == 1 && KQ == 0) {
            stage_book(r0, book);
            pairs(std::integral_constant<int, 0>{}, 0, r0, 0, 4 * NF, book);
        }
        if constexpr (SETS == 2 && KQ == 3) stage_book(r1, next);
        uint32_t szu[NF];                  // EXACT SQ: the group's scale and zero point (one register set: reloaded below)
        if constexpr (EXACT && SQ) {
#pragma unroll
            for (int i = 0; i < NF; ++i) szu[i] = KQ < 2 ? r0.sz[i].x : r0.sz[i].y;
        }
        uint4_t af[2 * MF];                    // activation fragments, read two rows ahead of their MFMAs
#pragma unroll
        for (int f = 0; f < 2; ++f) af[f] = *(const uint4_t*)(p[f / MF] + 16 * (f % MF) * kRowBytes);
#pragma unroll
        for (int f = 0; f < 2 * MF; ++f) {
            const int h = f / MF, fm = f % MF;
            if (f + 2 < 2 * MF) af[f + 2] = *(const uint4_t*)(p[(f + 2) / MF] + 16 * ((f + 2) % MF) * kRowBytes);
            if constexpr (EXACT && SQ) {
                const bool first = KQ % 2 == 0 && h == 0;
                const float4_t zero = {0, 0, 0, 0};
#pragma unroll
                for (int i = 0; i < NF; ++i) part[fm][i] = mfma_bits<BF16>(af[f], operand(b[h][i]), first ? zero : part[fm][i]);
                const uint32_t one = kSqOne<BF16>;
                X[fm] = mfma_bits<BF16>(af[f], uint4_t{one, one, one, one}, first ? zero : X[fm]);
            } else if constexpr (EXACT) {      // x first: a lane holds one row of W and four rows of x, as its scale and zero point are laid out
#pragma unroll
                for (int i = 0; i < NF; ++i) acc[fm][i] = mfma_bits<BF16>(af[f], operand(b[h][i]), acc[fm][i]);
                if constexpr (SPLIT) {
#pragma unroll
                    for (int i = 0; i < NF; ++i) acc[fm][i] = mfma_bits<BF16>(af[f], operand(bl[h][i]), acc[fm][i]);
                }
            } else {
#pragma unroll
                for (int i = 0; i < NF; ++i) acc[fm][i] = mfma_bits<BF16>(operand(b[h][i]), af[f], acc[fm][i]);
            }
            const int n0 = 4 * NF * fm / MF, n1 = 4 * NF * (fm + 1) / MF;
            if (h == 0) pairs(std::integral_constant<int, 2 * KQ + 1>{}, 1, r0, n0, n1, book);
            else if constexpr (KQ < 3) pairs(std::integral_constant<int, 2 * KQ + 2>{}, 0, r0, n0, n1, book);
            else if constexpr (SETS == 2) pairs(std::integral_constant<int, 0>{}, 0, r1, n0, n1, next);
            if constexpr (EXACT && SQ) {       // the group is complete: into the output
                if (KQ % 2 == 1 && h == 1) {
#pragma unroll
                    for (int i = 0; i < NF; ++i) {
                        const float s = f16_bits_to_f32((uint16_t)(szu[i] & 0xFFFFu)), z8 = f16_bits_to_f32((uint16_t)(szu[i] >> 16)) + 8.0f;
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[fm][i][e] = fmaf(s, fmaf(-z8, X[fm][e], part[fm][i][e]), acc[fm][i][e]);
                    }
                }
            }
            if (SETS == 1 && KQ == 3 && f == MF - 1) load(r0, j + 1);   // the packed words are spent
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    if (nt > 0) {
        load(r0, 0);
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) copy(i, i);
        if constexpr (SETS == 2) {
            stage_book(r0, books);
            pairs(std::integral_constant<int, 0>{}, 0, r0, 0, 4 * NF, books);
        }
    }
    // The waits in head() count the loads of the next tile's words, those of the last tile (never used) too.  The compiler may
    // not take an iteration out of the loop and drop its unused loads, which would leave activations unwaited for: no peeling,
    // and every word loaded is named behind the loop's last step.
#pragma clang loop unroll(disable)
    for (int j = 0; j < nt; ++j) {             // nothing conditional inside: the compiler then counts the loads in flight exactly
        head(std::integral_constant<int, 0>{}, j);
        body(std::integral_constant<int, 0>{}, j);
        head(std::integral_constant<int, 1>{}, j);
        body(std::integral_constant<int, 1>{}, j);
        head(std::integral_constant<int, 2>{}, j);
        body(std::integral_constant<int, 2>{}, j);
        head(std::integral_constant<int, 3>{}, j);
        body(std::integral_constant<int, 3>{}, j);
        if constexpr (SETS == 2) { keep(r1); r0 = r1; }
    }
    if constexpr (NW > 1)
        for (int j = 4 * nt; j < 4 * rounds; ++j) RWKVQ_BARRIER();     // a group with fewer column tiles than the longest
    mid_wait<0>();                             // no copy may still land in LDS below
}

template <bool BF16, int MF, int NW, bool EXACT, int NF>
__global__ void __launch_bounds__(64 * kMidWaves, 2) mid_kernel(MidArgs a) {
    constexpr int KW = kMidWaves / NW;
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    const int wg = blockIdx.x;
    static_assert(kMidMaxMats == 64, "one table entry per lane");
    const int mi = __builtin_popcountll(__builtin_amdgcn_ballot_w64(wg >= a.wg_end[threadIdx.x & 63]));
    const MidMat mt = a.m[mi];
    const int local = wg - (mi ? a.wg_end[mi - 1] : 0);
    const int m0 = (local % a.m_tiles) * 16 * MF, n0 = (local / a.m_tiles) * (16 * NF * NW);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nw = wave % NW, kg = wave / NW;
    float4_t acc[MF][NF];
#pragma unroll
    for (int f = 0; f < MF; ++f)
#pragma unroll
        for (int i = 0; i < NF; ++i) acc[f][i] = float4_t{0, 0, 0, 0};
    if (mt.fmt == FMT_SQ3) {
        const int KT = mt.K >> 8;
        if (!EXACT && mid_small_zero((const uint2_t*)mt.aux + (size_t)(n0 >> 4) * KT * 16, NF * NW * KT * 128, threadIdx.x, (uint32_t*)lds))
            mid_loop<BF16, FMT_SQ3, true, MF, NW, EXACT, NF>(a, mt, lds, m0, n0, wave, lane, acc);
        else mid_loop<BF16, FMT_SQ3, false, MF, NW, EXACT, NF>(a, mt, lds, m0, n0, wave, lane, acc);
    } else if (mt.fmt == FMT_VQ6) {
        mid_loop<BF16, FMT_VQ6, false, MF, NW, EXACT, NF>(a, mt, lds, m0, n0, wave, lane, acc);
    } else {
        mid_loop<BF16, FMT_VQ8, false, MF, NW, EXACT, NF>(a, mt, lds, m0, n0, wave, lane, acc);
    }

    // The K groups' partial sums meet in LDS, four rows of subtiles at a time; each group adds up and stores one of the rows
    // (eight groups: half of one), in group order.  The W operand comes first in the MFMA, so a lane holds output row
    // m = lane % 16 and four consecutive columns 4 (lane / 16) .. + 3 of every subtile.
    constexpr int PR = 4, SH = KW / PR;
    static_assert(KW == 4 || KW == 8, "a row or half a row per group");
#pragma unroll
    for (int ps = 0; ps < (MF + PR - 1) / PR; ++ps) {
        __syncthreads();
#pragma unroll
        for (int f = 0; f < PR && PR * ps + f < MF; ++f)
#pragma unroll
            for (int i = 0; i < NF; ++i) *(float4_t*)(lds + ((wave * PR + f) * NF + i) * 1024 + 16 * lane) = acc[PR * ps + f][i];
        if constexpr (EXACT && BF16) {
            static_assert(!EXACT || MF <= PR, "one pass");
            if (__builtin_expect(any_infinite(reinterpret_cast<float4_t (&)[MF * NF]>(acc)), 0)) {      // (see scaled_row_tile)
                const int R0 = n0 >> 4, tiles = mid_row_tiles(mt.N, R0, NF);
#pragma unroll 1
                for (int at = 0; at < MF * NF; ++at) {
                    float4_t* const sum = (float4_t*)(lds + (wave * PR * NF + at) * 1024 + 16 * lane);
                    *sum = if_infinite(*sum, scaled_row_tile(mt, R0 + mid_row_tile(at % NF, tiles), m0 + 16 * (at / NF), a.M, kg, KW, lane));
                }
            }
        }
        __syncthreads();
        const int f = kg / SH, m = m0 + 16 * (PR * ps + f) + (EXACT ? 4 * (lane >> 4) : lane & 15);
        constexpr int OWN = NF / SH > 0 ? NF / SH : 1;             // (NF = 1: every second group has none)
        if (PR * ps + f < MF && m < a.M && OWN * (kg % SH) < NF) {
#pragma unroll
            for (int ii = 0; ii < OWN; ++ii) {
                const int i = ii + OWN * (kg % SH);
                float4_t v = *(const float4_t*)(lds + ((nw * PR + f) * NF + i) * 1024 + 16 * lane);
#pragma unroll
                for (int g = 1; g < KW; ++g) {
                    const float4_t o = *(const float4_t*)(lds + (((g * NW + nw) * PR + f) * NF + i) * 1024 + 16 * lane);
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] += o[e];
                }
                if constexpr (EXACT) {
                    const int n = n0 + 16 * NF * nw + 16 * i + (lane & 15);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (n < mt.N && m + e < a.M) store_from_f32(mt.y, (size_t)(m + e) * mt.N + n, a.ydt, v[e]);
                    continue;
                }
                const size_t o = (size_t)m * mt.N + n0 + 16 * NF * nw + 16 * i + 4 * (lane >> 4);
                if (a.ydt == DT_F32) {
                    *(float4_t*)((float*)mt.y + o) = v;
                } else {
                    uint2_t pk;
                    if (a.ydt == DT_BF16) { pk.x = Elem<true>::pack(v[0], v[1]); pk.y = Elem<true>::pack(v[2], v[3]); }
                    else { pk.x = Elem<false>::pack(v[0], v[1]); pk.y = Elem<false>::pack(v[2], v[3]); }
                    *(uint2_t*)((uint16_t*)mt.y + o) = pk;
                }
            }
        }
    }
}

template <bool BF16, int MF, int NW, bool EXACT, int NF>
static hipError_t launch_mid_t(const MidArgs& a, int wgs, hipStream_t s) {
    static std::atomic<unsigned long long> raised{0ull};
    const hipError_t e = raise_lds((const void*)mid_kernel<BF16, MF, NW, EXACT, NF>, mid_lds(MF, NW, EXACT), raised);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((mid_kernel<BF16, MF, NW, EXACT, NF>), dim3(wgs), dim3(64 * kMidWaves), mid_lds(MF, NW, EXACT), s, a);
    return hipGetLastError();
}
template <bool BF16>
static hipError_t launch_mid_shape(const MidArgs& a, int mf, int nw, int nf, bool exact, int wgs, hipStream_t s) {
    if (exact) {
        if (!mid_exact_instance(mf, nf)) return hipErrorInvalidValue;
        if (mf == 1) return nf == 1 ? launch_mid_t<BF16, 1, 1, true, 1>(a, wgs, s) : launch_mid_t<BF16, 1, 1, true, 2>(a, wgs, s);
        if (nf == 1) return mf == 2   ? launch_mid_t<BF16, 2, 1, true, 1>(a, wgs, s)
                            : mf == 3 ? launch_mid_t<BF16, 3, 1, true, 1>(a, wgs, s) : launch_mid_t<BF16, 4, 1, true, 1>(a, wgs, s);
        if (nf == 2) return mf == 2   ? launch_mid_t<BF16, 2, 1, true, 2>(a, wgs, s)
                            : mf == 3 ? launch_mid_t<BF16, 3, 1, true, 2>(a, wgs, s) : launch_mid_t<BF16, 4, 1, true, 2>(a, wgs, s);
        return mf == 2   ? launch_mid_t<BF16, 2, 1, true, 4>(a, wgs, s)
               : mf == 3 ? launch_mid_t<BF16, 3, 1, true, 4>(a, wgs, s) : launch_mid_t<BF16, 4, 1, true, 4>(a, wgs, s);
    }
    if (nw == 1) return launch_mid_t<BF16, 4, 1, false, 4>(a, wgs, s);
    if (mf == 4) return launch_mid_t<BF16, 4, 2, false, 4>(a, wgs, s);
    if (mf == 6) return launch_mid_t<BF16, 6, 2, false, 4>(a, wgs, s);
    return launch_mid_t<BF16, 8, 2, false, 4>(a, wgs, s);
}

// Rows of x and of W per workgroup for a launch over `rows` rows of W.  One workgroup runs per compute unit; a round of
// them takes about 36 + 8.6 MF (measured at M = 1024, per 56 tiles of 256 columns: 70, 82, 105 us for MF = 4, 6, 8), and the
// cheapest number of rounds wins.  Splitting K over four groups whatever MF keeps the order of the sums, so the choice
// changes no bits.  Up to 128 rows, where that order is not promised, launches that leave half of the compute units
// without a workgroup split K over eight groups (NW = 1): 4096 x 4096 at M = 64 23 -> 14 us, 4096 x 14336 65 -> 34.
static void pick_mid(int M, long long rows, int* mf, int* nw) {
    *nw = 2;
    double best = 1e30;
    for (int f : {4, 6, 8}) {
        const long long wgs = rows / 128 * ((M + 16 * f - 1) / (16 * f));
        const double t = (double)((wgs + 255) / 256) * (36.0 + 8.6 * f);
        if (t < best) { best = t; *mf = f; }
    }
    if (M <= 128 && rows / 64 * ((M + 63) / 64) <= 256) { *mf = 4; *nw = 1; }
}

// A launch of rounds that follow one another closely runs an eighth longer than the rounds by themselves (the clock falls).
double mid_us(const MatDev* mats, int n_mats, int M) {
    double us = 0.0;
    for (int base = 0; base < n_mats; base += kMidMaxMats) {
        const int end = std::min(n_mats, base + kMidMaxMats);
        long long rows = 0;
        for (int i = base; i < end; ++i) rows += mats[i].N;
        int mf, nw;
        pick_mid(M, rows, &mf, &nw);
        LaunchLoad load;
        for (int i = base; i < end; ++i) load.add((long long)(mats[i].N / (64 * nw)) * ((M + 16 * mf - 1) / (16 * mf)), mats[i].K);
        us += 3.0 + load.columns(0.5) * 1.12 * (36.0 + 8.6 * mf) / 56.0;
    }
    return us;
}

hipError_t launch_mid(const MatDev* mats, int n_mats, int M, int x_dtype, int y_dtype, bool exact, hipStream_t s) {
    for (int base = 0; base < n_mats; base += kMidMaxMats) {
        MidArgs a;
        const int cnt = std::min(kMidMaxMats, n_mats - base);
        int order[kMidMaxMats], mf, nw, nf = 4;
        long long rows = 0;
        for (int i = 0; i < cnt; ++i) { order[i] = base + i; rows += mats[base + i].N; }
        std::stable_sort(order, order + cnt, [&](int p, int q) { return mats[p].K > mats[q].K; });   // long workgroups first
        if (exact) {
            nw = 1;
            mf = mid_exact_mf(M);
            long long narrow = 0;
            for (int i = 0; i < cnt; ++i) narrow += (long long)((M + 63) / 64) * ((mats[base + i].N + 31) / 32);
            nf = mid_exact_nf(mf, narrow);
        }
        else pick_mid(M, rows, &mf, &nw);
        a.m_tiles = (M + 16 * mf - 1) / (16 * mf);
        int wgs = 0;
        for (int i = 0; i < kMidMaxMats; ++i) {
            if (i < cnt) {
                const MatDev& m = mats[order[i]];
                wgs += a.m_tiles * ((m.N + 16 * nf * nw - 1) / (16 * nf * nw));
                a.m[i] = MidMat{m.codes, m.aux, m.x, m.y, m.N, m.K, m.fmt, 0};
                a.wg_end[i] = wgs;
            } else {
                a.m[i] = MidMat{nullptr, nullptr, nullptr, nullptr, 0, 0, 0, 0};
                a.wg_end[i] = 0x7FFFFFFF;
            }
        }
        a.M = M; a.ydt = y_dtype; a.pad = 0;
        const hipError_t e = x_dtype == DT_BF16 ? launch_mid_shape<true>(a, mf, nw, nf, exact, wgs, s) : launch_mid_shape<false>(a, mf, nw, nf, exact, wgs, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace rwkvq

// Matrix-core path for large batches (prefill): y[M][N] = x[M][K] * Deq(W)^T with tiles of W
// dequantized into LDS and multiplied by v_mfma_f32_16x16x32_{bf16,f16} in the type of x,
// binary32 accumulate.  Grouped launch: the tiles of several matrices (each SQ or VQ as its flag
// says, Sec. 3.1 Eq. "optimization goal") share one grid so that all compute units stay busy.
//
// What is fed to the multipliers: Deq(W) exactly as defined in Sec. 2.2 (SQ: (q - z) * s in
// binary32; VQ: the fp16 codebook entry) rounded once, to nearest even, to the type of x.
//
// Tiling: workgroup = 256 threads = 2 x 2 wavefronts, block tile 256 (m) x 256 (n) x 64 (k),
// wavefront tile 128 x 128 = 8 x 8 MFMA tiles (256 accumulator registers).  Two more instances,
// 256 x 128 (wavefront tile 128 x 64) and 128 x 256, serve launches that would otherwise
// leave compute units without a tile; the launcher picks per launch (pick_shape).  Both operand tiles
// live in LDS as rows of 128 bytes (64 k), with the eight 16-byte chunks of a row stored at
// chunk ^ (row & 7), so that the 16-row fragment reads of the 16 x 16 x 32 MFMAs and the tile
// writes are free of bank conflicts without padding (the conflict counter reads zero).
//   * activations: copied global -> LDS by the load unit itself (global_load_lds_dwordx4), no
//     registers and no vector-ALU work; each lane fetches the chunk that belongs at its slot;
//   * weights: packed words are fetched once per 256 columns, unpacked by the vector ALU one
//     k-step ahead of the matrix cores, and written with 16-byte LDS stores.
// Two LDS buffers for W and three for x (two with 8-bit VQ); one workgroup barrier per k-step;
// waits on the load counter are placed by hand (the activations of step i + 2 are in flight during
// the MFMAs of step i).  The unpack and the copies are cut into micro-slices placed right behind
// individual MFMAs (see mma_step).
//
// Workgroup -> tile order: the m-tile index runs fastest, so workgroups that are dispatched
// round-robin over the 8 XCDs keep one slice of x (256 rows) per XCD L2 when there are 8 m-tiles.
#include "matrix_core.h"
#include "../../include/rwkvq.h"

#include <algorithm>
#include <vector>

namespace rwkvq {

constexpr int kPfMaxMats = 64;
// A wavefront tile is MF x NB tiles of 16 x 16 (rows of x, rows of W), a block tile twice that in each direction; the k-step is 64
// columns.
constexpr int wg_rows_w(int NB) { return 32 * NB; }
constexpr int kTileBytes = 256 * kRowBytes;    // an activation tile (32 KB)
constexpr int w_tile_bytes(int NB) { return wg_rows_w(NB) * kRowBytes; }
constexpr int row_tiles(int NB) { return NB / 2; }         // of 16 rows of W that a wavefront unpacks
constexpr int kCb8Bytes = 1024;                // converted 8-bit-index codebook
// Activation tiles in LDS: three (the copy of a k-step is issued two k-steps ahead of its use, so
// that its round trip to the cache hides behind a whole k-step of MFMAs) except with 8-bit VQ,
// whose converted codebooks take the room of the third beside tiles of 256 rows of W.
constexpr int x_buffers(int fmt, int NB) { return fmt == FMT_VQ8 && NB == 8 ? 2 : 3; }
constexpr int pf_lds_bytes(int fmt, int NB) { return 2 * w_tile_bytes(NB) + x_buffers(fmt, NB) * kTileBytes + (fmt == FMT_VQ8 ? 2 * kCb8Bytes : 0); }

struct PfMat {
    const uint32_t* codes;
    const uint16_t* aux;
    const void* x;
    void* y;
    int N, K, fmt, first;       // first: row of W at which the launch begins
};
struct PfArgs {
    int wg_end[kPfMaxMats];
    PfMat m[kPfMaxMats];
    int M, ydt, m_tiles, pad;
};

// Packed words of one 256-column tile for the RT row tiles (of 16 rows) a thread unpacks.
template <int FMT, int RT> struct WRegs;
template <int RT> struct WRegs<FMT_SQ3, RT> { uint4_t a[RT]; uint2_t b[RT]; uint2_t sz[RT]; };   // sz: (scale,zero) x 2 units
template <int RT> struct WRegs<FMT_VQ6, RT> { uint4_t a[RT]; uint2_t b[RT]; uint32_t cb; };     // cb: codebook entry `lane`
template <int RT> struct WRegs<FMT_VQ8, RT> { uint4_t a[RT]; uint4_t b[RT]; uint4_t cb8; };     // cb8: entries 4*lane..+3

// Where a wavefront finds its packed words: uniform tile pointers for its row tiles.
template <int RT> struct WSrc {
    const uint32_t* rows[RT];  // start of row tile R0 + RT*wave + i (advance by tile words per T)
    const uint16_t* aux;       // SQ: scale/zero of row tile R0 + RT*wave (16 uint2 per tile and T); VQ: codebooks of the block row
    int KT;
};

template <int FMT, int RT>
__device__ __forceinline__ void w_load(WRegs<FMT, RT>& r, const WSrc<RT>& src, int T, int lane) {
    constexpr int tw = FMT == FMT_VQ8 ? 512 : 384;
#pragma unroll
    for (int i = 0; i < RT; ++i) {
        const uint32_t* tile = src.rows[i] + (size_t)T * tw;
        r.a[i] = *(const uint4_t*)(tile + 4 * lane);
        if constexpr (FMT == FMT_VQ8) r.b[i] = *(const uint4_t*)(tile + 256 + 4 * lane);
        else r.b[i] = *(const uint2_t*)(tile + 256 + 2 * lane);
    }
    if constexpr (FMT == FMT_SQ3) {
#pragma unroll
        for (int i = 0; i < RT; ++i)
            r.sz[i] = ((const uint2_t*)src.aux + ((size_t)i * src.KT + T) * 16)[lane & 15];
    } else if constexpr (FMT == FMT_VQ6) {
        r.cb = ((const uint32_t*)src.aux + (size_t)T * 64)[lane];
    } else {
        r.cb8 = ((const uint4_t*)src.aux + (size_t)T * 64)[lane];
    }
}

// Unpack k-step KQ (0..3: 64 columns) of the tile held in r and write it to the W tile in LDS.
template <bool BF16, int FMT, int KQ, int RT>
__device__ __forceinline__ void w_unpack(const WRegs<FMT, RT>& r, char* wt, const uint32_t* cb8, int wave, int lane) {
    constexpr int u = KQ >> 1, t0 = 2 * (KQ & 1);
    const int row0 = 16 * RT * wave + (lane & 15), kg = lane >> 4;
    // rows row0 + 16 i share row & 7, so the two chunk offsets are the same for all of them
    char* d0 = wt + tile_off(row0, kg);
    char* d1 = wt + tile_off(row0, 4 + kg);
    if constexpr (FMT == FMT_SQ3) {
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            const uint32_t w0 = u == 0 ? r.a[i].x : r.a[i].w, w1 = u == 0 ? r.a[i].y : r.b[i].x,
                           w2 = u == 0 ? r.a[i].z : r.b[i].y;
            const uint32_t szw = u == 0 ? r.sz[i].x : r.sz[i].y;
            const float s = f16_bits_to_f32((uint16_t)(szw & 0xFFFFu)), z = f16_bits_to_f32((uint16_t)(szw >> 16));
            *(uint4_t*)(d0 + 16 * i * kRowBytes) = sq_chunk<BF16, t0>(w0, w1, w2, s, z);
            *(uint4_t*)(d1 + 16 * i * kRowBytes) = sq_chunk<BF16, t0 + 1>(w0, w1, w2, s, z);
        }
    } else if constexpr (FMT == FMT_VQ6) {
        const uint32_t cb = Elem<BF16>::from_f16x2(r.cb);
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            const uint32_t w0 = u == 0 ? r.a[i].x : r.a[i].w, w1 = u == 0 ? r.a[i].y : r.b[i].x,
                           w2 = u == 0 ? r.a[i].z : r.b[i].y;
            *(uint4_t*)(d0 + 16 * i * kRowBytes) = vq6_chunk<t0>(w0, w1, w2, cb);
            *(uint4_t*)(d1 + 16 * i * kRowBytes) = vq6_chunk<t0 + 1>(w0, w1, w2, cb);
        }
    } else {
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            const uint32_t wa = u == 0 ? (t0 == 0 ? r.a[i].x : r.a[i].z) : (t0 == 0 ? r.b[i].x : r.b[i].z);
            const uint32_t wb = u == 0 ? (t0 == 0 ? r.a[i].y : r.a[i].w) : (t0 == 0 ? r.b[i].y : r.b[i].w);
            *(uint4_t*)(d0 + 16 * i * kRowBytes) = vq8_chunk(wa, cb8);
            *(uint4_t*)(d1 + 16 * i * kRowBytes) = vq8_chunk(wb, cb8);
        }
    }
}

// The same work cut into 32 micro-slices per row tile, one per MFMA of the previous k-step (see mma_step): a
// weight pair takes four of them (mask / address; subtract the zero point or start the look-up;
// scale; pack and, every fourth pair, store the finished 16-byte chunk).  Micro-slice S works on
// pair (S / 4) % 4 of chunk (S / 16) % 2 of row tile S / 32.  Each is two or three vector
// instructions: what the matrix core leaves room for behind one MFMA of the same wavefront.
template <int FMT> struct UnpackState {
    char *d0, *d1;            // LDS addresses of the lane's two chunks of row tile 0
    uint4_t stage;            // the chunk being assembled
    float s, z;               // SQ: scale and zero point of the current row tile and unit
    float lo, hi;             // SQ: the pair in flight
    uint32_t m;               // masked codes / look-up address / looked-up pair in flight
    uint32_t cb;              // VQ6: the lane's codebook entry, converted to the operand type
};

template <bool BF16, int FMT, int RT>
__device__ __forceinline__ void unpack_begin(UnpackState<FMT>& st, const WRegs<FMT, RT>& r, char* wt, int wave, int lane) {
    const int row0 = 16 * RT * wave + (lane & 15), kg = lane >> 4;
    st.d0 = wt + tile_off(row0, kg);
    st.d1 = wt + tile_off(row0, 4 + kg);
    if constexpr (FMT == FMT_VQ6) st.cb = Elem<BF16>::from_f16x2(r.cb);
}

template <bool BF16, int FMT, int KQ, int S, int RT>
__device__ __forceinline__ void unpack_micro(UnpackState<FMT>& st, const WRegs<FMT, RT>& r, const uint32_t* cb8) {
    constexpr int u = KQ >> 1, t0 = 2 * (KQ & 1);
    constexpr int i = S >> 5, c = (S >> 4) & 1, p = (S >> 2) & 3, q = S & 3, P = 4 * (t0 + c) + p;
    if constexpr (FMT == FMT_SQ3) {
        const uint32_t w0 = u == 0 ? r.a[i].x : r.a[i].w, w1 = u == 0 ? r.a[i].y : r.b[i].x,
                       w2 = u == 0 ? r.a[i].z : r.b[i].y;
        if constexpr (q == 0) {
            if constexpr ((S & 31) == 0) {
                const uint32_t szw = u == 0 ? r.sz[i].x : r.sz[i].y;
                st.s = f16_bits_to_f32((uint16_t)(szw & 0xFFFFu));
                st.z = f16_bits_to_f32((uint16_t)(szw >> 16));
            }
            st.m = sq_pair_mask<P>(w0, w1, w2);
        } else if constexpr (q == 1) {
            const half2_t h = __builtin_bit_cast(half2_t, st.m);
            st.lo = fmaf((float)h.x, sq_pair_unscale<P>(), -st.z);
            st.hi = fmaf((float)h.y, sq_pair_unscale<P>(), -st.z);
        } else if constexpr (q == 2) {
            st.lo = __fmul_rn(st.lo, st.s);
            st.hi = __fmul_rn(st.hi, st.s);
        } else {
            st.m = Elem<BF16>::pack(st.lo, st.hi);
        }
    } else if constexpr (FMT == FMT_VQ6) {
        const uint32_t w0 = u == 0 ? r.a[i].x : r.a[i].w, w1 = u == 0 ? r.a[i].y : r.b[i].x,
                       w2 = u == 0 ? r.a[i].z : r.b[i].y;
        if constexpr (q == 0) st.m = vq6_byteaddr<P>(w0, w1, w2);
        else if constexpr (q == 1) st.m = __builtin_amdgcn_ds_bpermute(st.m, st.cb);
    } else {
        const uint32_t wa = u == 0 ? (t0 == 0 ? r.a[i].x : r.a[i].z) : (t0 == 0 ? r.b[i].x : r.b[i].z);
        const uint32_t wb = u == 0 ? (t0 == 0 ? r.a[i].y : r.a[i].w) : (t0 == 0 ? r.b[i].y : r.b[i].w);
        const uint32_t w = c == 0 ? wa : wb;
        if constexpr (q == 0) st.m = (w >> (8 * p)) & 255u;
        else if constexpr (q == 1) st.m = cb8[st.m];
    }
    if constexpr (q == 3) {
        if constexpr (p == 0) st.stage.x = st.m;
        else if constexpr (p == 1) st.stage.y = st.m;
        else if constexpr (p == 2) st.stage.z = st.m;
        else {
            st.stage.w = st.m;
            *(uint4_t*)((c == 0 ? st.d0 : st.d1) + 16 * i * kRowBytes) = st.stage;
        }
    }
}

// Copy the activation tile, columns k0..k0+63 of the block's 256 rows, into an LDS tile, 16 bytes
// per lane and instruction, the load unit writing LDS directly.  LDS slot p (16 bytes) = row
// p/8, position p%8; the lane that owns slot p fetches the logical chunk the swizzle stores there.
// xoff[i] is the lane's byte offset (row * K * 2 + chunk * 16) from the tile's first row, computed
// once; xk = activations of the tile's first row at column k0 (uniform).
template <int I>
__device__ __forceinline__ void x_tile_dma_one(const char* xk, const uint32_t (&xoff)[8], char* xt, int wave) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(xk + xoff[I]),
                                     (__attribute__((address_space(3))) void*)(xt + (256 * I + 64 * wave) * 16),
                                     16, 0, 0);
}
template <int MF>
__device__ __forceinline__ void x_tile_dma(const char* xk, const uint32_t (&xoff)[8], char* xt, int wave) {
#pragma unroll
    for (int i = 0; i < MF; ++i)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(xk + xoff[i]),
                                         (__attribute__((address_space(3))) void*)(xt + (256 * i + 64 * wave) * 16),
                                         16, 0, 0);
}

// One k-step (64 columns) of the wavefront tile = 2 MF rows of NB MFMAs: x fragment f (m-subtile f % MF of column half f / MF)
// against the NB W fragments of that half.  x fragments are read kAhead rows ahead of their use and the W fragments of the second
// half during the last four rows of the first, so that an LDS round trip is hidden behind several rows of MFMAs.
constexpr int kAhead = 3;
template <int S> struct SliceTag { static constexpr int value = S; };

template <bool BF16, int MF, int NB, int F, int NI, class Slice>
__device__ __forceinline__ void mma_one(const uint4_t (&b)[NB], const uint4_t af, float4_t (&acc)[MF][NB], Slice& slice) {
    // One MFMA of x fragment F, then one micro-slice of vector-ALU work, fenced so that the
    // instruction scheduler leaves it there: a wavefront issues in order, and only the two or
    // three instructions placed right behind an MFMA run while the matrix core is busy with it
    // (left alone, the scheduler gathers the unpack work into long runs before its stores, and
    // the matrix core idles through them).
    Elem<BF16>::mfma(b[NI], af, acc[F % MF][NI]);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (MF == 8) {
        slice(SliceTag<NB * F + NI>{});
    } else {                                       // half the rows of x, half as many MFMAs: two micro-slices behind each
        slice(SliceTag<2 * (NB * F + NI)>{});
        slice(SliceTag<2 * (NB * F + NI) + 1>{});
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (NI < NB - 1) mma_one<BF16, MF, NB, F, NI + 1>(b, af, acc, slice);
}
template <bool BF16, int MF, int NB, int F, class Slice>
__device__ __forceinline__ void mma_row(const uint4_t (&b)[NB], const uint4_t af, float4_t (&acc)[MF][NB], Slice& slice) {
    mma_one<BF16, MF, NB, F, 0>(b, af, acc, slice);
}

template <bool BF16, int MF, int NB, int F, class Slice>
__device__ __forceinline__ void mma_rows(const char* const (&xa)[2], const char* wb1, uint4_t (&b)[NB], uint4_t (&b1)[NB],
                                         uint4_t (&a)[kAhead + 1], float4_t (&acc)[MF][NB], Slice& slice) {
    if constexpr (F < 2 * MF) {
        if constexpr (F + kAhead < 2 * MF)
            a[(F + kAhead) % (kAhead + 1)] = *(const uint4_t*)(xa[(F + kAhead) / MF] + 16 * ((F + kAhead) % MF) * kRowBytes);
        if constexpr (F >= MF - 4 && F < MF) {                  // the last four rows of the first half
            constexpr int J = F - (MF - 4);
#pragma unroll
            for (int q = J * NB / 4; q < (J + 1) * NB / 4; ++q) b1[q] = *(const uint4_t*)(wb1 + 16 * q * kRowBytes);
        }
        if constexpr (F < MF) mma_row<BF16, MF, NB, F>(b, a[F % (kAhead + 1)], acc, slice);
        else mma_row<BF16, MF, NB, F>(b1, a[F % (kAhead + 1)], acc, slice);
        mma_rows<BF16, MF, NB, F + 1>(xa, wb1, b, b1, a, acc, slice);
    }
}

// The k-step.  `slice(SliceTag<S>)` is called after MFMA S: the unpacking of the next k-step goes there.
template <bool BF16, int MF, int NB, class Slice>
__device__ __forceinline__ void mma_step(const char* xt, const char* wt, int wm, int wn, int lane,
                                         float4_t (&acc)[MF][NB], Slice slice) {
    const int r = lane & 15, kg = lane >> 4;
    const char* const xa[2] = {xt + tile_off(16 * MF * wm + r, kg), xt + tile_off(16 * MF * wm + r, 4 + kg)};
    const char* wb0 = wt + tile_off(16 * NB * wn + r, kg);
    const char* wb1 = wt + tile_off(16 * NB * wn + r, 4 + kg);
    uint4_t b[NB], b1[NB], a[kAhead + 1];
#pragma unroll
    for (int ni = 0; ni < NB; ++ni) b[ni] = *(const uint4_t*)(wb0 + 16 * ni * kRowBytes);
#pragma unroll
    for (int f = 0; f < kAhead; ++f) a[f] = *(const uint4_t*)(xa[0] + 16 * f * kRowBytes);
    mma_rows<BF16, MF, NB, 0>(xa, wb1, b, b1, a, acc, slice);
}

// Convert and stage the 8-bit-index codebook of a tile (256 entries) into LDS.
template <bool BF16, int RT>
__device__ __forceinline__ void cb8_store(const WRegs<FMT_VQ8, RT>& r, uint32_t* cb8, int wave, int lane) {
    if (wave == 0) {
        uint4_t c = {Elem<BF16>::from_f16x2(r.cb8.x), Elem<BF16>::from_f16x2(r.cb8.y),
                     Elem<BF16>::from_f16x2(r.cb8.z), Elem<BF16>::from_f16x2(r.cb8.w)};
        *(uint4_t*)(cb8 + 4 * lane) = c;
    }
}

// All matrices of one launch have the format FMT.  The k loop has no conditionals: past the last
// column tile the prefetches simply fetch the last tile again (never used).
// Block tiles (rows of x x rows of W): 256 x 256 (MF = NB = 8); for launches that would leave compute units without a tile 256 x 128
// (NB = 4: half the unpack with half the MFMAs) and, where fewer rows of x are padded that way, 128 x 256 (MF = 4: the same
// unpack on half the MFMAs).  All sum over k in the same order.
template <bool BF16, int FMT, int MF, int NB>
__global__ void __launch_bounds__(256, 1) prefill_kernel(PfArgs a) {
    constexpr int BMk = 32 * MF, BN = wg_rows_w(NB), RT = row_tiles(NB);      // rows of x and of W per workgroup
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    constexpr int XB = x_buffers(FMT, NB), LA = XB - 1;       // LA = k-steps between a copy and its use
    char* const wt0 = lds;
    char* const wt1 = lds + w_tile_bytes(NB);
    char* const xbase = lds + 2 * w_tile_bytes(NB);
    uint32_t* const cb8base = (uint32_t*)(xbase + XB * kTileBytes);
#define CB8(i) (cb8base + ((i) & 1) * (kCb8Bytes / 4))

    const int wg = blockIdx.x;
    static_assert(kPfMaxMats == 64, "one table entry per lane");
    const int mi_ = __builtin_popcountll(__builtin_amdgcn_ballot_w64(wg >= a.wg_end[threadIdx.x & 63]));
    const PfMat mt = a.m[mi_];
    const int local = wg - (mi_ ? a.wg_end[mi_ - 1] : 0);
    const int m0 = (local % a.m_tiles) * BMk, n0 = mt.first + (local / a.m_tiles) * BN;
    const int M = a.M, K = mt.K, KT = K >> 8, R0 = n0 >> 4;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 1, wn = wave & 1;

    // per-lane activation offsets (rows past M repeat row M - 1)
    uint32_t xoff[8];
#pragma unroll
    for (int i = 0; i < MF; ++i) {
        const int p = 256 * i + 64 * wave + lane;
        const int row = p >> 3, c = (p & 7) ^ (row & 7);
        const int rr = m0 + row < M ? row : M - 1 - m0;
        xoff[i] = (uint32_t)rr * (uint32_t)K * 2u + 16u * c;
    }
    const char* xrow0 = (const char*)mt.x + (size_t)m0 * K * 2;

    WSrc<RT> src;
    constexpr int tw = FMT == FMT_VQ8 ? 512 : 384;
#pragma unroll
    for (int i = 0; i < RT; ++i) src.rows[i] = mt.codes + (size_t)(R0 + RT * wave + i) * KT * tw;
    src.KT = KT;
    if constexpr (FMT == FMT_SQ3) src.aux = (const uint16_t*)((const uint2_t*)mt.aux + (size_t)(R0 + RT * wave) * KT * 16);
    else if constexpr (FMT == FMT_VQ6) src.aux = (const uint16_t*)((const uint32_t*)mt.aux + (size_t)(R0 >> 4) * KT * 64);
    else src.aux = (const uint16_t*)((const uint4_t*)mt.aux + (size_t)(R0 >> 4) * KT * 64);

    float4_t acc[MF][NB];
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = float4_t{0, 0, 0, 0};

    // The activation buffers form a ring (byte offsets from xbase): x0 holds the k-step being
    // multiplied, x1 the next one, x2 (three buffers) the one after.  A k-step's copy is issued LA
    // k-steps ahead; eight copy instructions per thread and k-step, so "all but the newest eight
    // memory operations done" is the wait that lets the newest copy stay in flight.
    int x0 = 0, x1 = kTileBytes, x2 = 2 * kTileBytes;
    const int hmax = 4 * KT - 1;                           // last k-step
    auto xk = [&](int h) { return xrow0 + (size_t)(h < hmax ? h : hmax) * kRowBytes; };
    auto rotate = [&] { if (XB == 3) { const int t = x0; x0 = x1; x1 = x2; x2 = t; } else { const int t = x0; x0 = x1; x1 = t; } };
    auto wait_step = [&] {                                 // all but the newest copy (MF instructions per thread)
        if (LA == 2) { if (MF == 8) RWKVQ_WAIT_VM8_LGKM0(); else RWKVQ_WAIT_VM4_LGKM0(); }
        else RWKVQ_WAIT_VM0_LGKM0();
    };

    // prologue: packed words of tile 0, k-step 0 (and 1) of the activations, k-step 0 of W
    WRegs<FMT, RT> wr;
    UnpackState<FMT> us;
    w_load<FMT, RT>(wr, src, 0, lane);
    x_tile_dma<MF>(xk(0), xoff, xbase + x0, wave);
    if (LA == 2) x_tile_dma<MF>(xk(1), xoff, xbase + x1, wave);
    if constexpr (FMT == FMT_VQ8) {
        cb8_store<BF16>(wr, CB8(0), wave, lane);
        RWKVQ_WAIT_VM0_LGKM0();
        RWKVQ_BARRIER();
    }
    w_unpack<BF16, FMT, 0, RT>(wr, wt0, CB8(0), wave, lane);
    RWKVQ_WAIT_VM0_LGKM0();
    RWKVQ_BARRIER();

    for (int T = 0; T < KT; ++T) {
        const int Tn = T + 1 < KT ? T + 1 : T;
        const int g = 4 * T;                               // k-step index of the tile's first step
        // k-step 0 of the tile is in W buffer 0; steps 1..3 come from the same packed words and are
        // unpacked, a few instructions at a time, behind the MFMAs of the step before; the eight
        // copy instructions of the activation tile LA steps ahead go behind MFMAs as well.
        {
            const char* xsrc = xk(g + LA);
            char* xdst = xbase + (LA == 2 ? x2 : x1);
            unpack_begin<BF16, FMT>(us, wr, wt1, wave, lane);
            mma_step<BF16, MF, NB>(xbase + x0, wt0, wm, wn, lane, acc, [&](auto tag) {
                constexpr int S = decltype(tag)::value;
                if constexpr (S % 8 == 4 && S / 8 < MF) x_tile_dma_one<S / 8>(xsrc, xoff, xdst, wave);
                unpack_micro<BF16, FMT, 1, S>(us, wr, CB8(T));
            });
        }
        wait_step();
        RWKVQ_BARRIER();
        rotate();

        {
            const char* xsrc = xk(g + 1 + LA);
            char* xdst = xbase + (LA == 2 ? x2 : x1);
            unpack_begin<BF16, FMT>(us, wr, wt0, wave, lane);
            mma_step<BF16, MF, NB>(xbase + x0, wt1, wm, wn, lane, acc, [&](auto tag) {
                constexpr int S = decltype(tag)::value;
                if constexpr (S % 8 == 4 && S / 8 < MF) x_tile_dma_one<S / 8>(xsrc, xoff, xdst, wave);
                unpack_micro<BF16, FMT, 2, S>(us, wr, CB8(T));
            });
        }
        wait_step();
        RWKVQ_BARRIER();
        rotate();

        {
            const char* xsrc = xk(g + 2 + LA);
            char* xdst = xbase + (LA == 2 ? x2 : x1);
            unpack_begin<BF16, FMT>(us, wr, wt1, wave, lane);
            mma_step<BF16, MF, NB>(xbase + x0, wt0, wm, wn, lane, acc, [&](auto tag) {
                constexpr int S = decltype(tag)::value;
                if constexpr (S % 8 == 4 && S / 8 < MF) x_tile_dma_one<S / 8>(xsrc, xoff, xdst, wave);
                unpack_micro<BF16, FMT, 3, S>(us, wr, CB8(T));
            });
        }
        wait_step();
        RWKVQ_BARRIER();
        rotate();

        // the packed words of this tile are spent: fetch the next tile's into the same registers
        // (before the activation copy, so that waiting for them leaves the copy in flight); they
        // have a whole MFMA step to arrive
        w_load<FMT, RT>(wr, src, Tn, lane);
        {
            const char* xsrc = xk(g + 3 + LA);
            char* xdst = xbase + (LA == 2 ? x2 : x1);
            mma_step<BF16, MF, NB>(xbase + x0, wt1, wm, wn, lane, acc, [&](auto tag) {
                constexpr int S = decltype(tag)::value;
                if constexpr (S % 8 == 4 && S / 8 < MF) x_tile_dma_one<S / 8>(xsrc, xoff, xdst, wave);
            });
        }
        if constexpr (FMT == FMT_VQ8) {
            cb8_store<BF16>(wr, CB8(T + 1), wave, lane);
            RWKVQ_WAIT_VM0_LGKM0();
            RWKVQ_BARRIER();
        } else {
            wait_step();                                   // the packed words have landed
        }
        w_unpack<BF16, FMT, 0, RT>(wr, wt0, CB8(T + 1), wave, lane);
        wait_step();
        RWKVQ_BARRIER();
        rotate();
    }

    // The MFMAs are opaque to the compiler's hazard checks: let the last ones drain before the
    // accumulators are read (the longest MFMA-to-read hazard is well under 32 cycles).
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");

    // epilogue: the W fragment is the A operand of the MFMA, so a lane holds, for every 16 x 16
    // tile, output row m = lane%16 and the four consecutive columns n = 4*(lane/16) + 0..3:
    // one 8-byte (or 16-byte for fp32) store per tile.
    const int N = mt.N;
#pragma unroll
    for (int mi = 0; mi < MF; ++mi) {
        const int m = m0 + 16 * MF * wm + 16 * mi + (lane & 15);
        if (m < M) {
#pragma unroll
            for (int ni = 0; ni < NB; ++ni) {
                const size_t o = (size_t)m * N + n0 + 16 * NB * wn + 16 * ni + 4 * (lane >> 4);
                const float4_t v = acc[mi][ni];
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
#undef CB8
}

// The kernels need more dynamic LDS than the default limit: raised once per kernel and device.  Two
// threads that get here together both raise it, which is harmless.
template <bool BF16, int FMT, int MF, int NB>
static hipError_t launch_shape(const PfArgs& a, int wgs, hipStream_t s) {
    static std::atomic<unsigned long long> raised{0ull};
    const hipError_t e = raise_lds((const void*)prefill_kernel<BF16, FMT, MF, NB>, pf_lds_bytes(FMT, NB), raised);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((prefill_kernel<BF16, FMT, MF, NB>), dim3(wgs), dim3(256), pf_lds_bytes(FMT, NB), s, a);
    return hipGetLastError();
}

// Rows of x and of W per workgroup, and the duration of a column tile in units of that of 256 x 256.
struct PfShape { int bm, bn; double cost; };
template <bool BF16, int FMT>
static hipError_t launch_fmt(const PfArgs& a, int wgs, const PfShape& p, hipStream_t s) {
    return p.bm == 128 ? launch_shape<BF16, FMT, 4, 8>(a, wgs, s) : p.bn == 128 ? launch_shape<BF16, FMT, 8, 4>(a, wgs, s)
                                                                  : launch_shape<BF16, FMT, 8, 8>(a, wgs, s);
}

// The shape for a launch whose matrices have `n_tiles` tiles of 256 rows of W in all.  One workgroup runs per compute unit, so a
// launch takes about ceil(workgroups / 256) rounds, and the cheapest of the three wins.  Measured on the 7B stack (cost of a
// column tile): half the rows of x do half the MFMAs at 0.71 of the rate, since the W tile is unpacked once per workgroup either
// way; half the rows of W, with half the unpack, cost 0.645 (4096 x 4096 at M = 2048 85 -> 74 us,
// 4096 x 14336 267 -> 232, 6-bit VQ 283 -> 225).
// rwkvq_set_option(RWKVQ_OPT_PREFILL_TILE_ROWS, 128 | 256) takes 128 x 256 or 256 x 256 (tests run both kernels).
constexpr PfShape kShapes[3] = {{256, 256, 1.0}, {128, 256, 0.705}, {256, 128, 0.645}};
static double rounds(long long wgs) { return (double)((wgs + 255) / 256); }
static PfShape pick_shape(int M, long long n_tiles) {
    const int forced = option(RWKVQ_OPT_PREFILL_TILE_ROWS);
    if (forced == 128 || forced == 256) return kShapes[forced == 128];
    PfShape best = kShapes[0];
    double least = 1e30;
    for (const PfShape& p : kShapes) {
        const double t = p.cost * rounds(n_tiles * (256 / p.bn) * ((M + p.bm - 1) / p.bm));
        if (t < least) { least = t; best = p; }
    }
    return best;
}

// A launch over matrices of one format: tiles of 256 rows of W, the shape, and where whole rounds of 256 x 256 tiles with what is left
// of them in tiles of half the rows of W end sooner than a last round with a few tiles ({key, receptance} of the 7B shapes at M =
// 2048, 576 tiles: 344 -> 306 us), how many of the tiles the whole rounds take (0: one launch).  Matrices of one K only: elsewhere
// the shorter ones fill the end.  Longest rows first.
struct PfPlan { int tiles, whole; PfShape p; };
static PfPlan plan_tiles(const std::vector<MatDev>& batch, int M) {
    PfPlan plan{0, 0, {}};
    for (const MatDev& m : batch) plan.tiles += m.N / 256;
    plan.p = pick_shape(M, plan.tiles);
    const PfShape& p = plan.p;
    const int m_tiles = (M + 255) / 256, whole = (int)((long long)plan.tiles * m_tiles / 256 * 256 / m_tiles);
    if (option(RWKVQ_OPT_PREFILL_TILE_ROWS) == 0 && whole > 0 && whole < plan.tiles && batch.front().K == batch.back().K &&
        rounds((long long)whole * m_tiles) + kShapes[2].cost * rounds((long long)(plan.tiles - whole) * 2 * m_tiles) + 0.05 <
            p.cost * rounds((long long)plan.tiles * (256 / p.bn) * ((M + p.bm - 1) / p.bm)))
        plan.whole = whole;
    return plan;
}

// The matrices of one launch after another: one format, at most 64, in order.
template <class F>
static void each_batch(const std::vector<MatDev>& sorted, F&& f) {
    for (int fmt = 0; fmt < 3; ++fmt) {
        std::vector<MatDev> batch;
        for (size_t i = 0; i <= sorted.size(); ++i) {
            if (i < sorted.size() && sorted[i].fmt == fmt) batch.push_back(sorted[i]);
            if (batch.empty() || ((int)batch.size() < kPfMaxMats && i < sorted.size())) continue;
            f(batch);
            batch.clear();
        }
    }
}
// Workgroups of a matrix with a long K run long: put those matrices first so that the end of a launch is filled by short workgroups.
static std::vector<MatDev> longest_first(const MatDev* mats, int n_mats) {
    std::vector<MatDev> sorted(mats, mats + n_mats);
    std::stable_sort(sorted.begin(), sorted.end(), [](const MatDev& a, const MatDev& b) { return a.K > b.K; });
    return sorted;
}

// Estimated duration here: 7.4 us per column tile of a 256-row workgroup, 3 us per launch.
static double tiles_us(const std::vector<MatDev>& mats, int M) {
    double us = 0.0;
    each_batch(longest_first(mats.data(), (int)mats.size()), [&](const std::vector<MatDev>& batch) {
        const PfPlan plan = plan_tiles(batch, M);
        const PfShape& p = plan.p;
        LaunchLoad load;
        for (const MatDev& m : batch) load.add((long long)(m.N / p.bn) * ((M + p.bm - 1) / p.bm), m.K);
        double t = load.columns(0.2) * p.cost * 7.4;
        if (plan.whole) {
            const int m_tiles = (M + 255) / 256;
            t = std::min(t, 3.0 + 7.4 * (batch.front().K >> 8) * (rounds((long long)plan.whole * m_tiles) +
                                                                  kShapes[2].cost * rounds((long long)(plan.tiles - plan.whole) * 2 * m_tiles)));
        }
        us += 3.0 + t;
    });
    return us;
}

// Up to kMidMaxM rows of x the kernels of midbatch.hip are an alternative: workgroups of a quarter of the size, K split over
// groups of wavefronts and all formats in one launch, which fills the device from small calls, for an unpack that serves 128
// rows of x instead of 256.  At M <= 128 they won every call measured; beyond, the cheaper estimate is taken.  Over 210 calls
// (o, {r, k, v, g}, {key, receptance}, value, 1 to 32 whole layers of the 7B shapes, 4 of 14B-class shapes; one and two
// formats; M = 129 .. 1536; us, here / there): none takes the slower one by more than 4 %.  There: {r, k, v, g} of two formats
// at M = 1024 178 / 140, 4096 x 4096 alone 82 / 41, value 269 / 120, one layer 595 / 454, 32 layers at 333 rows 6047 / 5453.
// Here: 14336 x 4096 alone 120 / 136, {r, k, v, g} of one format 125 / 142, four layers 1559 / 1722, 32 layers
// 12435 / 14509.  With whole rounds and a rest in the estimate (1650 calls, widths 1024 to 5120, M = 129 to 1536, bf16) 15 calls take the
// tiles that took the others, {key, receptance} and key alone: 14336 x 4096 SQ at M = 1536 221 -> 203, {key, receptance} of 14B-class
// shapes at 900 259 -> 248.  The order of a matrix's binary32 sums over K differs between the two, so for 128 < M <= kMidMaxM it depends
// on the sizes of the call; a forced tile height (RWKVQ_OPT_PREFILL_TILE_ROWS) stays here, with one order for every M > 128.
constexpr int kMidMaxM = 1536;
static bool mid_takes(const MatDev& m, int M) { return M <= kMidMaxM && m.K <= (1 << 20) && option(RWKVQ_OPT_PREFILL_TILE_ROWS) == 0; }

// Tiles t0 .. t1 - 1 of 256 rows of W, counted through the matrices of `batch`, all of one format.
static hipError_t launch_batch(const std::vector<MatDev>& batch, int t0, int t1, const PfShape& p, int M, int x_dtype, int y_dtype, hipStream_t s) {
    PfArgs a;
    int cnt = 0, wgs = 0, at = 0;
    a.M = M; a.ydt = y_dtype; a.m_tiles = (M + p.bm - 1) / p.bm; a.pad = 0;
    for (const MatDev& m : batch) {
        const int from = std::max(t0, at), to = std::min(t1, at + m.N / 256);
        if (from < to) {
            wgs += a.m_tiles * (to - from) * (256 / p.bn);
            a.m[cnt] = PfMat{m.codes, m.aux, m.x, m.y, m.N, m.K, m.fmt, 256 * (from - at)};
            a.wg_end[cnt++] = wgs;
        }
        at += m.N / 256;
    }
    for (int j = cnt; j < kPfMaxMats; ++j) {
        a.m[j] = PfMat{nullptr, nullptr, nullptr, nullptr, 0, 0, 0, 0};
        a.wg_end[j] = 0x7FFFFFFF;
    }
    const bool bf = x_dtype == DT_BF16;
    switch (batch[0].fmt) {
        case FMT_SQ3: return bf ? launch_fmt<true, FMT_SQ3>(a, wgs, p, s) : launch_fmt<false, FMT_SQ3>(a, wgs, p, s);
        case FMT_VQ6: return bf ? launch_fmt<true, FMT_VQ6>(a, wgs, p, s) : launch_fmt<false, FMT_VQ6>(a, wgs, p, s);
        default: return bf ? launch_fmt<true, FMT_VQ8>(a, wgs, p, s) : launch_fmt<false, FMT_VQ8>(a, wgs, p, s);
    }
}

static hipError_t launch_prefill_tiles(const MatDev* mats, int n_mats, int M, int x_dtype, int y_dtype, hipStream_t s) {
    hipError_t e = hipSuccess;
    each_batch(longest_first(mats, n_mats), [&](const std::vector<MatDev>& batch) {
        const PfPlan plan = plan_tiles(batch, M);
        if (e == hipSuccess) e = launch_batch(batch, 0, plan.whole ? plan.whole : plan.tiles, plan.whole ? kShapes[0] : plan.p, M, x_dtype, y_dtype, s);
        if (e == hipSuccess && plan.whole) e = launch_batch(batch, plan.whole, plan.tiles, kShapes[2], M, x_dtype, y_dtype, s);
    });
    return e;
}

hipError_t launch_prefill(const MatDev* mats, int n_mats, int M, int x_dtype, int y_dtype, hipStream_t s) {
    std::vector<MatDev> mid, tiles;
    for (int i = 0; i < n_mats; ++i) (mid_takes(mats[i], M) ? mid : tiles).push_back(mats[i]);    // (a K beyond its 32-bit offsets)
    if (M > 128 && !mid.empty() && tiles_us(mid, M) < mid_us(mid.data(), (int)mid.size(), M)) {
        tiles.assign(mats, mats + n_mats);
        mid.clear();
    }
    hipError_t e = mid.empty() ? hipSuccess : launch_mid(mid.data(), (int)mid.size(), M, x_dtype, y_dtype, false, s);
    if (e == hipSuccess && !tiles.empty()) e = launch_prefill_tiles(tiles.data(), (int)tiles.size(), M, x_dtype, y_dtype, s);
    return e;
}

}  // namespace rwkvq

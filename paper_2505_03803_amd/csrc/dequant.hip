// Prepack (canonical -> native layout) and dense dequantization kernels.
//
// Dequantization follows Sec. 2.2: SQ  w = (q - z) * s  per group of 128 input channels
// (inverse of Eq. "SQ"), VQ  (w[n,2j], w[n,2j+1]) = codebook[block(n, 2j)][index[n,j]]
// (Eq. "VQ").  The dense kernels are plain gathers: one thread per element.
#include "common.h"

namespace rwkvq {

// ------------------------------------------------------------------ prepack

// A wavefront per native tile of 16 rows x 256 columns: lane l holds row l & 15, and of both units of 128 columns the four
// chunks of eight columns 8 (l >> 4) .. + 7 in every 32.  A chunk of eight 3-bit codes or four 6-bit indices is 24 consecutive
// bits of the canonical row, a chunk of four 8-bit indices one word, so a lane takes whole chunks from the tile's 96 or 128
// bytes of its row and writes its native words with two stores.  Bound by the bytes read and written; the form before, a
// thread per native word, fetched each field by itself (two loads for most).  Measured (before -> here): codes of
// 14336 x 4096 with scales 124 -> 16 us, 4096 x 4096 39 -> 8.6;
// 6-bit indices of 14336 x 4096 66 -> 14, 8-bit 20 -> 17.
__device__ __forceinline__ void load_chunks24(const uint32_t* row, int kg, uint32_t (&f)[2][4]) {
    uint32_t w[24];
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        const uint4_t v = *(const uint4_t*)(row + 4 * i);
        w[4 * i] = v.x; w[4 * i + 1] = v.y; w[4 * i + 2] = v.z; w[4 * i + 3] = v.w;
    }
    // chunk kg of a step's three words: bits 24 kg .. 24 kg + 23, in the two words from (3 kg) / 4 on
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const uint32_t lo = kg < 2 ? w[3 * i] : w[3 * i + 1];
        const uint32_t hi = kg < 2 ? w[3 * i + 1] : w[3 * i + 2];
        const int sh = kg < 2 ? 24 * kg : 24 * kg - 32;
        f[i >> 2][i & 3] = (uint32_t)((((uint64_t)hi << 32) | lo) >> sh) & 0xFFFFFFu;
    }
}

__device__ __forceinline__ void store_tile6(uint32_t* tile, int lane, const uint32_t (&o)[6]) {
    *(uint4_t*)(tile + 4 * lane) = uint4_t{o[0], o[1], o[2], o[3]};
    *(uint2_t*)(tile + 256 + 2 * lane) = uint2_t{o[4], o[5]};
}

// Codes, and (lanes of the first column group) scale and zero of the row's two groups interleaved.
__global__ void __launch_bounds__(256) sq_prepack_kernel(const uint32_t* __restrict__ codes, const uint16_t* __restrict__ scales,
                                                         const uint16_t* __restrict__ zeros, int N, int K,
                                                         uint32_t* __restrict__ out, uint16_t* __restrict__ sz) {
    const size_t tile = (size_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int tiles_k = K / 256, lane = threadIdx.x & 63;
    if (tile >= (size_t)(N / 16) * tiles_k) return;
    const int T = (int)(tile % tiles_k);
    const size_t n = tile / tiles_k * 16 + (lane & 15);
    uint32_t f[2][4], o[6];
    load_chunks24(codes + n * (K * 3 / 32) + 24 * T, lane >> 4, f);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int w = 0; w < 3; ++w) {
            uint32_t word = 0;
#pragma unroll
            for (int e = 0; e < 2; ++e) {
#pragma unroll
                for (int p = 0; p < 5; ++p) {
                    const int c = 2 * (5 * w + p) + e;
                    word |= ((f[u][c >> 3] >> (3 * (c & 7))) & 7u) << (1 + 3 * p + 16 * e);
                }
                word |= ((f[u][3] >> (3 * (6 + e) + w)) & 1u) << (16 * e);     // pair 15: bit w of codes 30 and 31
            }
            o[3 * u + w] = word;
        }
    store_tile6(out + tile * 384, lane, o);
    if (lane < 16) {
        const uint32_t s2 = *(const uint32_t*)(scales + n * (K / kGroup) + 2 * T), z2 = *(const uint32_t*)(zeros + n * (K / kGroup) + 2 * T);
        *(uint2_t*)(sz + native_sz_index((int)n, 2 * T, K)) = uint2_t{(s2 & 0xFFFFu) | (z2 << 16), (s2 >> 16) | (z2 & 0xFFFF0000u)};
    }
}

template <int KBITS>
__global__ void __launch_bounds__(256) vq_prepack_kernel(const uint32_t* __restrict__ indices, int N, int K,
                                                         uint32_t* __restrict__ out) {
    const size_t tile = (size_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int tiles_k = K / 256, lane = threadIdx.x & 63;
    if (tile >= (size_t)(N / 16) * tiles_k) return;
    const int T = (int)(tile % tiles_k);
    const size_t n = tile / tiles_k * 16 + (lane & 15);
    const uint32_t* row = indices + n * (K / 2 * KBITS / 32) + (KBITS == 8 ? 32 : 24) * T;
    if constexpr (KBITS == 8) {
        uint32_t o[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) o[i] = row[4 * i + (lane >> 4)];
        uint32_t* t = out + tile * 512;
        *(uint4_t*)(t + 4 * lane) = uint4_t{o[0], o[1], o[2], o[3]};
        *(uint4_t*)(t + 256 + 4 * lane) = uint4_t{o[4], o[5], o[6], o[7]};
    } else {
        uint32_t f[2][4], o[6];
        load_chunks24(row, lane >> 4, f);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int w = 0; w < 3; ++w) {
                uint32_t word = (f[u][3] >> (18 + 2 * w)) & 3u;                  // index 15: bits 2w, 2w + 1 into bits 0, 1
#pragma unroll
                for (int p = 0; p < 5; ++p) {
                    const int P = 5 * w + p;
                    word |= ((f[u][P >> 2] >> (6 * (P & 3))) & 63u) << (2 + 6 * p);
                }
                o[3 * u + w] = word;
            }
        store_tile6(out + tile * 384, lane, o);
    }
}

// ------------------------------------------------------------------ dequant

// Element (n, k) of Deq(W) in binary32, from either layout.  This is the definition the
// streaming and matrix-core kernels are checked against; it is written for clarity, not speed.
__device__ float deq_element(const MatDev& m, int n, int k) {
    const int K = m.K;
    if (m.fmt == FMT_SQ3) {
        uint32_t q;
        float s, z;
        int g = k / kGroup;
        if (m.layout == 0) {
            q = canon_field(m.codes + (size_t)n * (K * 3 / 32), 3, k);
            s = f16_bits_to_f32(m.aux[(size_t)n * (K / kGroup) + g]);
            z = f16_bits_to_f32(m.aux2[(size_t)n * (K / kGroup) + g]);
        } else {
            TilePos p = tile_pos(n & 15, k & 255);
            const uint32_t* tile = m.codes + ((size_t)(n >> 4) * (K / 256) + (k >> 8)) * 384;
            uint32_t w[3];
            for (int i = 0; i < 3; ++i) w[i] = tile[tile6_word(p.lane, 3 * p.u + i)];
            q = native_sq_field(w, p.c);
            size_t o = native_sz_index(n, g, K);
            s = f16_bits_to_f32(m.aux[o]);
            z = f16_bits_to_f32(m.aux[o + 1]);
        }
        return sq_deq(q, s, z);
    }
    const int kbits = m.fmt == FMT_VQ8 ? 8 : 6;
    uint32_t idx;
    if (m.layout == 0) {
        idx = canon_field(m.codes + (size_t)n * (K / 2 * kbits / 32), kbits, k >> 1);
    } else {
        TilePos p = tile_pos(n & 15, k & 255);
        int P = p.c >> 1;
        if (kbits == 8) {
            const uint32_t* tile = m.codes + ((size_t)(n >> 4) * (K / 256) + (k >> 8)) * 512;
            uint32_t w = tile[tile8_word(p.lane, 4 * p.u + (P >> 2))];
            idx = (w >> (8 * (P & 3))) & 255u;
        } else {
            const uint32_t* tile = m.codes + ((size_t)(n >> 4) * (K / 256) + (k >> 8)) * 384;
            uint32_t w[3];
            for (int i = 0; i < 3; ++i) w[i] = tile[tile6_word(p.lane, 3 * p.u + i)];
            idx = native_vq6_index(w, P);
        }
    }
    size_t cb = (size_t)(n / kBlock) * (K / kBlock) + (k / kBlock);
    return f16_bits_to_f32(m.aux[((cb << kbits) + idx) * 2 + (k & 1)]);
}

__global__ void dequant_kernel(MatDev m, void* __restrict__ out, int dt) {
    size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    size_t total = (size_t)m.N * m.K;
    if (gid >= total) return;
    int n = (int)(gid / m.K), k = (int)(gid % m.K);
    store_from_f32(out, gid, dt, deq_element(m, n, k));
}

static inline unsigned blocks_for(size_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

hipError_t launch_sq_prepack(const uint32_t* codes, const uint16_t* scales, const uint16_t* zeros,
                             int N, int K, uint32_t* codes_native, uint16_t* sz_native, hipStream_t s) {
    const size_t tiles = (size_t)(N / 16) * (K / 256);
    hipLaunchKernelGGL(sq_prepack_kernel, dim3(blocks_for(tiles, 4)), dim3(256), 0, s, codes, scales, zeros, N, K,
                       codes_native, sz_native);
    return hipGetLastError();
}

hipError_t launch_vq_prepack(const uint32_t* indices, int N, int K, int kbits, uint32_t* out,
                             hipStream_t s) {
    const dim3 grid(blocks_for((size_t)(N / 16) * (K / 256), 4));
    if (kbits == 6) hipLaunchKernelGGL(vq_prepack_kernel<6>, grid, dim3(256), 0, s, indices, N, K, out);
    else hipLaunchKernelGGL(vq_prepack_kernel<8>, grid, dim3(256), 0, s, indices, N, K, out);
    return hipGetLastError();
}

hipError_t launch_dequant(const MatDev& m, void* w_out, int w_dtype, hipStream_t s) {
    size_t total = (size_t)m.N * m.K;
    hipLaunchKernelGGL(dequant_kernel, dim3(blocks_for(total, 256)), dim3(256), 0, s, m, w_out, w_dtype);
    return hipGetLastError();
}

// ------------------------------------------------------------------ reference GEMM

// y[m][n] = sum_k Deq(W)[n][k] * x[m][k], binary32 accumulate.  One block per (n, 8 rows of x);
// each thread strides over k, then the block reduces.  Works for both layouts and any M.
constexpr int kRefRows = 8;
__global__ void __launch_bounds__(256) ref_gemm_kernel(MatDev m, int M, int xdt, int ydt) {
    __shared__ float red[kRefRows][256];
    int n = blockIdx.x, m0 = blockIdx.y * kRefRows;
    float acc[kRefRows];
    for (int i = 0; i < kRefRows; ++i) acc[i] = 0.f;
    for (int k = threadIdx.x; k < m.K; k += 256) {
        float w = deq_element(m, n, k);
        for (int i = 0; i < kRefRows; ++i)
            if (m0 + i < M) acc[i] = fmaf(w, load_as_f32(m.x, (size_t)(m0 + i) * m.K + k, xdt), acc[i]);
    }
    for (int i = 0; i < kRefRows; ++i) red[i][threadIdx.x] = acc[i];
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s)
            for (int i = 0; i < kRefRows; ++i) red[i][threadIdx.x] += red[i][threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x < kRefRows && m0 + (int)threadIdx.x < M)
        store_from_f32(m.y, (size_t)(m0 + threadIdx.x) * m.N + n, ydt, red[threadIdx.x][0]);
}

hipError_t launch_ref_gemm(const MatDev& m, int M, int x_dtype, int y_dtype, hipStream_t s) {
    // grid.y is limited to 65535 blocks: M <= 524280 rows per launch is far beyond any use here.
    hipLaunchKernelGGL(ref_gemm_kernel, dim3(m.N, (M + kRefRows - 1) / kRefRows), dim3(256), 0, s, m, M,
                       x_dtype, y_dtype);
    return hipGetLastError();
}

}  // namespace rwkvq

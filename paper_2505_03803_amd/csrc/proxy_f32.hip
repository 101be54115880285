// The coarse-to-fine proxy of Sec. 3.1 for weight matrices stored as binary32: the recipe as the
// paper states it.  The flattened weights are sorted in ascending order ("Coarse-grained Proxy"),
// the intervals between neighbours are normalised (Eqs. "interval", "interval_norm"), and the
// entropy and the central moments of the normalised intervals give P_c and P_f (Eqs. "ie",
// "coarse_proxy", "fine_proxy").  Sixteen-bit matrices take the shortcut of proxy.hip (the set of
// occurring bit patterns); binary32 matrices of less than kSetMinCount weights are really
// sorted (larger ones: below, "partition and sets of values"):
//
//   * keys: the order-preserving map of the binary32 patterns to unsigned integers;
//   * least-significant-digit radix sort, four passes of 8 bits, each pass three steps:
//       sort_hist_kernel     per tile of 4096 keys, how many keys have each digit value;
//       sort_scan_kernel     running sums of those counts, digit-major (the position of every
//                            (digit, tile) run in the output);
//       sort_scatter_kernel  every key to its position: its rank among the keys of its digit within
//                            the tile comes from wavefront ballots (no atomics, the order of equal
//                            digits is kept, which a least-significant-digit sort needs), the tile is
//                            reordered in LDS so that runs leave as contiguous stores;
//   * gap_sum_kernel / gap_final_kernel: the sums over the intervals in binary64, in a fixed order
//     (a partial sum per 16384 intervals, then one workgroup adds the partial sums), with
//     t_i = G_i / mean(G) as in proxy.hip:  P_c = (1/n) sum t ln t,  v_k |M_k| = |sum (t-1)^k| / (n k (k-1)).
//
// Matrices of a call share the buffers; large ones are counted and concluded several at a time (SetGroup).
#include "common.h"
#include "proxy_ranges.h"
#include "../../include/rwkvq.h"

#include <algorithm>

namespace rwkvq {

constexpr int kSortThreads = 256;
constexpr int kSortRounds = 16;                              // keys per thread
constexpr int kSortTile = kSortThreads * kSortRounds;        // 4096 keys per workgroup
constexpr int kDigits = 256;
constexpr int kGapThreads = 256;
constexpr int kGapPerThread = 64;
constexpr int kGapTile = kGapThreads * kGapPerThread;        // 16384 intervals per workgroup
constexpr int kGapMaxTerms = 8;
constexpr int kGapSums = kGapMaxTerms + 1;                   // [0] = sum t ln t, [k] = sum (t-1)^k

__device__ __forceinline__ uint32_t f32_key(uint32_t bits) {      // a < b as numbers  =>  key(a) < key(b); -0 sorts below +0
    return (bits & 0x80000000u) ? ~bits : (bits | 0x80000000u);
}
__device__ __forceinline__ double key_f64(uint32_t key) {
    const uint32_t bits = (key & 0x80000000u) ? (key & 0x7FFFFFFFu) : ~key;
    return (double)__builtin_bit_cast(float, bits);
}

// Lanes of the wavefront whose 8-bit digit equals this lane's (among the lanes with valid = true).
__device__ __forceinline__ unsigned long long same_digit_lanes(uint32_t digit, bool valid) {
    unsigned long long m = __builtin_amdgcn_ballot_w64(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const bool bit = (digit >> b) & 1u;
        const unsigned long long set = __builtin_amdgcn_ballot_w64(bit);
        m &= bit ? set : ~set;
    }
    return m;
}
__device__ __forceinline__ unsigned long long lanes_below(int lane) { return (1ull << lane) - 1ull; }

// LDS traffic of one wavefront is served in issue order; the fences keep the compiler from moving
// a lane's read of a counter past the leader's update of it.
__device__ __forceinline__ void wave_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// counts[digit * n_tiles + tile] = number of keys of the tile whose digit (bits shift .. shift+7) has that value.
// FIRST: the input holds binary32 patterns, not keys yet.
template <bool FIRST>
__global__ void __launch_bounds__(kSortThreads) sort_hist_kernel(const uint32_t* __restrict__ in, uint32_t n, int shift,
                                                                 uint32_t* __restrict__ counts, uint32_t n_tiles) {
    __shared__ uint32_t h[kDigits];
    const int tid = threadIdx.x, lane = tid & 63;
    h[tid] = 0u;
    __syncthreads();
    const size_t base = (size_t)blockIdx.x * kSortTile;
#pragma unroll 4
    for (int r = 0; r < kSortRounds; ++r) {
        const size_t i = base + (size_t)r * kSortThreads + tid;
        const bool valid = i < n;
        uint32_t k = valid ? in[i] : 0u;
        if (FIRST) k = f32_key(k);
        const uint32_t d = (k >> shift) & 255u;
        // Counting needs no order: one LDS addition per key, except that a wavefront whose valid lanes all hold
        // the same digit (the low bytes of binary32 patterns that came from 16-bit values, a run of equal
        // weights) adds once - 64 additions to one address would be served one after the other.
        const unsigned long long live = __builtin_amdgcn_ballot_w64(valid);
        const uint32_t d0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)d);      // digit of the first valid lane
        const unsigned long long same = __builtin_amdgcn_ballot_w64(valid && d == d0);
        if (same == live) {
            if (valid && (live & lanes_below(lane)) == 0ull) atomicAdd(&h[d], (uint32_t)__builtin_popcountll(live));
        } else if (valid) {
            atomicAdd(&h[d], 1u);
        }
    }
    __syncthreads();
    counts[(size_t)tid * n_tiles + blockIdx.x] = h[tid];
}

// In place: counts[d][t] <- number of keys with digit d in tiles before t; totals[d] <- keys with digit d.
__global__ void __launch_bounds__(256) sort_scan_rows_kernel(uint32_t* __restrict__ counts, uint32_t n_tiles,
                                                             uint32_t* __restrict__ totals) {
    __shared__ uint32_t part[256];
    uint32_t* row = counts + (size_t)blockIdx.x * n_tiles;
    const int tid = threadIdx.x;
    const uint32_t per = (n_tiles + 255u) / 256u;
    const uint32_t lo = min(n_tiles, tid * per), hi = min(n_tiles, lo + per);
    uint32_t s = 0;
    for (uint32_t i = lo; i < hi; ++i) s += row[i];
    part[tid] = s;
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {                  // inclusive running sum of the 256 segment sums
        const uint32_t add = tid >= off ? part[tid - off] : 0u;
        __syncthreads();
        part[tid] += add;
        __syncthreads();
    }
    uint32_t run = tid ? part[tid - 1] : 0u;
    for (uint32_t i = lo; i < hi; ++i) { const uint32_t c = row[i]; row[i] = run; run += c; }
    if (tid == 255) totals[blockIdx.x] = part[255];
}

// totals[d] <- number of keys with a smaller digit.
__global__ void __launch_bounds__(256) sort_scan_totals_kernel(uint32_t* __restrict__ totals) {
    __shared__ uint32_t part[256];
    const int tid = threadIdx.x;
    const uint32_t mine = totals[tid];
    part[tid] = mine;
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {
        const uint32_t add = tid >= off ? part[tid - off] : 0u;
        __syncthreads();
        part[tid] += add;
        __syncthreads();
    }
    totals[tid] = part[tid] - mine;
}

// Every key of the tile to out[position of its (digit, tile) run + its rank in the run].  Order inside a tile:
// wavefront w owns keys 1024 w .. 1024 w + 1023, in rounds of 64.
template <bool FIRST>
__global__ void __launch_bounds__(kSortThreads) sort_scatter_kernel(const uint32_t* __restrict__ in, uint32_t* __restrict__ out,
                                                                    uint32_t n, int shift, const uint32_t* __restrict__ before,
                                                                    const uint32_t* __restrict__ smaller, uint32_t n_tiles) {
    __shared__ uint32_t seen[4][kDigits];     // per wavefront: keys of each digit so far; later: keys of the digit in earlier wavefronts
    __shared__ uint32_t start[kDigits];       // first slot of each digit in the tile's sorted order
    __shared__ uint32_t run_pos[kDigits];     // position in `out` of the tile's first key of each digit
    __shared__ uint32_t sorted[kSortTile];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int w = 0; w < 4; ++w) seen[w][tid] = 0u;
    run_pos[tid] = smaller[tid] + before[(size_t)tid * n_tiles + blockIdx.x];
    __syncthreads();
    const size_t base = (size_t)blockIdx.x * kSortTile + (size_t)wave * (kSortTile / 4);
    uint32_t key[kSortRounds], rank[kSortRounds];
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) {
        const size_t i = base + (size_t)r * 64 + lane;
        const bool valid = i < n;
        uint32_t k = valid ? in[i] : 0xFFFFFFFFu;
        if (FIRST && valid) k = f32_key(k);
        const uint32_t d = (k >> shift) & 255u;
        const unsigned long long m = same_digit_lanes(d, valid);
        const uint32_t below = (uint32_t)__builtin_popcountll(m & lanes_below(lane));
        const uint32_t old = seen[wave][d];
        wave_order();
        if (valid && below == 0u) seen[wave][d] = old + (uint32_t)__builtin_popcountll(m);
        wave_order();
        key[r] = k;
        rank[r] = old + below;                 // rank among the wavefront's keys of this digit
    }
    __syncthreads();
    {   // digit t: keys per wavefront -> keys in earlier wavefronts; tile totals -> first slots
        const uint32_t c0 = seen[0][tid], c1 = seen[1][tid], c2 = seen[2][tid], c3 = seen[3][tid];
        seen[0][tid] = 0u; seen[1][tid] = c0; seen[2][tid] = c0 + c1; seen[3][tid] = c0 + c1 + c2;
        const uint32_t total = c0 + c1 + c2 + c3;
        start[tid] = total;
        __syncthreads();
        for (int off = 1; off < 256; off <<= 1) {
            const uint32_t add = tid >= off ? start[tid - off] : 0u;
            __syncthreads();
            start[tid] += add;
            __syncthreads();
        }
        const uint32_t incl = start[tid];
        __syncthreads();
        start[tid] = incl - total;
        __syncthreads();
    }
    const size_t tile_base = (size_t)blockIdx.x * kSortTile;
    const uint32_t in_tile = (uint32_t)(n - tile_base < (size_t)kSortTile ? n - tile_base : (size_t)kSortTile);
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) {
        const size_t i = base + (size_t)r * 64 + lane;
        if (i < n) {
            const uint32_t d = (key[r] >> shift) & 255u;
            sorted[start[d] + seen[wave][d] + rank[r]] = key[r];
        }
    }
    __syncthreads();
    for (uint32_t s = tid; s < in_tile; s += kSortThreads) {
        const uint32_t k = sorted[s];
        const uint32_t d = (k >> shift) & 255u;
        out[(size_t)run_pos[d] + (s - start[d])] = k;
    }
}

// Partial sums over the intervals of one tile: partial[tile][0] = sum t ln t, [k] = sum (t - 1)^k, k = 2 .. terms.
__global__ void __launch_bounds__(kGapThreads) gap_sum_kernel(const uint32_t* __restrict__ keys, uint32_t count, int terms,
                                                              double* __restrict__ partial) {
    __shared__ double red[kGapThreads / 64][kGapSums];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t n = count - 1u;                                   // intervals
    const double span = key_f64(keys[count - 1]) - key_f64(keys[0]);
    double s[kGapSums];
#pragma unroll
    for (int k = 0; k < kGapSums; ++k) s[k] = 0.0;
    if (span > 0.0) {
        const double inv_mean = (double)n / span;
        const size_t base = (size_t)blockIdx.x * kGapTile;
        for (int j = 0; j < kGapPerThread; ++j) {
            const size_t i = base + (size_t)j * kGapThreads + tid;
            if (i < n) {
                const double g = key_f64(keys[i + 1]) - key_f64(keys[i]);    // exact: both are binary32 values
                const double t = g * inv_mean;
                if (t > 0.0) s[0] += t * log(t);
                const double u = t - 1.0;
                double p = u;
                for (int k = 2; k <= terms; ++k) { p *= u; s[k] += p; }
            }
        }
    }
#pragma unroll
    for (int k = 0; k < kGapSums; ++k) {
        double v = s[k];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
        if (lane == 0) red[wave][k] = v;
    }
    __syncthreads();
    if (tid < kGapSums) {
        double v = 0.0;
        for (int w = 0; w < kGapThreads / 64; ++w) v += red[w][tid];
        partial[(size_t)blockIdx.x * kGapSums + tid] = v;
    }
}

// One workgroup: the partial sums in tile order, then P_c, P_f and the decision of Eq. "multi_scale_proxy".
__global__ void __launch_bounds__(256) gap_final_kernel(const uint32_t* __restrict__ keys, uint32_t count, int terms,
                                                        const double* __restrict__ partial, uint32_t n_tiles, double tau_c,
                                                        double tau_f, double* __restrict__ out, int32_t* __restrict__ phi) {
    __shared__ double red[256][kGapSums];
    const int tid = threadIdx.x;
    double s[kGapSums];
#pragma unroll
    for (int k = 0; k < kGapSums; ++k) s[k] = 0.0;
    const uint32_t per = (n_tiles + 255u) / 256u;
    const uint32_t lo = min(n_tiles, tid * per), hi = min(n_tiles, lo + per);
    for (uint32_t t = lo; t < hi; ++t)
#pragma unroll
        for (int k = 0; k < kGapSums; ++k) s[k] += partial[(size_t)t * kGapSums + k];
#pragma unroll
    for (int k = 0; k < kGapSums; ++k) red[tid][k] = s[k];
    __syncthreads();
    if (tid == 0) {
        double tot[kGapSums];
        for (int k = 0; k < kGapSums; ++k) { tot[k] = 0.0; for (int i = 0; i < 256; ++i) tot[k] += red[i][k]; }
        const double n = (double)(count - 1u);
        const double span = key_f64(keys[count - 1]) - key_f64(keys[0]);
        double Pc = 0.0, Pf = 0.0;
        if (span > 0.0) {                        // a constant matrix has no intervals to normalise: both proxies 0
            Pc = tot[0] / n;
            for (int k = 2; k <= terms; ++k) Pf += fabs(tot[k]) / (n * (double)(k * (k - 1)));
        }
        out[0] = Pc;
        out[1] = Pf;
        *phi = (Pc < tau_c && Pf < tau_f) ? 1 : 0;
    }
}

// ------------------------------------------------------------------ large matrices: partition and sets of values
//
// From kSetMinCount weights on nothing is sorted through memory.  The sums need the distinct values in order and the number of
// equal neighbours, not the sorted sequence:
//
//   * set_count_kernel      8192 bins, a bin being the upper 13 bits of the key (sign, exponent, four bits of fraction): counts
//                           per workgroup of a contiguous range in LDS, then one reservation per workgroup and bin;
//   * set_plan_kernel       where each bin starts.  Bins of more than 1024 keys ("hot", of near-normal weights the ones
//                           within some octaves of the deviation) stand behind the others, in groups of at most 2047 keys;
//   * set_partition_kernel  every key to its bin: position = start + reservation + an LDS counter per bin.  The order inside a
//                           bin does not matter (and is not fixed), so no ranks are needed;
//   * set_sum_kernel        a hot bin is 2^19 patterns of one sign and exponent: a bitmap of 64 KB in LDS.  Intervals are
//                           distances of set bits times the exponent's unit, exact, and counted by distance.  A bin of more
//                           than 131072 keys and a 64th of all (piece_solo) is read by several workgroups that join their bitmaps in
//                           memory, and the last to finish sums.  A group of small bins is sorted (sort_group);
//   * set_final_kernel      intervals between bins, intervals of zero (t - 1 = -1), the partial sums in a fixed order, P_c, P_f.
//
// The sums depend only on sets and counts, so the result is the same on every run although the partition's order is not.
// Bound: the partition by memory (14336 x 4096: 470 MB in 110 us, 4.3 TB/s); the count by reading (4.9 TB/s); the sums by the LDS, which
// takes 17 clocks for 64 atomic operations: 626000 keys of the fullest bin of 14336 x 4096 are set in 82 us, by one compute unit, so
// that matrices share launches (launch_sets).  Bins of 2^17 patterns, of which the sums are better balanced (87 us instead of 105 there),
// cost the partition 40 us more: runs of a quarter of the length, and a table of ranks in LDS where this one is addressed by the bin.
// Between the two, 2^18: 142 and 89 us.  Four workgroups for a full bin, of which each reads all keys and keeps a quarter of the patterns, take
// as long per atomic operation and were slower (4096 x 4096 122 -> 152 us).
// Measured (us; radix sort, bins of 2^17 -> here): 768 x 768 157, 90 -> 55, 1024 x 1024 163, 95 -> 56, 4096 x 4096 502, 138 -> 122,
// 14336 x 4096 1957, 350 -> 307; the eight matrices of a layer of the 7B shapes 7060, 1320 -> 1040, of d = 1024 598 -> 331.
// 2^24 weights (bins of 2^17 -> here): values of bfloat16 181 -> 147, uniform in [-1/2, 1/2) 132 -> 131, in [0, 1) 125 -> 129, all equal
// 139 -> 125, half zero 187 -> 160, 2^(uniform from -40 to 20) 207 -> 134; bit patterns at random 569 -> 210 (2^20: 122 -> 71).  14336 x 4096:
// uniform 325 -> 322 and 325 -> 304, values of bfloat16 536 -> 414, half zero 504 -> 419.  Below kSetMinCount the sort.
constexpr uint32_t kSetMinCount = 1u << 19;                  // (the line: the workspace, sized for the sort, holds the tables)
constexpr int kBins = 8192, kBinShift = 19;
constexpr uint32_t kHot = 1024;                              // keys of a bin that is not hot, and of a group's bins but the last
constexpr int kBitmapWords = 1 << (kBinShift - 5);           // 16384
constexpr int kSetThreads = 1024;
constexpr int kSetRow = kGapSums + 1;                        // partial sums and the number of intervals above zero
constexpr int kSumThreads = 512, kSumWorkgroups = 512;       // (two workgroups per compute unit; one of 1024 threads: a call of a layer 85 us more)
constexpr int kTable = 3072;                                 // distances that are counted: six per thread, 12 KB beside the bitmap
constexpr uint32_t kDense = 1u << (kBinShift - 3);

struct SetHead { uint32_t min_key, max_key, groups, pieces, joints, pad; };
// One matrix of a call.
struct SetBuffers {
    const uint32_t* in;      // the weights
    uint32_t count, wgs;     // of them; counting (and partitioning) workgroups
    uint32_t solo, joint_max;
    double* out;             // P_c, P_f
    int32_t* phi;
    uint32_t* keys;          // partitioned: groups of small bins, then the hot bins, each in bin order; shared by launches
    uint32_t* reserved;      // [workgroup][bin]: keys of the bin reserved before
    SetHead* head;
    uint32_t* counts;        // [bin]
    double* logs;            // [kTable]: logarithms of 1, 2, ..
    uint32_t* least;         // [counting workgroup]: its smallest and largest key
    uint32_t* most;
    uint32_t* start;         // [bin]: position of the bin in keys
    uint32_t* group_from;    // [group + 1]: position of the group's first key
    uint32_t* bin_min;       // [bin], of occupied bins
    uint32_t* bin_max;
    uint4_t* piece;          // [piece]: bin, first position, keys, joint bitmap of a bin in several pieces
    uint32_t* done;          // [joint]: pieces finished
    uint32_t* joint;         // [joint][kBitmapWords]
    double* sums;            // [workgroups of set_sum_kernel, then joint bins][kSetRow]
};
// Matrices that are cleared, counted, planned and concluded in one launch each: four launches of 5, 15 and 13 us for one workgroup's
// work (and the ends of the counts) once per group instead of once per matrix.
constexpr int kSetGroup = 8;
struct SetGroup { SetBuffers b[kSetGroup]; };

static size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }
static size_t set_key_bytes(uint32_t count) { return align256((size_t)count * 4); }
// A matrix's own buffers from `base` on; returns their size.
static size_t set_tables(SetBuffers& b, char* base, uint32_t count, uint32_t range = kCountRange) {
    size_t o = 0;
    auto take = [&](size_t bytes) { char* p = base + o; o += align256(bytes); return p; };
    b.count = count; b.wgs = set_workgroups(count, range); b.solo = piece_solo(count); b.joint_max = piece_joint_max(count);
    b.reserved = (uint32_t*)take((size_t)b.wgs * kBins * 4);
    b.head = (SetHead*)take(sizeof(SetHead));
    b.counts = (uint32_t*)take(kBins * 4);
    b.logs = (double*)take(kTable * 8);
    b.least = (uint32_t*)take(256 * 4);
    b.most = (uint32_t*)take(256 * 4);
    b.start = (uint32_t*)take(kBins * 4);
    b.group_from = (uint32_t*)take(((size_t)count / kHot + 2) * 4);
    b.bin_min = (uint32_t*)take(kBins * 4);
    b.bin_max = (uint32_t*)take(kBins * 4);
    b.piece = (uint4_t*)take(((size_t)count / kHot + count / kPiece) * 16);
    b.done = (uint32_t*)take((size_t)b.joint_max * 4);
    b.joint = (uint32_t*)take((size_t)b.joint_max * kBitmapWords * 4);
    b.sums = (double*)take((size_t)(kSumWorkgroups + b.joint_max) * kSetRow * 8);
    return o;
}

__global__ void __launch_bounds__(256) set_clear_kernel(SetGroup g) {
    const SetBuffers& b = g.b[blockIdx.y];
    const uint32_t i = blockIdx.x * 256u + threadIdx.x, step = gridDim.x * 256u;
    for (uint32_t j = i; j < (uint32_t)kBins; j += step) b.counts[j] = 0u;
    for (uint32_t j = i; j < b.joint_max; j += step) b.done[j] = 0u;
    for (uint32_t j = i; j < (uint32_t)kTable; j += step) b.logs[j] = j ? log((double)j) : 0.0;
}

// Inclusive running sum over the lanes of the wavefront.
__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, true);     // row_shr 1, 2, 4, 8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);    // row_bcast 15 into rows 1 and 3
    return v + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);   // row_bcast 31 into rows 2 and 3
}

// Applies f to every pattern of the range, four loads of 16 bytes in flight per thread.
template <class F>
__device__ __forceinline__ void for_quads(const uint32_t* __restrict__ in, const SetRange& r, F f) {
    const uint4_t* q = (const uint4_t*)(in + r.lo);
    uint32_t i = threadIdx.x;
    for (; i + 3u * kSetThreads < r.quads; i += 4u * kSetThreads) {
        uint4_t v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = q[i + j * kSetThreads];
#pragma unroll
        for (int j = 0; j < 4; ++j) { f(v[j].x); f(v[j].y); f(v[j].z); f(v[j].w); }
    }
    for (; i < r.quads; i += kSetThreads) { const uint4_t v = q[i]; f(v.x); f(v.y); f(v.z); f(v.w); }
    if (threadIdx.x < r.rest) f(in[r.tail(threadIdx.x)]);
}

// Adds one to counter[bin] and gives its value before.  A wavefront whose lanes all hold one bin (equal weights) adds once.
__device__ __forceinline__ uint32_t count_bin(uint32_t* counter, uint32_t bin) {
    const unsigned long long live = __builtin_amdgcn_ballot_w64(true);
    const uint32_t b0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)bin);
    if (__builtin_amdgcn_ballot_w64(bin == b0) == live) {
        const uint32_t below = (uint32_t)__builtin_popcountll(live & lanes_below(threadIdx.x & 63));
        uint32_t old = 0u;
        if (below == 0u) old = atomicAdd(&counter[bin], (uint32_t)__builtin_popcountll(live));
        return (uint32_t)__builtin_amdgcn_readfirstlane((int)old) + below;
    }
    return atomicAdd(&counter[bin], 1u);
}

__global__ void __launch_bounds__(kSetThreads) set_count_kernel(SetGroup g) {
    extern __shared__ uint32_t h[];                              // [kBins]
    const SetBuffers& b = g.b[blockIdx.y];
    if (blockIdx.x >= b.wgs) return;
    const int tid = threadIdx.x;
    for (int j = tid; j < kBins / 4; j += kSetThreads) ((uint4_t*)h)[j] = uint4_t{0u, 0u, 0u, 0u};
    __syncthreads();
    uint32_t least = 0xFFFFFFFFu, most = 0u;
    for_quads(b.in, set_range(b.count, blockIdx.x, b.wgs), [&](uint32_t bits) {
        const uint32_t k = f32_key(bits);
        least = min(least, k); most = max(most, k);
        count_bin(h, k >> kBinShift);
    });
#pragma unroll
    for (int off = 32; off; off >>= 1) {
        least = min(least, (uint32_t)__shfl_xor((int)least, off, 64));
        most = max(most, (uint32_t)__shfl_xor((int)most, off, 64));
    }
    __shared__ uint32_t wave_least[kSetThreads / 64], wave_most[kSetThreads / 64];
    if ((tid & 63) == 0) { wave_least[tid >> 6] = least; wave_most[tid >> 6] = most; }
    __syncthreads();
    if (tid == 0) {                                              // (one address for all wavefronts: 90 us of additions in a row)
        for (int w = 0; w < kSetThreads / 64; ++w) { least = min(least, wave_least[w]); most = max(most, wave_most[w]); }
        b.least[blockIdx.x] = least;
        b.most[blockIdx.x] = most;
    }
    uint32_t* mine = b.reserved + (size_t)blockIdx.x * kBins;
    // eight reservations in flight per thread, each workgroup from another bin on
    constexpr int kOwn = kBins / kSetThreads;
    uint32_t c[kOwn], got[kOwn];
    auto bin = [&](int r) { return (uint32_t)(tid + r * kSetThreads + kBins / 256 * (int)blockIdx.x) & (kBins - 1); };
#pragma unroll
    for (int r = 0; r < kOwn; ++r) c[r] = h[bin(r)];
#pragma unroll
    for (int r = 0; r < kOwn; ++r) if (c[r]) got[r] = atomicAdd(&b.counts[bin(r)], c[r]);
#pragma unroll
    for (int r = 0; r < kOwn; ++r) if (c[r]) mine[bin(r)] = got[r];
}

// One workgroup per matrix; a thread takes kOwn consecutive bins.
__global__ void __launch_bounds__(kSetThreads) set_plan_kernel(SetGroup g) {
    const SetBuffers& b = g.b[blockIdx.x];
    const uint32_t wgs = b.wgs, solo = b.solo;
    __shared__ uint32_t wave_sum[kSetThreads / 64][5];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int kOwn = kBins / kSetThreads;
    uint32_t c[kOwn];
#pragma unroll
    for (int j = 0; j < kOwn / 4; ++j) {
        const uint4_t v = ((const uint4_t*)b.counts)[kOwn / 4 * tid + j];
        c[4 * j] = v.x; c[4 * j + 1] = v.y; c[4 * j + 2] = v.z; c[4 * j + 3] = v.w;
    }
    // keys in small bins, keys in hot bins, pieces of the fullest bins (they come first), hot bins of several pieces, other pieces
    uint32_t own[5] = {0u, 0u, 0u, 0u, 0u};
    const uint32_t full = b.count / 512u;
#pragma unroll
    for (int j = 0; j < kOwn; ++j) {
        if (c[j] <= kHot) own[0] += c[j];
        else { own[1] += c[j]; own[c[j] > full ? 2 : 4] += piece_count(c[j], solo); own[3] += c[j] > solo ? 1u : 0u; }
    }
    uint32_t run[5], total[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        uint32_t v = own[i];
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) { const uint32_t a = (uint32_t)__shfl_up((int)v, off, 64); if (lane >= off) v += a; }
        if (lane == 63) wave_sum[wave][i] = v;
        run[i] = v - own[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        total[i] = 0u;
#pragma unroll
        for (int w = 0; w < kSetThreads / 64; ++w) { if (w < wave) run[i] += wave_sum[w][i]; total[i] += wave_sum[w][i]; }
        __builtin_amdgcn_sched_barrier(0);        // sixteen at a time
    }
#pragma unroll
    for (int q = 0; q < kOwn / 4; ++q) {
        uint32_t at[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t n = c[4 * q + j];
            if (n <= kHot) {
                at[j] = run[0];
                run[0] += n;
                // a group begins with the first bin at or behind a multiple of kHot (a bin holds no more than that)
                if (run[0] / kHot != at[j] / kHot) b.group_from[run[0] / kHot] = run[0];
            } else {
                at[j] = total[0] + run[1];
                for (uint32_t f = 0u; f < n; f += piece_keys(n, f, solo))
                    b.piece[n > full ? run[2]++ : total[2] + run[4]++] = uint4_t{(uint32_t)(kOwn * tid + 4 * q + j), at[j] + f, piece_keys(n, f, solo), n > solo ? run[3] : 0xFFFFFFFFu};
                run[1] += n; run[3] += n > solo ? 1u : 0u;
            }
        }
        ((uint4_t*)b.start)[kOwn / 4 * tid + q] = uint4_t{at[0], at[1], at[2], at[3]};
    }
    if (wave == 0) {
        uint32_t least = 0xFFFFFFFFu, most = 0u;
        for (uint32_t i = lane; i < wgs; i += 64u) { least = min(least, b.least[i]); most = max(most, b.most[i]); }
#pragma unroll
        for (int off = 32; off; off >>= 1) {
            least = min(least, (uint32_t)__shfl_xor((int)least, off, 64));
            most = max(most, (uint32_t)__shfl_xor((int)most, off, 64));
        }
        if (lane == 0) { b.head->min_key = least; b.head->max_key = most; }
    }
    if (tid == 0) {
        const uint32_t groups = total[0] ? (total[0] - 1u) / kHot + 1u : 0u;
        b.group_from[0] = 0u;
        if (groups) b.group_from[groups] = total[0];
        b.head->groups = groups; b.head->pieces = total[2] + total[4]; b.head->joints = total[3];
    }
}

// Stored where it is met, a key is a request of four bytes to a line of its own: 16384 keys at a time are brought into the
// order of their bins in LDS first, so that a wavefront's store meets runs; a thread keeps the positions of eight bins in registers.
// What bounds it: memory (see above); beside it the LDS, five accesses per key, 76 of 110 us at 14336 x 4096.
constexpr int kTileKeys = 16 * kSetThreads;
__global__ void __launch_bounds__(kSetThreads) set_partition_kernel(SetGroup g) {
    const SetBuffers& b = g.b[blockIdx.y];
    if (blockIdx.x >= b.wgs) return;
    extern __shared__ uint32_t first[];                          // [kBins]: keys of the bin in the tile, then its first place
    constexpr int kOwn = kBins / kSetThreads, kQuads = kTileKeys / kSetThreads / 4;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t* __restrict__ in = b.in;
    const uint32_t* mine = b.reserved + (size_t)blockIdx.x * kBins;
    uint32_t* out = b.keys;
    const SetRange r = set_range(b.count, blockIdx.x, b.wgs);
    {                                                            // the joint bitmaps that the sums will need
        const uint32_t quads = b.head->joints * (uint32_t)(kBitmapWords / 4);
        for (uint32_t j = blockIdx.x * (uint32_t)kSetThreads + tid; j < quads; j += b.wgs * (uint32_t)kSetThreads)
            ((uint4_t*)b.joint)[j] = uint4_t{0u, 0u, 0u, 0u};
    }
    uint32_t* const to = first + kBins;                          // [kBins]: position in `keys` of the bin's first key, less its first place
    uint32_t* const tile = to + kBins;                           // [kTileKeys]
    uint32_t* const wave_sum = tile + kTileKeys;                 // [kSetThreads / 64]
    uint32_t pos[kOwn];                                          // (bins that the range does not hold: never used)
#pragma unroll
    for (int i = 0; i < kOwn; i += 4) {
        const uint4_t p = *(const uint4_t*)(b.start + kOwn * tid + i) + *(const uint4_t*)(mine + kOwn * tid + i);
        pos[i] = p.x; pos[i + 1] = p.y; pos[i + 2] = p.z; pos[i + 3] = p.w;
    }
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < kOwn; i += 4) *(uint4_t*)(first + kOwn * tid + i) = uint4_t{0u, 0u, 0u, 0u};
    };
    clear();
    const uint32_t quads = r.quads;
    const uint4_t* src = (const uint4_t*)(in + r.lo);
    uint4_t v[kQuads];
    auto fetch = [&](uint32_t base) {
#pragma unroll
        for (int q = 0; q < kQuads; ++q) {
            const uint32_t i = base + (uint32_t)(tid + q * kSetThreads);
            v[q] = i < quads ? src[i] : uint4_t{0u, 0u, 0u, 0u};
        }
    };
    fetch(0u);
    __syncthreads();
#pragma unroll 1
    for (uint32_t base = 0u; base < quads; base += kTileKeys / 4) {
        const uint32_t in_tile = 4u * min(quads - base, (uint32_t)(kTileKeys / 4));
        uint32_t key[4 * kQuads], at[4 * kQuads];                // at: rank among the tile's keys of the bin
#pragma unroll
        for (int q = 0; q < kQuads; ++q) {
            const uint32_t k[4] = {v[q].x, v[q].y, v[q].z, v[q].w};
#pragma unroll
            for (int j = 0; j < 4; ++j) { key[4 * q + j] = f32_key(k[j]); at[4 * q + j] = 0u; }
            if (4u * (uint32_t)(tid + q * kSetThreads) < in_tile)
#pragma unroll
                for (int j = 0; j < 4; ++j) at[4 * q + j] = count_bin(first, key[4 * q + j] >> kBinShift);
        }
        fetch(base + kTileKeys / 4);
        __syncthreads();
        uint32_t n[kOwn], own = 0u;
#pragma unroll
        for (int i = 0; i < kOwn; i += 4) {
            const uint4_t c = *(const uint4_t*)(first + kOwn * tid + i);
            n[i] = c.x; n[i + 1] = c.y; n[i + 2] = c.z; n[i + 3] = c.w;
            own += c.x + c.y + c.z + c.w;
        }
        uint32_t place = wave_scan(own);
        if (lane == 63) wave_sum[wave] = place;
        place -= own;
        __syncthreads();
        uint32_t before[kSetThreads / 64];
#pragma unroll
        for (int w = 0; w < kSetThreads / 64; ++w) before[w] = wave_sum[w];
#pragma unroll
        for (int w = 0; w < kSetThreads / 64; ++w) place += w < wave ? before[w] : 0u;
#pragma unroll
        for (int i = 0; i < kOwn; i += 4) {
            uint32_t f[4], t[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) { f[j] = place; t[j] = pos[i + j] - place; pos[i + j] += n[i + j]; place += n[i + j]; }
            *(uint4_t*)(first + kOwn * tid + i) = uint4_t{f[0], f[1], f[2], f[3]};
            *(uint4_t*)(to + kOwn * tid + i) = uint4_t{t[0], t[1], t[2], t[3]};
        }
        __syncthreads();
        // all look-ups of a thread before its first store, here and below: a trip to the LDS for all of them, not for each
#pragma unroll
        for (int j = 0; j < 4 * kQuads; ++j) at[j] += first[key[j] >> kBinShift];
#pragma unroll
        for (int q = 0; q < kQuads; ++q)
            if (4u * (uint32_t)(tid + q * kSetThreads) < in_tile)
#pragma unroll
                for (int j = 0; j < 4; ++j) tile[at[4 * q + j]] = key[4 * q + j];
        __syncthreads();
        clear();
#pragma unroll
        for (int j = 0; j < 4 * kQuads; ++j) key[j] = tile[tid + j * kSetThreads];       // (behind the last one: any key, not stored)
#pragma unroll
        for (int j = 0; j < 4 * kQuads; ++j) at[j] = to[key[j] >> kBinShift];
#pragma unroll
        for (int j = 0; j < 4 * kQuads; ++j) {
            const uint32_t i = (uint32_t)(tid + j * kSetThreads);
            if (i < in_tile) out[at[j] + i] = key[j];
        }
        __syncthreads();
    }
    // the last keys, fewer than four: positions behind those of the tiles
#pragma unroll
    for (int i = 0; i < kOwn; ++i) to[kOwn * tid + i] = pos[i];
    __syncthreads();
    if ((uint32_t)tid < r.rest) {
        const uint32_t k = f32_key(in[r.tail(tid)]);
        out[atomicAdd(&to[k >> kBinShift], 1u)] = k;
    }
}

__device__ __forceinline__ void add_interval(double (&s)[kSetRow], double t, int terms) {
    const double u = t - 1.0;
    double p = u;
#pragma unroll
    for (int k = 2; k < kGapSums; ++k) { if (k > terms) break; p *= u; s[k] += p; }
}

// t ln t, 0 if t is not above zero.  ln t from the logarithm of the upper eleven bits of its fraction, which the table holds, and six
// terms of the series of the rest, which is below 2^-10: the error is that of the last addition.  (The library's logarithm has so many constants
// that keeping them over the loops around it spills a hundred registers.)
__device__ __forceinline__ double t_log_t(double t, const double* __restrict__ logs) {
    if (!(t > 0.0)) return 0.0;
    int e;
    const double m = frexp(t, &e) * 2048.0;                                   // 1024 <= m < 2048
    const int q = min(max((int)m, 1024), 2047);                               // (an infinite t, of a matrix of equal weights: within the table)
    const double x = (m - (double)q) / (double)q;
    const double series = x * fma(x, fma(x, fma(x, fma(x, fma(x, -1.0 / 6.0, 0.2), -0.25), 1.0 / 3.0), -0.5), 1.0);
    return t * (fma((double)(e - 11), 0.69314718055994530942, logs[q]) + series);
}

// Sum over the workgroup in a fixed order; thread i < kSetRow returns with row i's total.
template <int THREADS>
__device__ __forceinline__ double block_sum(const double (&s)[kSetRow], double (*red)[kSetRow], int terms) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kSetRow; ++k) {
        double v = s[k];
        if (k <= terms || k == kGapSums)                           // (the others are zero)
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
        if (lane == 0) red[wave][k] = v;
        __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    double v = 0.0;
    if (tid < kSetRow)
#pragma unroll 1
        for (int w = 0; w < THREADS / 64; ++w) v += red[w][tid];
    return v;
}

// Sum over the wavefront, in every lane.
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true);      // quad_perm [1, 0, 3, 2]
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true);      // quad_perm [2, 3, 0, 1]
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, true);     // row_half_mirror
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, true);     // row_mirror
    const auto rows = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = (uint32_t)rows[0] + (uint32_t)rows[1];
    const auto halves = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return (uint32_t)halves[0] + (uint32_t)halves[1];
}

// Where a hot bin's bitmap holds 32 of its patterns: a thread's kWords consecutive words, and one that is left out, so that the same word of
// 64 threads is in 64 banks.
constexpr int kWords = kBitmapWords / kSumThreads, kBitmapSize = kBitmapWords + kBitmapWords / kWords;
__device__ __forceinline__ uint32_t bitmap_at(uint32_t word) { return word + word / kWords; }
// Sums over the intervals inside one hot bin, whose patterns are the bitmap `data`: added to s.  Distances below kTable are counted
// (`counted`), and their binary64 terms evaluated once per bin; ln t of a distance is the table's logarithm of a whole number and the
// unit's.  A thread has its words of the bitmap one after another: bit by bit where few are set (one loop over all of a thread's words, whose
// lanes' trips differ less than word by word), 32 patterns at once for distances up to eight where many are (dense).
struct Scale { double inv_mean, log_fraction; int exponent; };               // inv_mean = fraction 2^exponent
__device__ __forceinline__ void add_bitmap(const uint32_t* data, uint32_t bin, const Scale& scale, int terms, bool dense, const SetBuffers& b,
                                           uint32_t* counted, int* wave_last, double (&s)[kSetRow]) {
    constexpr int kWaves = kSumThreads / 64;
    static_assert(kTable % kSumThreads == 0, "distances per thread");
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));              // (what follows from it is made again per bin, not kept over the loop around)
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), word0 = kWords * tid;
    const uint32_t* const own = data + bitmap_at(word0);
    // one exponent: neighbours d patterns apart differ by d units (exactly, also in binary64)
    const uint32_t bin_key = bin << kBinShift, pattern = (bin_key & 0x80000000u) ? bin_key & 0x7FFFFFFFu : ~bin_key;
    const int ex = (int)((pattern >> 23) & 255u);
    const double unit_gap = ldexp(1.0, (ex ? ex : 1) - 150);
    const double log_unit = fma((double)(scale.exponent + (ex ? ex : 1) - 150), 0.69314718055994530942, scale.log_fraction);   // of unit_gap inv_mean
#pragma unroll
    for (int d = 0; d < kTable; d += kSumThreads) counted[d + tid] = 0u;
    if (tid == 0) counted[kTable] = 0u;
    int last = -1;
    uint32_t total = 0u;
#pragma unroll
    for (int j = 0; j < kWords; ++j) {
        const uint32_t x = own[j];
        total += __builtin_popcount(x);
        if (x) last = 32 * (word0 + j) + 31 - __builtin_clz(x);
    }
    // the last set bit before the thread's comes from the threads before
    int prev = last;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) { const int a = __shfl_up(prev, off, 64); if (lane >= off) prev = max(prev, a); }
    if (lane == 63) wave_last[wave] = prev;
    prev = __shfl_up(prev, 1, 64);
    if (lane == 0) prev = -1;
    __syncthreads();
    int top = -1;
#pragma unroll
    for (int v = 0; v < kWaves; ++v) { const int l = wave_last[v]; if (v < wave) prev = max(prev, l); top = max(top, l); }
    if (tid == 0) b.bin_max[bin] = bin_key + (uint32_t)top;
    const int before = prev;
    const uint32_t present = total;
    double logs[kTable / kSumThreads];                                        // asked for here: a trip to memory behind the words
#pragma unroll
    for (int d = 0; d < kTable / kSumThreads; ++d) logs[d] = b.logs[d * kSumThreads + tid];
    if (!dense) {
        // bit by bit over the thread's words: the lanes' numbers of bits differ less over all of them than word by word
        const uint32_t *at = own, *const end = own + kWords;
        uint32_t x = *at;
        int base = 32 * word0;
        if (prev < 0 && last >= 0) {                                          // the first of all: no interval in front of it
            while (!x) { x = *++at; base += 32; }
            prev = base + __builtin_ctz(x);
            x &= x - 1u;
            b.bin_min[bin] = bin_key + (uint32_t)prev;
            total -= 1u;
        }
#pragma unroll 1
        while (at != end) {
            if (x) {
                const int here = base + __builtin_ctz(x);
                x &= x - 1u;
                atomicAdd(&counted[min(here - prev, kTable)], 1u);
                prev = here;
            }
            if (!x) {                                                         // (the word behind the last one: left out, not used)
                x = *++at;
                base += 32;
            }
        }
    } else {
        // distances 1 .. 8 are found for 32 patterns at once, the others bit by bit
        uint32_t beyond[9], prior = tid ? own[-2] : 0u;    // patterns with none of the d in front of them
#pragma unroll
        for (int d = 0; d <= 8; ++d) beyond[d] = 0u;
#pragma unroll 1
        for (int j = 0; j < kWords; ++j) {
            const uint32_t x = own[j];
            uint32_t far = x;
#pragma unroll
            for (int d = 1; d <= 8; ++d) {
                far &= ~((x << d) | (prior >> (32 - d)));
                beyond[d] += __builtin_popcount(far);
            }
#pragma unroll 1
            while (far) {
                const int bit = __builtin_ctz(far), at = 32 * (word0 + j) + bit;
                far &= far - 1u;
                const uint32_t below = x & ((1u << bit) - 1u);
                const int from = below ? 32 * (word0 + j) + 31 - __builtin_clz(below) : prev;
                if (from < 0) {
                    b.bin_min[bin] = bin_key + (uint32_t)at;
                    total -= 1u;                                              // no interval in front of the first
                } else {
                    atomicAdd(&counted[min(at - from, kTable)], 1u);
                }
            }
            if (x) prev = 32 * (word0 + j) + 31 - __builtin_clz(x);
            prior = x;
        }
#pragma unroll
        for (int d = 1; d <= 8; ++d) {
            const uint32_t all = wave_sum_u32((d == 1 ? present : beyond[d - 1]) - beyond[d]);
            if (lane == d) atomicAdd(&counted[d], all);
        }
    }
    s[kGapSums] += (double)total;
    __syncthreads();
    if (counted[kTable]) {                                                    // longer ones, a term each: in front of the lowest bit of a word
        prev = before;
#pragma unroll 1
        for (int j = 0; j < kWords; ++j) {
            const uint32_t x = own[j];
            if (!x) continue;
            const int at = 32 * (word0 + j) + __builtin_ctz(x);
            if (prev >= 0 && at - prev >= kTable) {
                const double t = (double)(at - prev) * unit_gap * scale.inv_mean;
                s[0] += t_log_t(t, b.logs);
                add_interval(s, t, terms);
            }
            prev = 32 * (word0 + j) + 31 - __builtin_clz(x);
        }
    }
#pragma unroll
    for (int i = 0; i < kTable / kSumThreads; ++i) {
        const int d = i * kSumThreads + tid;
        const uint32_t times = counted[d];
        if (times) {
            const double m = (double)times, t = (double)d * unit_gap * scale.inv_mean, u = t - 1.0;
            double p = m * u;
            if (t > 0.0) s[0] += m * (t * (logs[i] + log_unit));              // (t = 0: an infinite span)
#pragma unroll
            for (int k = 2; k < kGapSums; ++k) { if (k > terms) break; p *= u; s[k] += p; }
        }
    }
}

// Bitonic sort of a group: thread t holds keys 4 t .. 4 t + 3 of up to 2048 (`size` of them, a power of two from 256 on, the rest
// of the threads only meet the barriers).  Steps of up to 128 keys stay within a wavefront, in registers (strides 1 and 2) and
// by lane exchanges; the six longer ones of 2048 keys go through LDS, in two buffers that alternate, a barrier each.
// With all 66 steps through LDS, 2^24 random patterns took 1070 us instead of 605, 4096 x 4096 normal weights 173 instead of 161.
template <int L>
__device__ __forceinline__ uint32_t from_lane_xor(uint32_t v) {
    if constexpr (L == 1) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true);     // quad_perm [1, 0, 3, 2]
    else if constexpr (L == 2) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true);    // [2, 3, 0, 1]
    else if constexpr (L == 8) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xF, 0xF, true);   // row_ror 8
    else if constexpr (L == 32) return (uint32_t)__shfl_xor((int)v, 32, 64);
    else return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, (L << 10) | 0x1F);                                  // 4, 16
}
__device__ __forceinline__ void in_order(uint32_t& a, uint32_t& b, bool up) {
    const uint32_t lo = min(a, b), hi = max(a, b);
    a = up ? lo : hi;
    b = up ? hi : lo;
}
// The steps of strides S, S / 2, .., 1 of a merge, S <= 128.
template <int S>
__device__ __forceinline__ void merge_within(uint32_t (&k)[4], int lane, bool up) {
    if constexpr (S >= 4) {
        const bool least = ((lane & (S / 4)) == 0) == up;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t o = from_lane_xor<S / 4>(k[j]);
            k[j] = least ? min(k[j], o) : max(k[j], o);
        }
        merge_within<S / 2>(k, lane, up);
    } else {
        in_order(k[0], k[2], up); in_order(k[1], k[3], up);
        in_order(k[0], k[1], up); in_order(k[2], k[3], up);
    }
}
template <int LEN>
__device__ __forceinline__ void sort_within(uint32_t (&k)[4], uint32_t tid) {       // 4 LEN / 4 .. 256 keys in order, directions as the next merge wants
    if constexpr (LEN == 2) {
        in_order(k[0], k[1], true); in_order(k[2], k[3], false);
    } else {
        sort_within<LEN / 2>(k, tid);
        merge_within<LEN / 2>(k, tid & 63, (4 * tid & LEN) == 0);
    }
}
// Leaves the sorted keys in data (its first or its second half) and returns where, behind a barrier.
__device__ __forceinline__ const uint32_t* sort_group(uint32_t (&k)[4], uint32_t* data, uint32_t size, uint32_t tid) {
    const bool mine = 4u * tid < size;                                          // (whole wavefronts)
    uint32_t* buf = data;
    if (mine) sort_within<256>(k, tid);
    for (uint32_t len = 512u; len <= size; len *= 2u) {
        const bool up = (4u * tid & len) == 0u;
        for (uint32_t stride = len / 2u; stride >= 256u; stride /= 2u) {
            if (mine) *(uint4_t*)(buf + 4 * tid) = uint4_t{k[0], k[1], k[2], k[3]};
            __syncthreads();
            if (mine) {
                const uint4_t o = *(const uint4_t*)(buf + (4u * tid ^ stride));
                const uint32_t ov[4] = {o.x, o.y, o.z, o.w};
                const bool least = ((4u * tid & stride) == 0u) == up;
#pragma unroll
                for (int j = 0; j < 4; ++j) k[j] = least ? min(k[j], ov[j]) : max(k[j], ov[j]);
            }
            buf = buf == data ? data + 2048 : data;
        }
        if (mine) merge_within<128>(k, tid & 63, up);
    }
    if (mine) *(uint4_t*)(buf + 4 * tid) = uint4_t{k[0], k[1], k[2], k[3]};
    __syncthreads();
    return buf;
}

__global__ void __launch_bounds__(kSumThreads, 4) set_sum_kernel(SetGroup g, int terms) {
    const SetBuffers& b = g.b[blockIdx.y];
    __shared__ __attribute__((aligned(16))) uint32_t data[kBitmapSize];     // a bitmap or a group's keys
    __shared__ uint32_t counted[kTable + 1];                                   // intervals of each distance
    __shared__ double red[kSumThreads / 64][kSetRow];
    __shared__ int wave_last[kSumThreads / 64];
    __shared__ int last_piece;
    const int tid = threadIdx.x;
    const SetHead head = *b.head;
    Scale scale;
    scale.inv_mean = (double)(b.count - 1u) / (key_f64(head.max_key) - key_f64(head.min_key));
    const double fraction = frexp(scale.inv_mean, &scale.exponent);
    scale.log_fraction = t_log_t(fraction, b.logs) / fraction;
    double s[kSetRow], sum = 0.0;                                             // of the workgroup's units, whose choice is fixed
#pragma unroll
    for (int k = 0; k < kSetRow; ++k) s[k] = 0.0;
    // the groups (a loop of its own: nothing of it is kept in registers over the bitmaps)
#pragma unroll 1
    for (uint32_t group = gridDim.x - 1u - blockIdx.x; group < head.groups; group += gridDim.x) {
        __syncthreads();                                                      // the keys of the group before are read
        const uint32_t from = b.group_from[group], n = b.group_from[group + 1u] - from;      // at most 2047
        uint32_t size = 256u, own[4];
        while (size < n) size *= 2u;
#pragma unroll
        for (uint32_t j = 0; j < 4u; ++j) own[j] = 4u * tid + j < n ? b.keys[from + 4u * tid + j] : 0xFFFFFFFFu;
        const uint32_t* sorted = sort_group(own, data, size, tid);
#pragma unroll 1
        for (uint32_t i = tid; i < n; i += kSumThreads) {
            const uint32_t k = sorted[i], bin = k >> kBinShift;
            if (i == 0u || sorted[i - 1u] >> kBinShift != bin) b.bin_min[bin] = k;
            if (i + 1u == n || sorted[i + 1u] >> kBinShift != bin) { b.bin_max[bin] = k; continue; }
            const uint32_t k1 = sorted[i + 1u];
            if (k1 == k) continue;
            const double t = (key_f64(k1) - key_f64(k)) * scale.inv_mean;
            s[0] += t_log_t(t, b.logs);
            s[kGapSums] += 1.0;
            add_interval(s, t, terms);
        }
    }
    // the bitmaps
    uint32_t row = 0xFFFFFFFFu;                                               // of a joint bin that the sums are of
#pragma unroll 1
    for (uint32_t unit = blockIdx.x; ; unit += gridDim.x) {
        const bool more = unit < head.pieces;
        const uint4_t piece = more ? b.piece[unit] : uint4_t{0u, 0u, 0u, 0u};
        const bool joined = more && piece.w != 0xFFFFFFFFu;
        __syncthreads();                                                      // data and counts of the unit before are read
        if (!more || joined || row != 0xFFFFFFFFu) {
            // which workgroup sums a joint bin is not fixed: its sums get a row of their own, what comes before is put aside in
            // front of every piece, so that the order of additions is the same
            const double v = block_sum<kSumThreads>(s, red, terms);
            if (row == 0xFFFFFFFFu) sum += v;
            else if (tid < kSetRow) b.sums[(size_t)(kSumWorkgroups + row) * kSetRow + tid] = v;
            row = 0xFFFFFFFFu;
#pragma unroll
            for (int k = 0; k < kSetRow; ++k) s[k] = 0.0;
            if (!more) break;
        }
        const uint32_t bin = piece.x, n = piece.z;                            // n <= 2^26: counters from here on cannot wrap
#pragma unroll
        for (int j = 0; j < kWords / 4; ++j) ((uint4_t*)data)[j * kSumThreads + tid] = uint4_t{0u, 0u, 0u, 0u};
        if (tid < (kBitmapSize - kBitmapWords) / 4) ((uint4_t*)data)[kBitmapWords / 4 + tid] = uint4_t{0u, 0u, 0u, 0u};
        __syncthreads();
        {
            // quads of keys, of which a thread has four in flight, and the up to three keys in front of and behind them
            const uint32_t* own = b.keys + piece.y;
            const uint32_t lead = min((0u - piece.y) & 3u, n), quads = (n - lead) / 4u;
            const uint4_t* src = (const uint4_t*)(own + lead);
            auto set = [&](uint32_t k) { atomicOr(&data[bitmap_at((k >> 5) & (kBitmapWords - 1))], 1u << (k & 31u)); };
            auto set_new = [&](uint32_t k) {                                  // few different keys: most are there already
                uint32_t* const at = &data[bitmap_at((k >> 5) & (kBitmapWords - 1))];
                if (!(*(volatile uint32_t*)at >> (k & 31u) & 1u)) atomicOr(at, 1u << (k & 31u));
            };
            uint32_t i = tid;
            asm volatile("" : "+v"(i));                                       // (made again per bin, not kept over the loop around: it would spill)
            if (i < lead) set(own[i]);
            else if (i >= 4u && i - 4u < n - lead - 4u * quads) set(own[n - 1u - (i - 4u)]);
            // a round: kInFlight quads per thread, those of the next round in flight; past the end the last quad again
            constexpr uint32_t kInFlight = 4u, kRound = kInFlight * kSumThreads;
            uint4_t even[kInFlight], odd[kInFlight];
            bool coarse = false;
            auto fetch = [&](uint4_t (&k)[kInFlight], uint32_t round) {
#pragma unroll
                for (uint32_t j = 0; j < kInFlight; ++j) k[j] = src[min(i + round * kRound + j * kSumThreads, quads - 1u)];
                __builtin_amdgcn_sched_barrier(0);
            };
            auto use = [&](const uint4_t (&k)[kInFlight], uint32_t round) {
#pragma unroll
                for (uint32_t j = 0; j < kInFlight; ++j) {
                    const uint4_t now = k[j];
                    if (i + round * kRound + j * kSumThreads < quads) {
                        // (a wavefront of equal keys: one of them)
                        const unsigned long long live = __builtin_amdgcn_ballot_w64(true);
                        if (__builtin_amdgcn_ballot_w64(now.x == (uint32_t)__builtin_amdgcn_readfirstlane((int)now.x)) == live) {
                            if ((live & lanes_below(i & 63u)) == 0ull) set(now.x);
                            if (__builtin_amdgcn_ballot_w64(now.x == now.y && now.x == now.z && now.x == now.w) == live) continue;
                        } else if (coarse) {
                            set_new(now.x); set_new(now.y); set_new(now.z); set_new(now.w);
                            continue;
                        } else {
                            set(now.x);
                        }
                        set(now.y); set(now.z); set(now.w);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            if ((uint32_t)__builtin_amdgcn_readfirstlane((int)i) < quads) {   // (whole wavefronts)
                const uint32_t rounds = (quads + kRound - 1u) / kRound;
                fetch(even, 0u);
                // values of bfloat16, and others with nothing in their lower bits: 64 lanes would add to a few words one after another
                coarse = __builtin_amdgcn_ballot_w64((even[0].x ^ (uint32_t)__builtin_amdgcn_readfirstlane((int)even[0].x)) & 0xFFFu) == 0ull;
                if (rounds == 1u) {
                    use(even, 0u);
                } else {
#pragma unroll 1
                    for (uint32_t r = 0u; r < rounds; r += 2u) {
                        fetch(odd, r + 1u);
                        use(even, r);
                        fetch(even, r + 2u);
                        use(odd, r + 1u);
                    }
                }
            }
        }
        __syncthreads();
        if (joined) {
            uint32_t* joint = b.joint + (size_t)piece.w * kBitmapWords;
            for (int j = tid; j < kBitmapWords; j += kSumThreads)
                if (const uint32_t x = data[bitmap_at(j)]) atomicOr(&joint[j], x);
            // Every access to the joint bitmap is an atomic operation of the device, served where all compute units see it: that they are
            // done is all the counter below has to wait for.  (A fence would also write back what the L2 holds of other stores: 2^24 uniform
            // weights took 150 us with one, 126 without.)
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            if (tid == 0) last_piece = atomicAdd(&b.done[piece.w], 1u) == (b.counts[bin] - 1u) / kPiece;
            __syncthreads();
            if (!last_piece) continue;
            for (int j = tid; j < kBitmapWords; j += kSumThreads)
                data[bitmap_at(j)] = __hip_atomic_load(&joint[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            row = piece.w;
        }
        add_bitmap(data, bin, scale, terms, b.counts[bin] >= kDense, b, counted, wave_last, s);
    }
    if (tid < kSetRow) b.sums[(size_t)blockIdx.x * kSetRow + tid] = sum;
}

__global__ void __launch_bounds__(kSetThreads) set_final_kernel(SetGroup g, int terms, double tau_c, double tau_f) {
    const SetBuffers& b = g.b[blockIdx.x];
    const uint32_t count = b.count;
    __shared__ uint16_t list[kBins];                                          // the occupied bins
    __shared__ double red[kSetThreads / 64][kSetRow];
    __shared__ double tot[kSetRow];
    __shared__ uint32_t wave_sum[kSetThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const SetHead head = *b.head;
    const double span = key_f64(head.max_key) - key_f64(head.min_key);
    const double inv_mean = (double)(count - 1u) / span;
    double s[kSetRow];
#pragma unroll
    for (int k = 0; k < kSetRow; ++k) s[k] = 0.0;
    for (uint32_t i = tid; i < kSumWorkgroups + head.joints; i += kSetThreads) {
#pragma unroll
        for (int k = 0; k < kSetRow; ++k) s[k] += b.sums[(size_t)i * kSetRow + k];
    }
    constexpr int kOwn = kBins / kSetThreads;                                 // consecutive bins of a thread
    uint32_t own = 0u, occupied = 0u;
#pragma unroll
    for (int j = 0; j < kOwn; ++j) occupied |= (b.counts[kOwn * tid + j] ? 1u : 0u) << j;
    own = __builtin_popcount(occupied);
    uint32_t at = own, bins = 0u;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) { const uint32_t a = (uint32_t)__shfl_up((int)at, off, 64); if (lane >= off) at += a; }
    if (lane == 63) wave_sum[wave] = at;
    at -= own;
    __syncthreads();
    for (int v = 0; v < kSetThreads / 64; ++v) { if (v < wave) at += wave_sum[v]; bins += wave_sum[v]; }
    for (; occupied; occupied &= occupied - 1u) list[at++] = (uint16_t)(kOwn * tid + __builtin_ctz(occupied));
    __syncthreads();
    // the interval in front of every occupied bin but the first
    for (uint32_t i = tid + 1u; i < bins; i += kSetThreads) {
        const double t = (key_f64(b.bin_min[list[i]]) - key_f64(b.bin_max[list[i - 1u]])) * inv_mean;     // (zero between -0 and +0)
        if (t > 0.0) s[0] += t * log(t);
        s[kGapSums] += 1.0;
        add_interval(s, t, terms);
    }
    const double v = block_sum<kSetThreads>(s, red, terms);
    if (tid < kSetRow) tot[tid] = v;
    __syncthreads();
    if (tid == 0) {
        const double n = (double)(count - 1u), equal = n - tot[kGapSums];                         // intervals between equal weights
        double Pc = 0.0, Pf = 0.0;
        if (span > 0.0) {                        // a constant matrix has no intervals to normalise: both proxies 0
            Pc = tot[0] / n;
            for (int k = 2; k <= terms; ++k) Pf += fabs(tot[k] + (k & 1 ? -equal : equal)) / (n * (double)(k * (k - 1)));
        }
        b.out[0] = Pc;
        b.out[1] = Pf;
        *b.phi = (Pc < tau_c && Pf < tau_f) ? 1 : 0;
    }
}

// keys: room for the partitioned keys of the largest matrix at least
static hipError_t launch_sets(SetGroup& g, int n, char* keys, size_t key_bytes, int terms, double tau_c, double tau_f, hipStream_t s) {
    constexpr int lds = kBins * 4, lds_partition = (2 * kBins + kTileKeys + kSetThreads / 64) * 4;     // 32 and 128 KB
    static std::atomic<unsigned long long> raised{0ull};
    const hipError_t e = raise_lds((const void*)set_partition_kernel, lds_partition, raised);
    if (e != hipSuccess) return e;
    uint32_t wgs = 0;
    for (int i = 0; i < n; ++i) wgs = std::max(wgs, g.b[i].wgs);
    hipLaunchKernelGGL(set_clear_kernel, dim3(8, n), dim3(256), 0, s, g);
    hipLaunchKernelGGL(set_count_kernel, dim3(wgs, n), dim3(kSetThreads), lds, s, g);
    hipLaunchKernelGGL(set_plan_kernel, dim3(n), dim3(kSetThreads), 0, s, g);
    // Matrices share launches as the keys have room for them, the largest first and then what still fits: the fullest bins of a large
    // one, which a workgroup reads for long, beside the others' (the layer of the 7B shapes: two launches of a large and two
    // small matrices and one of two).
    int order[kSetGroup], left = n;
    for (int i = 0; i < n; ++i) order[i] = i;
    std::stable_sort(order, order + n, [&](int p, int q) { return g.b[p].count > g.b[q].count; });
    while (left) {
        SetGroup part{};
        int in_part = 0, kept = 0;
        uint32_t part_wgs = 0;
        size_t at = 0;
        for (int i = 0; i < left; ++i) {
            SetBuffers& b = g.b[order[i]];
            if (in_part && at + set_key_bytes(b.count) > key_bytes) { order[kept++] = order[i]; continue; }
            b.keys = (uint32_t*)(keys + at);
            at += set_key_bytes(b.count);
            part_wgs = std::max(part_wgs, b.wgs);
            part.b[in_part++] = b;
        }
        left = kept;
        hipLaunchKernelGGL(set_partition_kernel, dim3(part_wgs, in_part), dim3(kSetThreads), lds_partition, s, part);
        hipLaunchKernelGGL(set_sum_kernel, dim3(kSumWorkgroups, in_part), dim3(kSumThreads), 0, s, part, terms);
    }
    hipLaunchKernelGGL(set_final_kernel, dim3(n), dim3(kSetThreads), 0, s, g, terms, tau_c, tau_f);
    return hipGetLastError();
}

struct F32Layout { size_t keys_a, keys_b, counts, totals, partial, bytes; };
static F32Layout f32_layout(unsigned long long max_count) {
    const size_t tiles = (size_t)((max_count + kSortTile - 1) / kSortTile);
    const size_t gap_tiles = (size_t)((max_count + kGapTile - 1) / kGapTile);
    F32Layout L;
    size_t o = 0;
    L.keys_a = o; o += align256((size_t)max_count * 4);
    L.keys_b = o; o += align256((size_t)max_count * 4);
    L.counts = o; o += align256(tiles * kDigits * 4);
    L.totals = o; o += align256(kDigits * 4);
    L.partial = o; o += align256(gap_tiles * kGapSums * 8);
    L.bytes = o;
    return L;
}

size_t proxy_f32_workspace_bytes(const int* Ns, const int* Ks, int n_mats) {
    unsigned long long mx = 0;
    for (int i = 0; i < n_mats; ++i) {
        const unsigned long long c = (unsigned long long)Ns[i] * (unsigned long long)Ks[i];
        mx = c > mx ? c : mx;
    }
    return f32_layout(mx).bytes;
}

hipError_t launch_proxy_f32(const void* const* ws, const int* Ns, const int* Ks, int n_mats, int terms, double tau_c,
                            double tau_f, void* workspace, double* out, int32_t* phi, hipStream_t s) {
    unsigned long long mx = 0;
    for (int i = 0; i < n_mats; ++i) {
        const unsigned long long c = (unsigned long long)Ns[i] * (unsigned long long)Ks[i];
        mx = c > mx ? c : mx;
    }
    const F32Layout L = f32_layout(mx);
    char* base = (char*)workspace;
    uint32_t* buf[2] = {(uint32_t*)(base + L.keys_a), (uint32_t*)(base + L.keys_b)};
    uint32_t* counts = (uint32_t*)(base + L.counts);
    uint32_t* totals = (uint32_t*)(base + L.totals);
    double* partial = (double*)(base + L.partial);
    SetGroup g{};
    int in_group = 0;
    size_t keys = 0, tables = 0;                   // bytes of the group: the largest matrix's keys, and every one's tables
    auto flush = [&]() {
        // Small matrices by themselves are dealt to more workgroups, where their tables still fit (768 x 768 71 -> 55 us, 2048 x 2048 94 -> 78).
        uint32_t wgs = 0, range = kCountRange;
        size_t more = 0;
        for (int i = 0; i < in_group; ++i) { SetBuffers b{}; more += set_tables(b, nullptr, g.b[i].count, kCountRangeAlone); wgs += set_workgroups(g.b[i].count); }
        if (wgs < 256u && keys + more <= L.bytes) { range = kCountRangeAlone; tables = more; }
        char* at = base + (L.bytes - tables);
        for (int i = 0; i < in_group; ++i) at += set_tables(g.b[i], at, g.b[i].count, range);
        const hipError_t e = in_group ? launch_sets(g, in_group, base, L.bytes - tables, terms, tau_c, tau_f, s) : hipSuccess;
        in_group = 0; keys = tables = 0;
        return e;
    };
    for (int i = 0; i < n_mats; ++i) {
        const uint32_t count = (uint32_t)((unsigned long long)Ns[i] * (unsigned long long)Ks[i]);
        const uint32_t tiles = (uint32_t)(((unsigned long long)count + kSortTile - 1) / kSortTile);   // count may be 2^32 - 1
        const uint32_t* src = (const uint32_t*)ws[i];
        // (the workspace is sized for the sort's two key buffers and its counts; the sets take less from kSetMinCount on)
        SetBuffers b{};
        const size_t own_keys = set_key_bytes(count), own = count >= kSetMinCount ? set_tables(b, nullptr, count) : 0;
        if (count >= kSetMinCount && own_keys + own <= L.bytes) {
            if (in_group == kSetGroup || std::max(keys, own_keys) + tables + own > L.bytes) {
                const hipError_t e = flush();
                if (e != hipSuccess) return e;
            }
            b.in = src; b.out = out + 2 * i; b.phi = phi + i;
            g.b[in_group++] = b;
            keys = std::max(keys, own_keys); tables += own;
            continue;
        }
        const hipError_t flushed = flush();        // (the sort uses the same workspace)
        if (flushed != hipSuccess) return flushed;
        for (int pass = 0; pass < 4; ++pass) {
            uint32_t* dst = buf[pass & 1];
            if (pass == 0) hipLaunchKernelGGL(sort_hist_kernel<true>, dim3(tiles), dim3(kSortThreads), 0, s, src, count, 0, counts, tiles);
            else hipLaunchKernelGGL(sort_hist_kernel<false>, dim3(tiles), dim3(kSortThreads), 0, s, src, count, 8 * pass, counts, tiles);
            hipLaunchKernelGGL(sort_scan_rows_kernel, dim3(kDigits), dim3(256), 0, s, counts, tiles, totals);
            hipLaunchKernelGGL(sort_scan_totals_kernel, dim3(1), dim3(256), 0, s, totals);
            if (pass == 0) hipLaunchKernelGGL(sort_scatter_kernel<true>, dim3(tiles), dim3(kSortThreads), 0, s, src, dst, count, 0, counts, totals, tiles);
            else hipLaunchKernelGGL(sort_scatter_kernel<false>, dim3(tiles), dim3(kSortThreads), 0, s, src, dst, count, 8 * pass, counts, totals, tiles);
            hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
            src = dst;
        }
        const uint32_t gap_tiles = (uint32_t)(((unsigned long long)count - 1 + kGapTile - 1) / kGapTile);
        hipLaunchKernelGGL(gap_sum_kernel, dim3(gap_tiles), dim3(kGapThreads), 0, s, src, count, terms, partial);
        hipLaunchKernelGGL(gap_final_kernel, dim3(1), dim3(256), 0, s, src, count, terms, partial, gap_tiles, tau_c, tau_f,
                           out + 2 * i, phi + i);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return flush();
}

}  // namespace rwkvq

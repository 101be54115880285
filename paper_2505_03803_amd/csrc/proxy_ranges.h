// How the keys of a binary32 matrix are dealt to workgroups (proxy_f32.hip, "partition and sets of values").  A matrix may have
// 2^32 - 1 of them, so no sum below may pass 2^32.  Plain constant expressions, which the kernels and host code both evaluate.
#pragma once
#include <stdint.h>

namespace rwkvq {

constexpr uint32_t kCountRange = 49152;        // fewest keys per counting workgroup
constexpr uint32_t kCountRangeAlone = 16384;   // the same where the matrices of a launch are too few to fill the device
constexpr uint32_t kPiece = 131072;            // keys of a piece of a hot bin that several workgroups read

constexpr uint32_t set_workgroups(uint32_t count, uint32_t range = kCountRange) { return count / range < 256u ? count / range : 256u; }

// The contiguous range of keys of a counting or partitioning workgroup: quads groups of four from lo (a multiple of four) on,
// then rest < 4 single keys.
struct SetRange {
    uint32_t lo, quads, rest;
    constexpr uint32_t tail(uint32_t i) const { return lo + 4u * quads + i; }      // i < rest
};
constexpr SetRange set_range(uint32_t count, uint32_t wg, uint32_t wgs) {
    const uint32_t per = ((count - 1u) / wgs + 4u) & ~3u;
    const unsigned long long l = (unsigned long long)per * wg, h = l + per;
    const uint32_t lo = l < count ? (uint32_t)l : count, hi = h < count ? (uint32_t)h : count;
    return SetRange{lo, (hi - lo) / 4u, (hi - lo) % 4u};
}

// Most keys of a hot bin that one workgroup reads alone, of `count` in all.  Pieces join their bitmaps of 64 KB in memory, and the last to
// finish reads the joint one again: that pays only where the bin would outlast the rest of a launch of 256 compute units.  Us: 14336 x 4096
// uniform weights, whose fullest 32 bins hold a 64th each, alone 346, in pieces 322, uniform in [0, 1) 334 and 304, near-normal ones (a
// 94th) alone 314, in pieces 322; with 2^24 weights, where a 64th takes 30 us, uniform in [0, 1) alone 129, in pieces 132, near-normal
// ones 124 and 130.  (Pieces of 65536 keys: 14336 x 4096 near-normal 348.)
constexpr uint32_t piece_solo_share(uint32_t count) { return count < 1u << 25 ? 64u : 72u; }
constexpr uint32_t piece_solo(uint32_t count) { return count / piece_solo_share(count) > kPiece ? count / piece_solo_share(count) : kPiece; }
// Most bins of more keys than that.
constexpr uint32_t piece_joint_max(uint32_t count) { return count / kPiece < piece_solo_share(count) ? count / kPiece : piece_solo_share(count); }
// Pieces of a hot bin of n keys, and the keys of the one that begins with its key f < n.
constexpr uint32_t piece_count(uint32_t n, uint32_t solo) { return n > solo ? (n - 1u) / kPiece + 1u : 1u; }
constexpr uint32_t piece_keys(uint32_t n, uint32_t f, uint32_t solo) { return n <= solo || n - f < kPiece ? n - f : kPiece; }

}  // namespace rwkvq

// The ranges that the binary32 proxy deals to its workgroups (csrc/proxy_ranges.h), up to the largest matrix of 2^32 - 1 weights:
// together they are the keys 0 .. count - 1, each once, in 32-bit arithmetic that never wraps; and so are the pieces of a bin.
#include "proxy_ranges.h"

#include <cstdio>
#include <initializer_list>

using namespace rwkvq;
typedef unsigned long long u64;

int main() {
    int bad = 0;
    u64 checked = 0;
    auto check_range = [&](uint32_t count, uint32_t wgs) {
        u64 next = 0;
        for (uint32_t wg = 0; wg < wgs; ++wg) {
            const SetRange r = set_range(count, wg, wgs);
            if (next != r.lo || (r.lo % 4u && r.quads) || r.rest > 3u) ++bad;
            next += 4ull * r.quads;
            // every thread of a workgroup of 1024 that takes a single key takes the next one
            for (uint32_t tid = 0; tid < 1024u; ++tid)
                if (tid < r.rest && (u64)r.tail(tid) != next + tid) ++bad;
            next += r.rest;
            // the counter of a thread's strided loop over the quads
            if (r.quads && (u64)r.quads + 4u * 1024u > 0xFFFFFFFFull) ++bad;
        }
        if (next != count) ++bad;
    };
    auto check = [&](uint32_t count) {
        check_range(count, set_workgroups(count));
        if (set_workgroups(count) < 256u) check_range(count, set_workgroups(count, kCountRangeAlone));
        // a bin that holds every key, and the largest that one workgroup reads
        const uint32_t solo = piece_solo(count);
        if (count / (solo + 1u) > piece_joint_max(count)) ++bad;            // bins of several pieces at once
        for (const uint32_t n : {count, solo}) {
            u64 keys = 0, pieces = 0;
            for (uint32_t f = 0; f < n; f += piece_keys(n, f, solo)) {
                if (f != keys || piece_keys(n, f, solo) > (n > solo ? kPiece : solo) || piece_keys(n, f, solo) == 0u) ++bad;
                keys += piece_keys(n, f, solo);
                ++pieces;
                if (keys > n) { ++bad; break; }
            }
            if (keys != n || pieces != piece_count(n, solo) || (n <= solo && pieces != 1u) || solo > (1u << 26)) ++bad;
        }
        ++checked;
    };
    for (uint32_t d = 0; d < 2100u; ++d) check(0xFFFFFFFFu - d);
    for (uint32_t d = 0; d < 600u; ++d) { check((1u << 19) + d); check((1u << 31) + d - 300u); check(256u * kCountRange + d - 300u); }
    for (u64 c = 1u << 19; c <= 0xFFFFFFFFull; c += c / 7 + 1) check((uint32_t)c);
    std::printf("checked %llu bad %d\n", checked, bad);
    return bad != 0;
}

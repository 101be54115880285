// The row tiles that the kernels for 17 to 128 unrounded rows read (csrc/mid_tiles.h): whatever N mod 32 and N mod 64 are, every byte that a
// wavefront asks for lies inside the matrix, and the places that are stored hold their own rows.
#include "mid_tiles.h"

#include <cstdio>
#include <initializer_list>

using namespace rwkvq;

int main() {
    int bad = 0;
    unsigned long long checked = 0;
    const int columns[] = {256, 512, 2304, 14336, 20480};
    for (int NF : {1, 2, 4})
      for (int N = 16; N <= 640; N += 16)
        for (int K : columns)
            for (int tile_bytes : {1536, 2048, 128}) {      // codes (SQ and 6-bit indices, 8-bit indices), scales and zero points
                const int KT = K / 256;
                const long long matrix = (long long)(N / 16) * KT * tile_bytes;
                for (int n0 = 0; n0 < N; n0 += 16 * NF) {
                    const int R0 = n0 >> 4, tiles = mid_row_tiles(N, R0, NF);
                    const long long base = (long long)R0 * KT * tile_bytes;
                    if (tiles < 1 || tiles > NF) ++bad;
                    for (int i = 0; i < NF; ++i)
                        for (int T = 0; T < KT; ++T) {
                            const int at = mid_tile_offset(mid_row_tile(i, tiles), T, KT, tile_bytes);
                            // the lanes read the whole tile and nothing beside it
                            if (at < 0 || base + at + tile_bytes > matrix) ++bad;
                            if (n0 + 16 * i < N && base + at != ((long long)(R0 + i) * KT + T) * tile_bytes) ++bad;
                            ++checked;
                        }
                }
            }
    // every number of rows of x and of workgroups has an instance of the size that the grid is made for, and enough rows of x
    for (int M = 1; M <= 128; ++M)
        for (long long narrow : {1ll, 128ll, 129ll, 256ll, 257ll, 100000ll}) {
            const int mf = mid_exact_mf(M), nf = mid_exact_nf(mf, narrow);
            if (!mid_exact_instance(mf, nf) || 16 * mf * ((M + 63) / 64) < M || 16 * mf > 64) ++bad;
            ++checked;
        }
    std::printf("checked %llu bad %d\n", checked, bad);
    return bad != 0;
}

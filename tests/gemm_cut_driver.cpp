// How the contractions whose columns are tokens cut their grid of tiles (GemmCut), walked on the host for many grids:
//  - every tile has exactly one place;
//  - the (max, sum) slots that the merge reads are those that are written, and no two share an entry or leave the room;
//  - no workgroup has more tiles than with equal groups of columns.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "a3po_common.h"
#include "a3po_launch.h"

using namespace a3po;

static void fail(const char *what, int64_t M, int64_t N, int per)
{
    std::printf("%s: M %lld N %lld workgroups per XCD %d\n", what, (long long)M, (long long)N, per);
    std::exit(1);
}

static int64_t walk(int64_t M, int64_t N, int nxcd, int per)
{
    const int64_t room = gemm_partial_entries(N);
    const GemmCut c = gemm_cut(M, N, nxcd, per, room);
    const GemmShape plain = gemm_shape(M, N, nxcd, per);
    const int mt = plain.mtiles, nt = plain.ntiles;
    if (c.tiles0 + c.part[1].ntiles != nt) fail("columns", M, N, per);
    if (gemm_cut_entries(c, N, nxcd) > room) fail("more partials than there is room for", M, N, per);
    std::vector<int> hit((size_t)mt * nt, 0);
    std::vector<std::vector<char>> wrote(2);
    for (int i = 0; i < 2; ++i) wrote[i].assign((size_t)nxcd * std::max(1, c.part[i].ml) * nt, 0);
    int64_t most = 0;
    for (int x = 0; x < nxcd; ++x)
        for (int slot = 0; slot < per; ++slot) {
            int64_t mine = 0;
            for (int64_t p = (int64_t)x * c.pairs / nxcd; p < (int64_t)(x + 1) * c.pairs / nxcd; ++p) {
                const int i = p >= c.pairs0;
                const GemmShape &s = c.part[i];
                const int64_t q = i ? p - c.pairs0 : p;
                const int nl = slot % s.ncol, ml = slot / s.ncol;
                const int64_t row = q % s.rounds * s.ml + ml, col = (i ? c.tiles0 : 0) + q / s.rounds * s.ncol + nl;
                if (ml >= s.ml || row >= mt || col >= (i ? nt : c.tiles0)) continue;
                ++hit[(size_t)(row * nt + col)];
                wrote[i][(size_t)(((int64_t)x * s.ml + ml) * nt + col)] = 1;
                ++mine;
            }
            most = std::max(most, mine);
        }
    for (int h : hit)
        if (h != 1) fail("a tile has no place or several", M, N, per);
    for (int col = 0; col < nt; ++col) {
        const int i = col >= c.tiles0;  // the rule of lmhead_finish_kernel
        const GemmShape &s = c.part[i];
        const int64_t g0 = i ? c.pairs0 + (int64_t)((col - c.tiles0) / s.ncol) * s.rounds : (int64_t)(col / s.ncol) * s.rounds;
        for (int p = 0; p < nxcd * s.ml; ++p) {
            const int x = p / s.ml, m = p % s.ml;
            const int64_t lo = std::max((int64_t)x * c.pairs / nxcd, g0);
            const int64_t hi = std::min((int64_t)(x + 1) * c.pairs / nxcd, g0 + s.rounds);
            if ((lo < hi && (lo - g0) * s.ml + m < mt) != (bool)wrote[i][(size_t)p * nt + col])
                fail("a partial is read that is not written, or the other way round", M, N, per);
        }
    }
    const int64_t pairs = (int64_t)plain.groups * plain.rounds;
    if (most > (pairs + nxcd - 1) / nxcd) fail("a workgroup has more tiles than with equal groups", M, N, per);
    return (c.pairs + nxcd - 1) / nxcd;
}

int main()
{
    for (int per : {32, 30, 28, 16, 8, 4})
        for (int64_t mt = 1; mt <= 620; mt = mt < 40 ? mt + 1 : mt + 29)
            for (int64_t nt = 1; nt <= 40; ++nt)
                for (int64_t cut : {0, 1, 255}) walk(mt * kGemmTile - cut, nt * kGemmTile - cut, 8, per);
    for (int64_t mt = 1; mt <= 60; ++mt)
        for (int64_t nt = 1; nt <= 20; ++nt) walk(mt * kGemmTile, nt * kGemmTile, 1, 32);
    // rounds of tiles for 594 rows (a vocabulary of 151,936), by columns
    const int want[][2] = {{4, 10}, {5, 13}, {7, 17}, {9, 22}, {10, 25}, {11, 27}, {13, 32}, {16, 38}, {17, 41}, {32, 75}};
    for (const auto &w : want)
        if (walk(594 * kGemmTile, w[0] * kGemmTile, 8, 32) != w[1]) fail("rounds", 594 * kGemmTile, w[0] * kGemmTile, 32);
    std::puts("ok");
}

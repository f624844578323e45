// How the contraction kernel shares a grid of tiles out (GemmShape), walked on the host for many grids:
//  - every tile has exactly one place;
//  - the (max, sum) slots that the merge reads are those that are written, and there is room for them;
//  - no compute unit has more tiles than with blocks of a quarter of an XCD's workgroups x 4 columns, whatever the grid.
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

static void walk(int64_t M, int64_t N, int nxcd, int per)
{
    const GemmShape s = gemm_shape(M, N, nxcd, per);
    const int64_t pairs = (int64_t)s.groups * s.rounds;
    std::vector<int> hit((size_t)s.mtiles * s.ntiles, 0);
    std::vector<char> wrote((size_t)nxcd * s.ml * s.ntiles, 0);
    int64_t most = 0;
    for (int x = 0; x < nxcd; ++x)
        for (int slot = 0; slot < per; ++slot) {
            const int nl = slot % s.ncol, ml = slot / s.ncol;
            if (ml >= s.ml) continue;
            int64_t mine = 0;
            for (int64_t p = (int64_t)x * pairs / nxcd; p < (int64_t)(x + 1) * pairs / nxcd; ++p) {
                const int64_t mt = p % s.rounds * s.ml + ml, nt = p / s.rounds * s.ncol + nl;
                if (mt >= s.mtiles || nt >= s.ntiles) continue;
                ++hit[(size_t)(mt * s.ntiles + nt)];
                wrote[(size_t)(((int64_t)x * s.ml + ml) * s.ntiles + nt)] = 1;
                ++mine;
            }
            most = std::max(most, mine);
        }
    for (int h : hit)
        if (h != 1) fail("a tile has no place or several", M, N, per);
    for (int nt = 0; nt < s.ntiles; ++nt) {
        const int64_t g0 = (int64_t)(nt / s.ncol) * s.rounds;  // the rule of lmhead_finish_kernel
        for (int p = 0; p < nxcd * s.ml; ++p) {
            const int x = p / s.ml, m = p % s.ml;
            const int64_t lo = std::max((int64_t)x * pairs / nxcd, g0);
            const int64_t hi = std::min((int64_t)(x + 1) * pairs / nxcd, g0 + s.rounds);
            if ((lo < hi && (lo - g0) * s.ml + m < s.mtiles) != (bool)wrote[(size_t)p * s.ntiles + nt])
                fail("a partial is read that is not written, or the other way round", M, N, per);
        }
    }
    if ((size_t)nxcd * s.ml * N > gemm_partial_entries(N)) fail("more partials than there is room for", M, N, per);
    const int64_t fixed = (((int64_t)s.ntiles + 3) / 4) * ((s.mtiles + per / 4 - 1) / (per / 4));
    if (most > (fixed + nxcd - 1) / nxcd) fail("a compute unit has more tiles than with fixed blocks", M, N, per);
}

int main()
{
    for (int per : {32, 30, 28, 16})
        for (int64_t mt = 1; mt <= 620; mt = mt < 40 ? mt + 1 : mt + 29)
            for (int64_t nt = 1; nt <= 64; ++nt)
                for (int64_t cut : {0, 1, 255}) walk(mt * kGemmTile - cut, nt * kGemmTile - cut, 8, per);
    for (int64_t mt = 1; mt <= 60; ++mt)
        for (int64_t nt = 1; nt <= 20; ++nt) walk(mt * kGemmTile, nt * kGemmTile, 1, 32);
    std::puts("ok");
}

// Which loss calls go through the kernels of short batches (few_rows_parts), and into how many parts they cut a row:
//  - the partials fit the scratch area, the last workgroup has a thread for every row, no compute unit has more than two parts;
//  - batches lie on the side of the lines that they were measured to be faster on;
//  - the device is not asked about a batch that the kernels take on no device.
#include "a3po_few.hip"

#include <cstdio>
#include <cstdlib>

static int asked = 0;
static a3po::GemmGrid chip;
namespace a3po {
GemmGrid gemm_grid()
{
    ++asked;
    return chip;
}
}

using namespace a3po;

static int parts(int dt, int64_t T, int64_t V)
{
    LossArgs a = {};
    a.dt = dt;
    a.T = T;
    a.V = a.ld = V;
    const int before = asked, n = few_rows_parts(a);
    const int64_t row = V * (dt == A3PO_F32 ? 4 : 2), bytes = T * row;
    auto fail = [&](const char *what) {
        std::printf("%s: %lld rows of %lld, %s: %d parts\n", what, (long long)T, (long long)V, dt == A3PO_F32 ? "fp32" : "bf16", n);
        std::exit(1);
    };
    if (n < 0 || n == 1) fail("parts");
    if (n > 0) {
        if (T > 256 || row < 16384 || bytes > ((int64_t)(row > 20 * 16384 ? 64 : 32) << 20)) fail("beyond the lines");
        if (T * n > 2 * (int64_t)chip.nxcd * chip.per_xcd || row / n < 8192) fail("too many parts");
        if (T * n > (int64_t)(kLossScratchBytes / sizeof(float4)) || T > kTokThreads) fail("no room");
    }
    const bool none = T <= 0 || T > 256 || row < 16384 || bytes > ((int64_t)64 << 20) || (row <= 20 * 16384 && bytes > ((int64_t)32 << 20));
    if (none && asked != before) fail("device asked for nothing");
    return n;
}

int main()
{
    for (GemmGrid g : {GemmGrid{8, 32}, GemmGrid{8, 8}, GemmGrid{1, 38}}) {
        chip = g;
        for (int dt : {A3PO_BF16, A3PO_F32})
            for (int64_t T = 0; T < 400; ++T)
                for (int64_t V = 1; V < ((int64_t)1 << 31); V += 1 + V / 5) parts(dt, T, V);
    }
    chip = {8, 32};
    const struct {
        int dt;
        int64_t T, V;
        int parts;
    } want[] = {{A3PO_BF16, 1, 151936, 32}, {A3PO_BF16, 64, 151936, 8}, {A3PO_BF16, 110, 151936, 4}, {A3PO_BF16, 111, 151936, 0},
                {A3PO_BF16, 256, 32000, 2}, {A3PO_BF16, 257, 32000, 0}, {A3PO_F32, 64, 151936, 8}, {A3PO_F32, 110, 151936, 4},
                {A3PO_F32, 111, 151936, 0}, {A3PO_F32, 64, 81920, 8}, {A3PO_F32, 103, 81920, 0}, {A3PO_F32, 103, 81921, 4},
                {A3PO_BF16, 64, 8191, 0}, {A3PO_BF16, 64, 8192, 2}};
    for (const auto &w : want)
        if (parts(w.dt, w.T, w.V) != w.parts) {
            std::printf("%lld rows of %lld: %d parts, not %d\n", (long long)w.T, (long long)w.V, parts(w.dt, w.T, w.V), w.parts);
            return 1;
        }
    std::puts("ok");
}

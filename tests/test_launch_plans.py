"""The sharing-out of work that the launchers do, walked on the host (no GPU needed)."""
import os
import subprocess

from paper_2512_06547_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def run_on_host(source, tmp_path, kernels=False):
    """Compiles a program and runs it here; `kernels`: its source holds some, which are compiled along but not run."""
    exe = str(tmp_path / "plan")
    how = build.FLAGS if kernels else ["--offload-arch=gfx950", "--offload-host-only", "-O2", "-std=c++17",
                                       "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC]
    subprocess.check_call([build.HIPCC, "-x", "hip", *how, source, "-o", exe], stderr=subprocess.DEVNULL)
    done = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert done.returncode == 0, done.stdout
    return done.stdout


def test_every_tile_has_one_place_and_no_unit_more_than_its_share(tmp_path):
    assert run_on_host(os.path.join(HERE, "gemm_plan_driver.cpp"), tmp_path) == "ok\n"


def test_every_row_length_has_a_kernel_and_the_threads_it_is_fastest_with(tmp_path):
    assert run_on_host(os.path.join(HERE, "row_plan_driver.cpp"), tmp_path) == "ok\n"


def test_histogram_workgroups_are_bounded_by_what_their_merge_costs(tmp_path):
    """Workgroups merge one after the other, some 12 ns each: the merge stays below 4 us plus the time that a fifth of
    the memory's rate takes for the values (4 bytes and a selection byte each, 1.2 TB/s), and there are never fewer
    workgroups than for a smaller input."""
    source = tmp_path / "hist.cpp"
    source.write_text('''#include <cstdio>
#include "a3po_common.h"
#include "a3po_launch.h"
int main()
{
    for (int64_t T = 1; T < ((int64_t)1 << 36); T += 1 + T / 7)
        std::printf("%lld %lld\\n", (long long)T, (long long)a3po::histogram_blocks(T));
}
''')
    plan = [tuple(map(int, line.split())) for line in run_on_host(str(source), tmp_path).splitlines()]
    assert plan[0] == (1, 1) and all(a[1] <= b[1] for a, b in zip(plan, plan[1:]))
    for T, blocks in plan:
        assert blocks * 12e-9 <= 4e-6 + 5 * T / 1.2e12, (T, blocks)
        assert (T + blocks - 1) // blocks < 2 ** 32, "a workgroup counts in 32 bits"


def test_few_token_tiles_cover_the_vocabulary_evenly(tmp_path):
    """Every row block of 16 vocabulary entries lies in one tile, no compute unit has more of them than an even share
    rounded up, and there are no more tiles in a round than compute units."""
    source = tmp_path / "few.cpp"
    source.write_text('''#include <cstdio>
#include "a3po_common.h"
#include "a3po_launch.h"
using namespace a3po;
int main()
{
    for (int64_t cus : {256, 64, 38})
        for (int64_t V = 1; V < 700000; V += V < 9000 ? 1 : 97) {
            const FewTiles f = few_tiles(V, cus);
            const int64_t blocks = (V + 15) / 16, held = f.nfull * 16ll + (int64_t)(f.ntiles - f.nfull) * f.last_blocks;
            const int64_t rounds = f.nfull / cus, share = (blocks + cus - 1) / cus;
            const bool ok = f.nfull % cus == 0 && f.ntiles > f.nfull && f.ntiles - f.nfull <= cus && f.last_blocks >= 1 &&
                            f.last_blocks <= 16 && held >= blocks && held - blocks < f.last_blocks &&
                            rounds * 16 + f.last_blocks <= share && f.slots == (f.ntiles < cus ? f.ntiles : cus);
            if (!ok) return std::printf("V %lld on %lld\\\\n", (long long)V, (long long)cus), 1;
        }
}
''')
    assert run_on_host(str(source), tmp_path) == ""


def test_few_token_tiles_are_whole_where_the_products_bind(tmp_path):
    """From 193 tokens on the last round is spread over all compute units only where a wavefront then has one row block;
    up to 192 always.  Either way every row block lies in one tile."""
    source = tmp_path / "few.cpp"
    source.write_text('''#include <cstdio>
#include "a3po_common.h"
#include "a3po_launch.h"
using namespace a3po;
int main()
{
    for (int64_t T : {1, 64, 192, 193, 256})
        for (int64_t V = 1; V < 300000; V += 61) {
            const FewTiles f = few_tiles_of(T, V, 256), even = few_tiles(V, 256);
            const int64_t blocks = (V + 15) / 16, held = f.nfull * 16ll + (int64_t)(f.ntiles - f.nfull) * f.last_blocks;
            const bool whole = T > 192 && even.last_blocks > 8;
            const bool ok = f.nfull == even.nfull && f.last_blocks == (whole ? 16 : even.last_blocks) && held >= blocks &&
                            held - blocks < f.last_blocks && f.ntiles <= even.ntiles && f.slots == (f.ntiles < 256 ? f.ntiles : 256);
            if (!ok) return std::printf("T %lld V %lld\\n", (long long)T, (long long)V), 1;
        }
}
''')
    assert run_on_host(str(source), tmp_path) == ""


def test_uneven_column_groups_leave_no_tile_out_and_no_unit_worse_off(tmp_path):
    assert run_on_host(os.path.join(HERE, "gemm_cut_driver.cpp"), tmp_path) == "ok\n"


def test_short_batches_are_cut_to_fit_and_cost_the_others_nothing(tmp_path):
    assert run_on_host(os.path.join(HERE, "few_rows_plan_driver.cpp"), tmp_path, kernels=True) == "ok\n"

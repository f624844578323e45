"""The sharing-out of the contraction kernel's tiles, walked on the host (no GPU needed)."""
import os
import subprocess

from paper_2512_06547_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_every_tile_has_one_place_and_no_unit_more_than_its_share(tmp_path):
    exe = str(tmp_path / "gemm_plan")
    subprocess.check_call([build.HIPCC, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-O2", "-std=c++17",
                           "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC,
                           os.path.join(HERE, "gemm_plan_driver.cpp"), "-o", exe], stderr=subprocess.DEVNULL)
    done = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert done.returncode == 0 and done.stdout == "ok\n", done.stdout

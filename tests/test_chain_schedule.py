"""The chain kernels' cooling stages, their own source compiled for the CPU
(host_schedule.hip) and stepped against floor(step stages / steps): stage counts
beside 2^30 and up to 2^31 - 1, where a stage's remainder and the next one's
share do not fit in 31 bits, among them."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    from paper_1411_4622_amd import build
    exe = str(tmp_path_factory.mktemp("schedule") / "host_schedule")
    subprocess.run([build._hipcc(), "--offload-arch=" + build.ARCH, "--cuda-host-only", "-x", "hip", "-std=c++17", "-O1",
                    "-w", "-I", os.path.join(ROOT, "include"), "-I", build.CSRC,
                    os.path.join(HERE, "host_schedule.hip"), "-o", exe], check=True, timeout=300)
    return exe


@pytest.mark.parametrize("n_steps,n_stages,first,last", [
    (1, 1, 0, 0), (100, 7, 0, 99), (7, 100, 0, 6), (64, 64, 0, 63), (5_000_000, 1000, 0, 100_000),
    (5_000_000, 1000, 4_900_000, 4_999_999), (10**12, 3, 10**12 - 5, 10**12 - 1),
    (2**30, 2**30 + 1, 0, 1000), (1_500_000_000, 2**31 - 1, 0, 1000), (2**31 - 2, 2**31 - 1, 10**9, 10**9 + 1000),
    (3 * 2**30 + 7, 2**31 - 1, 5, 1000), (2**31 - 1, 2**30 + 5, 2**31 - 1000, 2**31 - 2)])
def test_stage_of_every_step(driver, n_steps, n_stages, first, last):
    out = subprocess.run([driver], input="%d %d %d %d\n" % (n_steps, n_stages, first, last), capture_output=True,
                         text=True, timeout=60, check=True)
    assert out.stdout.split() == ["-1"]

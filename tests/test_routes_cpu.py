"""The kernel that fdtd_step_n launches for small boards, without a GPU: bricks alone
and beside one other stepping board, the marching kernel beside two and more where that
shares the device better, and while the caller records the call."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not shutil.which(hipcc):
        pytest.skip("hipcc not found")
    exe = str(tmp_path_factory.mktemp("host") / "routes")
    subprocess.check_call([hipcc, "-x", "hip", "--cuda-host-only", "-std=c++17", "-O1",
                           "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_1008_2602_amd", "csrc"),
                           os.path.join(HERE, "host", "routes.cpp"), "-o", exe,
                           "-Wl,--unresolved-symbols=ignore-all"],
                          stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    out = subprocess.run([exe], check=True, capture_output=True, text=True, timeout=60).stdout
    return {line.split()[0]: "".join(line.split()[1:]) for line in out.splitlines()}


def test_boards_stepping_at_once(routes):
    assert routes["alone"] == "BBBB"
    assert routes["three_at_once"] == "BBM" "MMM"
    # the first two of each turn, then the third beside them, then the third alone
    assert routes["waited_for"] == "MMMB" + "BBMB" * 7
    assert routes["recorded"] == "MM" "BB"
    # two on another device; here one still stepping, then two
    assert routes["other_device"] == "BB" "BB"
    assert routes["released"] == "M" "B"
    assert routes["left"] == "0"


def test_boards_that_march_in_a_crowd(routes):
    """Alone, two others, the board beside them: those whose bricks cost the device 1.5
    times what marching does change over, all others keep their kernel."""
    got = {k[6:]: v for k, v in routes.items() if k.startswith("crowd_")}
    changes = {"48x43x30", "60x60x30", "64x40x60"}
    for size, v in got.items():
        assert v == ("MBBM" if size == "300x300x40" else "BBBM" if size in changes else "BBBB"), size

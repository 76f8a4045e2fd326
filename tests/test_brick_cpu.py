"""Which boards are stepped in bricks, and in which shape: the choice (a rule on sizes
and compute units) evaluated without a GPU at the sizes that the GPU tests run."""
import os
import shutil
import subprocess

import pytest

from _bricks import B87, B88, B128, B1010, B168, CUS, EDGES, MARCHING, SHAPES

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_choice_covers_every_shape(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not shutil.which(hipcc):
        pytest.skip("hipcc not found")
    exe = str(tmp_path / "brick_pick")
    subprocess.check_call([hipcc, "-x", "hip", "--cuda-host-only", "-std=c++17", "-O1",
                           "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_1008_2602_amd", "csrc"),
                           os.path.join(HERE, "host", "brick_pick.cpp"), "-o", exe,
                           "-Wl,--unresolved-symbols=ignore-all"],
                          stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    want = {**EDGES, **SHAPES}
    args = [str(v) for n in want for v in n]
    out = subprocess.run([exe, str(CUS), *args], check=True, capture_output=True, text=True).stdout
    got = [tuple(int(v) for v in line.split()) for line in out.splitlines()]
    assert dict(zip(want, got)) == want
    assert set(got) == {B87, B88, B128, B1010, B168, MARCHING}
    # a device with few compute units would need several rounds of bricks
    out = subprocess.run([exe, "16", *args], check=True, capture_output=True, text=True).stdout
    assert out.splitlines()[list(want).index((48, 43, 30))] == "0 0"

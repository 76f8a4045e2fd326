"""The handles' pinned buffers (results pass through them) without a GPU: every live
handle has one of its own, released ones serve the next handles of their size, no
more than 256 MiB of them are kept, and all are freed when the last handle goes
whose device memory is freed with it."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def counts(tmp_path_factory):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not shutil.which(hipcc):
        pytest.skip("hipcc not found")
    exe = str(tmp_path_factory.mktemp("host") / "pinned")
    subprocess.check_call([hipcc, "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_1008_2602_amd", "csrc"),
                           os.path.join(HERE, "host", "pinned.cpp"), "-o", exe, "-lpthread",
                           "-Wl,--unresolved-symbols=ignore-all"],
                          stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    out = subprocess.run([exe], check=True, capture_output=True, text=True, timeout=60).stdout
    rows = [line.split() for line in out.splitlines()]
    return {r[0]: {r[q]: int(r[q + 1]) for q in (1, 3, 5)} for r in rows}


def test_buffers_are_reused_bounded_and_given_back(counts):
    # released beside other work: nothing freed, one buffer made for ten handles
    assert counts["in_turn_callers"] == {"made": 1, "freed": 0, "live": 1}
    # the first takes the kept one; the next two share a size class with each other and the last
    assert counts["several_sizes"] == {"made": 2, "freed": 3, "live": -1}
    # 150 of 4 MiB: 64 fit 256 MiB, the others are freed as they go
    assert counts["many_large"] == {"made": 150, "freed": 86, "live": 64}
    assert counts["given_back"] == {"made": 1, "freed": 65, "live": -64}
    assert counts["refused"] == {"made": 1, "freed": 1, "live": 0}
    assert counts["threads"]["live"] == 0
    assert 16 <= counts["threads"]["made"] <= 800

"""Results on their way to the host (read_out) without a GPU: random pieces through
halves of random sizes come back as stored, in stream order, with the watchdog flag of
their time, and without any allocation (the library throws nothing across its C
entries, and the allocation-free probe spectrum stays so)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_pieces_come_back_as_stored_without_allocating(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not shutil.which(hipcc):
        pytest.skip("hipcc not found")
    exe = str(tmp_path / "readout")
    subprocess.check_call([hipcc, "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_1008_2602_amd", "csrc"),
                           os.path.join(HERE, "host", "readout.cpp"), "-o", exe,
                           "-Wl,--unresolved-symbols=ignore-all"],
                          stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    out = subprocess.run([exe], check=True, capture_output=True, text=True, timeout=60).stdout.split()
    r = {out[q]: int(out[q + 1]) for q in range(0, len(out), 2)}
    assert r["trials"] == 3000 and r["turns"] > 10000
    assert r["wrong"] == 0
    assert r["allocations"] == 0

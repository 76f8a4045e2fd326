"""Work lists of the one-step shapes (but 64 x 15): every tile plane once, and on each XCD
the last partial round's tiles in the number of pieces that a plain evaluation of the
rule gives (as before the two-step kernels' lists had a rule of their own)."""
import math
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def work_list(tmp_path_factory):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not shutil.which(hipcc):
        pytest.skip("hipcc not found")
    exe = str(tmp_path_factory.mktemp("host") / "one_step_list")
    subprocess.check_call([hipcc, "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_1008_2602_amd", "csrc"),
                           os.path.join(HERE, "host", "one_step_list.cpp"), "-o", exe,
                           "-Wl,--unresolved-symbols=ignore-all"],
                          stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)

    def run(*args):
        return subprocess.run([exe, *map(str, args)], check=True, capture_output=True, text=True).stdout.splitlines()
    return run


def pieces(m, planes, slots):
    """m tiles of a partial round in S pieces: S x (planes / S + 1) per round of slots,
    taken where it saves 3 % and no piece falls below two planes."""
    best, S = float(planes), 1
    for s in range(2, 17):
        if planes / s < 2:
            break
        cost = math.ceil(m * s / slots) * (planes / s + 1)
        if cost < 0.97 * best:
            best, S = cost, s
    return S


@pytest.mark.parametrize("case", [(444, 364, 60, 64, 13, 32), (444, 364, 60, 64, 3, 160), (301, 283, 44, 64, 11, 32),
                                  (48, 43, 30, 64, 14, 32), (300, 200, 40, 128, 6, 64), (900, 800, 20, 64, 7, 64),
                                  (2, 2, 3, 64, 3, 32), (130, 60, 1, 64, 9, 32)], ids=str)
def test_one_step_lists(work_list, case):
    nx, ny, nz, tx, rows, slots = case
    lines = work_list(*case)
    cx, cy = -(-nx // tx), -(-ny // rows)
    L = len(lines) // 8
    assert len(lines) == 8 * L
    planes, index, acc = {}, 0, 0.0
    for x in range(8):
        run = [tuple(map(int, e.split())) for e in lines[x * L:(x + 1) * L] if e != "idle"]
        mine = []
        while index < cx * cy and (x == 7 or acc + 0.5 * nz <= cx * cy * nz * (x + 1) / 8):
            mine.append((index % cx, index // cx))
            acc += nz
            index += 1
        m = len(mine) % slots
        S = pieces(m, nz, slots) if m else 1
        whole, cut = mine[:len(mine) - m], mine[len(mine) - m:]
        want = [(*t, 0, nz) for t in whole]
        want += [(*t, nz * q // S, nz * (q + 1) // S) for q in range(S) for t in cut]
        assert run == want, x
        for a, b, kb, ke in run:
            planes.setdefault((a, b), []).extend(range(kb, ke))
    assert set(planes) == {(a, b) for a in range(cx) for b in range(cy)}
    assert all(sorted(p) == list(range(nz)) for p in planes.values())

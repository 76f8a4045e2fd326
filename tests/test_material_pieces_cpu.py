"""Which kernels step boards with rebuilt coefficients: whole 64 x 14 material tiles where
the launch has many of them, and the split (64 x 10 tiles where every node is rebuilt)
where few blocks are in flight; every tile plane of a board once, alone and in a batch."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def pieces(tmp_path_factory):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not shutil.which(hipcc):
        pytest.skip("hipcc not found")
    exe = str(tmp_path_factory.mktemp("host") / "material_pieces")
    subprocess.check_call([hipcc, "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_1008_2602_amd", "csrc"),
                           os.path.join(HERE, "host", "material_pieces.cpp"), "-o", exe,
                           "-Wl,--unresolved-symbols=ignore-all"],
                          stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)

    def run(copies, *boards):
        flat = [str(v) for b in boards for v in b]
        out = {"alone": [], "batch": []}
        for line in subprocess.run([exe, "256", str(copies), *flat], check=True, capture_output=True,
                                   text=True).stdout.splitlines():
            how, kernel, *rest = line.split()
            out[how].append((kernel, *map(int, rest)))
        return out
    return run


ROWS = {"plain": 11, "conduct": 11, "tall": 11, "short": 7}      # rows that a tile owns


def kernels(found, boards):
    """The kernels in use, after checking that each (column strip, row, plane) of every
    board is in one piece."""
    for b, (nx, ny, nz, *_) in enumerate(boards):
        seen = set()
        for kernel, board, tx, ty, kb, ke in found:
            if board != b:
                continue
            own = ROWS[kernel]
            for j in range(ty * own, min(ny, ty * own + own)):
                for k in range(kb, ke):
                    assert (tx, j, k) not in seen
                    seen.add((tx, j, k))
        assert len(seen) == -(-nx // 64) * ny * nz
    return {f[0] for f in found}


def slab(nx, ny, nz):
    return nx, ny, nz, nz // 2, nz // 2 + 4


def filled(nx, ny, nz):
    return nx, ny, nz, 0, nz + 1


WHOLE, SHORT, SPLIT = {"tall"}, {"short"}, {"short", "plain"}


@pytest.mark.parametrize("copies, board, alone, batch", [
    (1, filled(56, 39, 48), SHORT, SHORT), (4, filled(56, 39, 48), SHORT, WHOLE),
    (1, filled(27, 45, 65), SHORT, SHORT), (1, filled(26, 101, 36), SHORT, SHORT),
    (4, filled(20, 35, 50), SHORT, SHORT), (1, filled(15, 228, 11), SHORT, SHORT),
    (3, filled(28, 145, 12), SHORT, SHORT), (1, filled(2, 2, 2), SHORT, SHORT),          # one tile of either
    (1, filled(128, 77, 60), WHOLE, WHOLE), (1, filled(200, 200, 60), WHOLE, WHOLE),
    (1, filled(444, 364, 60), WHOLE, WHOLE), (1, filled(1048, 792, 88), SHORT, SHORT),   # past the line
    (4, filled(128, 386, 20), WHOLE, WHOLE),                                             # both in rounds
    (1, slab(64, 32, 86), SPLIT, SPLIT), (2, slab(64, 32, 86), SPLIT, SPLIT), (3, slab(64, 32, 86), SPLIT, WHOLE),
    (1, slab(64, 88, 60), SPLIT, SPLIT), (1, slab(64, 89, 60), WHOLE, WHOLE),            # 8 and 9 tiles
    (1, slab(48, 43, 30), WHOLE, WHOLE), (1, slab(48, 43, 33), SPLIT, SPLIT),            # pieces of two and three planes
    (1, slab(444, 364, 60), WHOLE, WHOLE),
], ids=str)
def test_the_kernels_of_a_launch(pieces, copies, board, alone, batch):
    found = pieces(copies, board)
    boards = [board] * copies
    assert kernels(found["alone"], boards) == alone
    assert kernels(found["batch"], boards) == batch


def test_boards_of_both_kinds_in_one_batch(pieces):
    boards = [slab(64, 32, 86), slab(64, 32, 86), filled(56, 39, 48)]
    for use, batch in ((boards, WHOLE), (boards[1:], SPLIT)):
        found = pieces(1, *use)
        assert kernels(found["alone"], use) == {"short", "plain"}
        assert kernels(found["batch"], use) == batch
    # past the line a board keeps its split, whatever the others run
    use = [slab(1048, 792, 88), slab(444, 364, 60)]
    found = pieces(1, *use)
    assert kernels([f for f in found["batch"] if f[1] == 1], use[:0]) == WHOLE
    assert kernels(found["batch"], use) == {"tall", "short", "plain"}

"""Several small boards stepped at once, each on its own stream, from one thread and
from several: whichever kernel a call takes (bricks or, beside two other stepping
boards, the marching kernel), every board ends with the bits it has alone."""
import threading

import numpy as np
import pytest

import boardgen

pytestmark = pytest.mark.gpu

FIELDS = range(12)
# per board: call lengths that change kernel, field copy and graph from call to call
CALLS = [[7, 64, 100, 3, 333], [2, 33, 2100, 5, 64], [100, 101, 32, 1, 70], [3, 2051, 64, 65, 2], [64, 64, 1, 200, 9]]


@pytest.fixture(scope="module")
def F():
    import torch
    assert torch.cuda.is_available()
    torch.cuda.set_device(0)
    from paper_1008_2602_amd import fdtd
    return fdtd


def boards():
    out = []
    for q, c in enumerate(CALLS):
        b = boardgen.table1_board(steps=sum(c), source="resistive") if q != 3 else boardgen.small_board(steps=sum(c))
        for s in b.sources:
            s.J0 *= 1 + q
            s.t0, s.sigma = 4e-11, 2e-11
        b.plane_dft = (b.nz // 2, np.array([2e9, 5e9])) if q == 1 else None
        b.dft_freqs = np.array([3e9, 7e9]) if q == 2 else None
        out.append(b)
    return out


def results(F, g, ids, b):
    shape = (b.nz + 1, b.ny + 1, b.nx + 1)
    out = [F.fdtd_get_probe(g, p, b.steps) for p in ids] + [F.fdtd_get_field(g, c, shape) for c in FIELDS]
    if b.plane_dft is not None:
        out.append(F.fdtd_get_plane_dft(g, b.ny, b.nx))
    return out


@pytest.fixture(scope="module")
def alone(F):
    out = []
    for b, calls in zip(boards(), CALLS):
        g, ids = F.grid_from_board(b)
        for n in calls:
            F.fdtd_step_n(g, n)
            F.fdtd_synchronize(g)
        out.append(results(F, g, ids, b))
        F.fdtd_destroy_grid(g)
    assert all(np.abs(o[0]).max() > 0 for o in out)
    return out


def compare(F, hs, bs, alone):
    for q, ((g, ids), b) in enumerate(zip(hs, bs)):
        for c, (x, y) in enumerate(zip(results(F, g, ids, b), alone[q])):
            assert np.array_equal(x, y), (q, c)


@pytest.mark.parametrize("order", ["in_turn", "waiting", "threads"])
def test_boards_stepped_at_once_equal_alone(F, alone, order):
    print(f"[gpu] concurrent boards {order}", flush=True)
    bs = boards()
    hs = [F.grid_from_board(b) for b in bs]
    try:
        if order == "threads":
            errors = []

            def work(q):
                try:
                    for r, n in enumerate(CALLS[q]):
                        F.fdtd_step_n(hs[q][0], n)
                        if (r + q) % 3 == 0:
                            F.fdtd_synchronize(hs[q][0])
                except Exception as e:                   # reported by the test's own thread
                    errors.append(e)
            ts = [threading.Thread(target=work, args=(q,)) for q in range(len(hs))]
            for t in ts:
                t.start()
            for t in ts:
                t.join(60)
            assert not errors and not any(t.is_alive() for t in ts)
        else:
            for r in range(5):
                for q, (g, _) in enumerate(hs):
                    F.fdtd_step_n(g, CALLS[q][r])
                    if order == "waiting" and (r + q) % 2:
                        F.fdtd_synchronize(g)
        compare(F, hs, bs, alone)
    finally:
        for g, _ in hs:
            F.fdtd_destroy_grid(g)

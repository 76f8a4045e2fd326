"""The small-board kernel (bricks, the default for plain boards of up to a few
10^5 cells) against the marching kernel (a tile shape set): the same bits from an
arbitrary state, at sizes around the bricks' edges in every shape, with sources of
both kinds, probes, a plane DFT, narrow and wide class maps and odd step counts, and
over a call long enough to be replayed as a graph from either field copy."""
import numpy as np
import pytest

import boardgen

pytestmark = pytest.mark.gpu

FIELDS = range(12)
MARCH = (64, 10, 2)


@pytest.fixture(scope="module")
def F():
    import torch
    assert torch.cuda.is_available()
    torch.cuda.set_device(0)
    from paper_1008_2602_amd import fdtd
    return fdtd


def outcome(F, b, chunks, tile, init=None):
    g, ids = F.grid_from_board(b, max_steps=sum(chunks), tile=tile)
    shape = (b.nz + 1, b.ny + 1, b.nx + 1)
    try:
        if init is not None:
            for c in FIELDS:
                F.fdtd_set_field(g, c, init[c])
        for n in chunks:
            F.fdtd_step_n(g, n)
        out = [F.fdtd_get_probe(g, p, sum(chunks)) for p in ids]
        out += [F.fdtd_get_field(g, c, shape) for c in FIELDS]
        if b.plane_dft is not None:
            out.append(F.fdtd_get_plane_dft(g, b.ny, b.nx))
        return out
    finally:
        F.fdtd_destroy_grid(g)


# one brick and less; exact and ragged multiples of each shape's 28 columns, rows
# and planes (8x7: 4 x 3, 8x8: 4 x 4, 12x8: 8 x 4, 10x10: 6 x 6, 16x8: 12 x 4)
SIZES = [(8, 7, 6), (28, 8, 9), (29, 13, 10), (56, 44, 30), (57, 41, 45), (66, 46, 30), (84, 66, 42),
         (81, 67, 37), (131, 61, 41)]


@pytest.mark.parametrize("wide", [False, True], ids=["narrow", "wide"])
@pytest.mark.parametrize("n", SIZES, ids=str)
def test_bricks_give_the_marching_kernels_bits(F, n, wide):
    nx, ny, nz = n
    print(f"[gpu] bricks {n} wide={wide}", flush=True)
    b = boardgen.random_tiny(nx + ny + nz, nx=nx, ny=ny, nz=nz, npml=2, steps=1)
    rng = np.random.default_rng(3)
    if wide:
        b.eps_r_cell[:] = rng.uniform(1.0, 6.0, b.eps_r_cell.shape).astype(np.float32)
        b.eps_r_cell[:] = np.round(b.eps_r_cell * 2) / 2
    for s in b.sources:
        s.t0, s.sigma = 4e-12, 2e-12
    taken = {(s.i, s.j, s.k) for s in b.sources}
    i, j, k = nx // 2, ny // 2, nz // 2
    if (i, j, k) not in taken and not b.pec_edge_mask[k, j, i] & 4:
        b.sources.append(boardgen.Source(i, j, k, boardgen.DGAUSS, 2.0, 4e-12, 2e-12, R=25.0))
    b.plane_dft = (nz // 2, np.array([3e9, 17e9]))
    init = [rng.standard_normal((nz + 1, ny + 1, nx + 1)).astype(np.float32) for _ in FIELDS]
    got = outcome(F, b, [5, 2, 4], None, init)
    want = outcome(F, b, [5, 2, 4], MARCH, init)
    for q, (x, y) in enumerate(zip(got, want)):
        assert np.array_equal(x, y), q


def test_long_calls_from_either_field_copy(F):
    """2051 steps (graph replays and an odd last step) twice: the second call starts
    from the other field copy."""
    b = boardgen.table1_board(steps=4102, source="resistive")
    b.dft_freqs = np.array([2e9, 5e9])
    got = outcome(F, b, [2051, 2051], None)
    want = outcome(F, b, [2051, 2051], MARCH)
    assert np.abs(want[0]).max() > 0
    for q, (x, y) in enumerate(zip(got, want)):
        assert np.array_equal(x, y), q

"""Every brick shape of the small-board kernel, and the kernel that a handle reports:
the marching kernel's bits from an arbitrary state with PMLs that differ per face and
are absent on some or all of them, and over calls long enough to replay graphs."""
import numpy as np
import pytest

import boardgen
from _bricks import CUS, EDGES, MARCHING, SHAPES
from test_gpu_brick import MARCH

pytestmark = pytest.mark.gpu

FIELDS = range(12)


@pytest.fixture(scope="module")
def F():
    import torch
    assert torch.cuda.is_available()
    torch.cuda.set_device(0)
    assert torch.cuda.get_device_properties(0).multi_processor_count == CUS
    from paper_1008_2602_amd import fdtd
    return fdtd


def outcome(F, b, chunks, tile, brick, init=None):
    g, ids = F.grid_from_board(b, max_steps=sum(chunks), tile=tile)
    shape = (b.nz + 1, b.ny + 1, b.nx + 1)
    try:
        assert F.fdtd_get_route(g).brick_rows == 0      # nothing is decided before the set-up
        for c in FIELDS if init is not None else ():
            F.fdtd_set_field(g, c, init[c])
        for n in chunks:
            F.fdtd_step_n(g, n)
        r = F.fdtd_get_route(g)
        assert (r.brick_rows, r.brick_planes) == brick
        assert (r.material_tile_y, r.whole_tiles, r.plain_planes) == (0, 0, 0)
        assert (1 << 20) <= r.pinned_bytes <= (4 << 20) + 256
        out = [F.fdtd_get_probe(g, p, sum(chunks)) for p in ids]
        out += [F.fdtd_get_field(g, c, shape) for c in FIELDS]
        if b.plane_dft is not None:
            out.append(F.fdtd_get_plane_dft(g, b.ny, b.nx))
        return out
    finally:
        F.fdtd_destroy_grid(g)


def board(n, npml, wide=False):
    nx, ny, nz = n
    rng = np.random.default_rng(nx + ny + nz)
    eps, mask = boardgen.air(nx, ny, nz)
    boardgen.fill_box(eps, 0, nx, ny // 4, ny, 0, max(1, nz // 2), 3.4)
    if wide:
        eps[:] = np.round(rng.uniform(1.0, 6.0, eps.shape) * 2).astype(np.float32) / 2
    if nx > 4 and ny > 4 and nz > 4:
        boardgen.pec_sheet(mask, nz // 2, 1, nx - 1, 2, ny - 2)
    b = boardgen.Board(f"brick{n}", nx, ny, nz, 1e-3, 1.2e-3, 0.5e-3, eps, mask, npml=npml, steps=1)
    i, j, k = nx // 2, max(1, ny // 2), nz // 2
    if k + 2 < nz:
        k += 1                                          # above the sheet
    b.sources = [boardgen.Source(i, j, k, boardgen.GAUSS, 1e6, 4e-12, 2e-12)]
    if i >= 2 and j >= 2:
        b.sources.append(boardgen.Source(i - 1, j - 1, k, boardgen.DGAUSS, 2.0, 4e-12, 2e-12, R=25.0))
    b.probes = [(i, j, k), (max(1, nx // 4), max(1, ny // 4), 0), (nx, ny, nz - 1)]
    b.plane_dft = (nz // 2, np.array([3e9, 17e9]))
    return b


def pmls(n):
    """Uneven with bare faces, all bare, one axis only."""
    d = [min(3, (v - 1) // 3) for v in n]               # leaves cells between two opposite slabs
    return [(0, d[0], d[1], 0, max(0, d[2] - 1), d[2]), (0,) * 6, (0, 0, 0, 0, d[2], d[2])]


@pytest.mark.parametrize("case", list(SHAPES.items()), ids=lambda c: "x".join(map(str, c[0])))
def test_every_shape_gives_the_marching_kernels_bits(F, case):
    n, brick = case
    nx, ny, nz = n
    rng = np.random.default_rng(3)
    init = [rng.standard_normal((nz + 1, ny + 1, nx + 1)).astype(np.float32) for _ in FIELDS]
    for q, npml in enumerate(pmls(n)):
        print(f"[gpu] bricks {n} pml {npml}", flush=True)
        b = board(n, npml, wide=q == 1)
        got = outcome(F, b, [5, 2, 4], None, brick, init)
        want = outcome(F, b, [5, 2, 4], MARCH, MARCHING, init)
        assert np.abs(want[-2]).max() > 0 or npml == (0,) * 6
        for c, (x, y) in enumerate(zip(got, want)):
            assert np.array_equal(x, y), (npml, c)


@pytest.mark.parametrize("n", [(48, 43, 36), (113, 44, 37), (57, 41, 45), (81, 67, 37)], ids=str)
def test_long_calls_of_every_shape(F, n):
    """2051 steps (graph replays and an odd last step) twice, the second from the other
    field copy."""
    print(f"[gpu] long calls {n}", flush=True)
    b = board(n, (4, 3, 2, 4, 3, 3))
    brick = {**EDGES, **SHAPES}[n]
    got = outcome(F, b, [2051, 2051], None, brick)
    want = outcome(F, b, [2051, 2051], MARCH, MARCHING)
    assert np.abs(want[0]).max() > 0
    for q, (x, y) in enumerate(zip(got, want)):
        assert np.array_equal(x, y), q


@pytest.mark.parametrize("case", list(EDGES.items()), ids=lambda c: "x".join(map(str, c[0])))
def test_kernel_of_the_edge_sizes(F, case):
    n, brick = case
    b = boardgen.random_tiny(sum(n), nx=n[0], ny=n[1], nz=n[2], npml=2, steps=2)
    outcome(F, b, [2], None, brick)

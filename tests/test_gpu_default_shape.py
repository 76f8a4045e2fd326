"""The default shape 64 x 14 x 2 set by name: what a handle runs untouched (bricks on
small boards), so the tuner, which times shapes by name, finds the kernel that users
get; the 64 x 14 x 2 marching kernel on the same small boards through a batched call."""
import numpy as np
import pytest

import boardgen
from test_gpu_brick import MARCH

pytestmark = pytest.mark.gpu

DEFAULT = (64, 14, 2)
FIELDS = range(12)


@pytest.fixture(scope="module")
def F():
    import torch
    assert torch.cuda.is_available()
    torch.cuda.set_device(0)
    from paper_1008_2602_amd import fdtd
    return fdtd


def results(F, g, ids, b, steps):
    shape = (b.nz + 1, b.ny + 1, b.nx + 1)
    return ([F.fdtd_get_probe(g, p, steps) for p in ids] + [F.fdtd_get_field(g, c, shape) for c in FIELDS]
            + [F.fdtd_get_plane_dft(g, b.ny, b.nx)])


def board(which, steps):
    b = boardgen.table1_board(steps=steps, source="resistive") if which == "table1" else boardgen.small_board(steps=steps)
    b.plane_dft = (b.nz // 2, np.array([2e9, 5e9]))
    return b


@pytest.mark.parametrize("which", ["table1", "small"])
def test_default_by_name_and_batched(F, which):
    """Bricks untouched, by name, and after another shape; the marching kernel of the
    default shape in a batched call and another marching shape: the same bits."""
    n = 75
    print(f"[gpu] default shape {which}", flush=True)
    b = board(which, n)
    outs = []
    for how in ("untouched", "named", "returned", "batched", "march"):
        g, ids = F.grid_from_board(b, tile={"named": DEFAULT, "march": MARCH}.get(how))
        try:
            if how == "returned":
                F.fdtd_set_tile(g, *MARCH)
                F.fdtd_step_n(g, 7)
                assert F.fdtd_get_route(g).brick_rows == 0
                F.fdtd_set_tile(g, *DEFAULT)
                F.fdtd_step_n(g, n - 7)
            elif how == "batched":
                F.fdtd_step_many([g], [n])
            else:
                F.fdtd_step_n(g, n)
            i, r = F.fdtd_get_info(g), F.fdtd_get_route(g)
            assert (i.tile_x, i.tile_y, i.tile_steps) == (MARCH if how == "march" else DEFAULT)
            assert (r.brick_rows > 0) == (how != "march")
            outs.append(results(F, g, ids, b, n))
        finally:
            F.fdtd_destroy_grid(g)
    assert np.abs(outs[0][0]).max() > 0
    for out in outs[1:]:
        for q, (x, y) in enumerate(zip(out, outs[0])):
            assert np.array_equal(x, y), q


@pytest.mark.parametrize("which", ["table1", "small"])
def test_tuner_keeps_the_kernel_an_untouched_handle_runs(F, which, tmp_path):
    """Bricks against the fastest marching shape, us per step: 4.7 and 5.9 on the Table 1
    board, 8.1 and 8.4 on the small board (too close to be timed anew here)."""
    from paper_1008_2602_amd import tune
    b = board(which, 8)
    b.plane_dft = None
    tiles = [tune.tune_board(b)]                         # the shipped choice
    if which == "table1":
        tiles.append(tune.tune_board(b, path=str(tmp_path / "tiles.json")))
    for tile in tiles:
        g, _ = F.grid_from_board(b, tile=tile)
        try:
            F.fdtd_step_n(g, 2)
            assert F.fdtd_get_route(g).brick_rows > 0, tile
        finally:
            F.fdtd_destroy_grid(g)

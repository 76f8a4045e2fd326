"""Small boards with rebuilt coefficients, whose tiles run the split kernels while few
blocks are in flight and whole material tiles in larger batches: the kernels that the
handle reports, and the node passes' bits alone and beside copies."""
import numpy as np
import pytest

from test_gpu_eps import NODE_ONLY
from test_gpu_lossy import slab_board
from test_gpu_marching import FIELDS, outcome

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    import torch
    assert torch.cuda.is_available()
    torch.cuda.set_device(0)
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the sizes are those of 256 compute units")
    from paper_1008_2602_amd import fdtd
    return fdtd


def board(kind, nx, ny, nz):
    b = slab_board(5, kind == "lossy", nx, ny, nz, True)
    if kind == "filled":
        b.eps_r_cell[:] = 4.2
    return b


# kind, sizes, whole tiles, rows of the material variant's tiles
CASES = [("slab", 64, 32, 86, 0, 10), ("lossy", 64, 32, 86, 0, 10), ("slab", 48, 43, 30, 1, 14),
         ("filled", 56, 39, 48, 1, 10), ("filled", 27, 45, 65, 1, 10), ("filled", 128, 77, 60, 1, 14),
         ("filled", 152, 63, 23, 1, 10)]


@pytest.mark.parametrize("case", CASES, ids=str)
def test_small_material_boards(F, case):
    kind, nx, ny, nz, whole, rows = case
    print(f"[gpu] small material {case}", flush=True)
    b = board(kind, nx, ny, nz)
    want = outcome(F, b, NODE_ONLY)[1]
    got = outcome(F, b, None)[1]
    for q, (x, y) in enumerate(zip(got, want)):
        assert np.array_equal(x, y), q
    g, _ = F.grid_from_board(b, max_steps=1)
    try:
        F.fdtd_step_n(g, 0)
        r = F.fdtd_get_route(g)
        assert (r.whole_tiles, r.material_tile_y) == (whole, rows)
    finally:
        F.fdtd_destroy_grid(g)


@pytest.mark.parametrize("copies", [2, 3, 5])    # 64 x 32 x 86: 6 tiles split, 9 and 15 whole
@pytest.mark.parametrize("kind", ["slab", "lossy", "filled"])
def test_batches_of_small_material_boards(F, kind, copies):
    print(f"[gpu] small material batch {kind} x{copies}", flush=True)
    b = board(kind, 64, 32, 86)
    shape = (b.nz + 1, b.ny + 1, b.nx + 1)
    steps = 7

    def make():
        g, ids = F.grid_from_board(b, max_steps=steps)
        rng = np.random.default_rng(3)
        for c in range(6):
            a = np.zeros(shape, np.float32)
            a[1:-1, 1:-1, 1:-1] = rng.standard_normal((b.nz - 1, b.ny - 1, b.nx - 1))
            if c < 3:
                a[(b.pec_edge_mask & (1 << c)) != 0] = 0
            F.fdtd_set_field(g, c, a)
        return g, ids

    def read(g, ids):
        return [F.fdtd_get_probe(g, p, steps) for p in ids] + [F.fdtd_get_field(g, c, shape) for c in FIELDS]

    made = [make() for _ in range(copies + 1)]
    try:
        F.fdtd_step_n(made[-1][0], steps)
        want = read(*made[-1])
        F.fdtd_step_many([g for g, _ in made[:-1]], [steps] * copies)
        for g, ids in made[:-1]:
            for q, (x, y) in enumerate(zip(read(g, ids), want)):
                assert np.array_equal(x, y), q
    finally:
        for g, _ in made:
            F.fdtd_destroy_grid(g)

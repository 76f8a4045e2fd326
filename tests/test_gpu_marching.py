"""The two-step marching kernels where a block walks a whole deep column (its ring of
z coefficients refilled on the way) and where a material board changes from whole
tiles of the material kernel to pieces: the same bits as the one-step kernel or the
node passes, from an arbitrary state."""
import numpy as np
import pytest

import boardgen
from test_gpu_eps import NODE_ONLY, two_step_equals_node_passes
from test_gpu_lossy import slab_board
from test_gpu_parity import FIELDS as NAMES, compare_fields, random_state

pytestmark = pytest.mark.gpu

FIELDS = range(12)
# 2 x 130 tiles of 64 x 14 x 2: more than the device's 256 blocks, so tiles stay
# whole but for a few
NX, NY = 66, 1430
ONE_STEP = (64, 15, 1)


@pytest.fixture(scope="module")
def F():
    import torch
    assert torch.cuda.is_available()
    torch.cuda.set_device(0)
    from paper_1008_2602_amd import fdtd
    return fdtd


def outcome(F, b, tile, steps=5):
    g, ids = F.grid_from_board(b, max_steps=steps, tile=tile)
    shape = (b.nz + 1, b.ny + 1, b.nx + 1)
    rng = np.random.default_rng(5)
    some = rng.standard_normal(100003).astype(np.float32)
    try:
        for c in range(6):   # E and H off the walls and PEC edges; D and B start from zero
            a = np.zeros(shape, np.float32)
            inner = a[1:-1, 1:-1, 1:-1]
            inner[:] = np.resize(np.roll(some, 17 * c), inner.shape)
            if c < 3:
                a[(b.pec_edge_mask & (1 << c)) != 0] = 0
            F.fdtd_set_field(g, c, a)
        F.fdtd_step_n(g, steps)
        info = F.fdtd_get_info(g)
        return info, [F.fdtd_get_probe(g, p, steps) for p in ids] + [F.fdtd_get_field(g, c, shape) for c in FIELDS]
    finally:
        F.fdtd_destroy_grid(g)


@pytest.mark.parametrize("tile", [(64, 14, 2), (64, 9, 2)], ids=str)
@pytest.mark.parametrize("nz", [66, 131])
def test_deep_columns_refill_the_z_coefficients(F, nz, tile):
    print(f"[gpu] deep columns nz={nz} {tile}", flush=True)
    b = slab_board(5, False, NX, NY, nz, False)
    got = outcome(F, b, tile)[1]
    want = outcome(F, b, ONE_STEP)[1]
    for q, (x, y) in enumerate(zip(got, want)):
        assert np.array_equal(x, y), q


# about 200 tile planes per compute unit (of 256): 260 tiles of 196 planes and of 197
@pytest.mark.parametrize("nz", [196, 197])
@pytest.mark.parametrize("lossy", [False, True], ids=["eps_rw", "eps_rw+lossy"])
def test_material_boards_either_side_of_the_whole_tile_rule(F, nz, lossy):
    print(f"[gpu] material rule nz={nz} lossy={lossy}", flush=True)
    b = slab_board(5, lossy, NX, NY, nz, True)
    info, got = outcome(F, b, None)
    assert info.material_two_step == 1 and info.material_split > 0
    want = outcome(F, b, NODE_ONLY)[1]
    for q, (x, y) in enumerate(zip(got, want)):
        assert np.array_equal(x, y), q


def test_classes_of_repeating_and_changing_rows(F, oracle_mod):
    """Node classes where runs of equal cells of 1 to 9 columns, PEC marks, a
    conductivity step and both kinds of sources meet: 5 steps from an arbitrary state
    against the oracle."""
    nx, ny, nz = 61, 24, 20
    rng = np.random.default_rng(8)
    eps, mask = boardgen.air(nx, ny, nz)
    for k in range(nz):
        for j in range(ny):
            i = 0
            while i < nx:
                w = int(rng.integers(1, 10))
                eps[k, j, i:i + w] = rng.choice([1.0, 2.2, 4.2])
                i += w
    boardgen.pec_sheet(mask, 10, 6, 40, 6, 17)
    b = boardgen.Board("rows", nx, ny, nz, 0.5e-3, 0.5e-3, 0.1e-3, eps, mask, npml=(4,) * 6, steps=5,
                       pml_eps_rw=True)
    sig = np.zeros(eps.shape, np.float32)
    sig[8:12, 6:18, 9:10] = 0.05
    sig[8:12, 6:18, 20:41] = 0.02
    b.sigma_cell = sig
    b.sources = [boardgen.Source(30, 12, 12, boardgen.GAUSS, 2.0, 4e-12, 1.2e-12, R=20.0),
                 boardgen.Source(31, 12, 12, boardgen.DGAUSS, 1e6, 5e-12, 1.5e-12)]
    b.probes = [(32, 12, 12)]
    st = random_state(oracle_mod, b, seed=2)
    init = {n: st[n].copy() for n in NAMES}
    ref = oracle_mod.run(b, state=st)
    compare_fields(ref.state, two_step_equals_node_passes(F, b, init), b, 2e-5, elem_tol=1e-5)

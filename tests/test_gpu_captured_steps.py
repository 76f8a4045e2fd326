"""Stepping recorded into the caller's own HIP graph.  The field kernels take the step
and the field copy from the device counters, so a recorded fdtd_step_n advances the
board at every replay; a small board, whose pairs of steps otherwise run in bricks
that are told which copy to read, does as well."""
import numpy as np
import pytest

import boardgen

pytestmark = pytest.mark.gpu

FIELDS = range(12)


@pytest.fixture(scope="module")
def F():
    import torch
    assert torch.cuda.is_available()
    torch.cuda.set_device(0)
    from paper_1008_2602_amd import fdtd
    return fdtd


def images(F, g, b):
    shape = (b.nz + 1, b.ny + 1, b.nx + 1)
    return [F.fdtd_get_field(g, c, shape) for c in FIELDS]


# 2 steps: one launch, so every other replay starts from the other field copy;
# 3: a pair and a single step; 40: more than a chunk of the library's own graphs
@pytest.mark.parametrize("n", [2, 3, 40])
def test_replays_of_a_recorded_call_advance_the_board(F, n):
    import torch
    replays = 5
    b = boardgen.table1_board(steps=4 + (replays + 1) * n, source="resistive")
    print(f"[gpu] captured step_n({n})", flush=True)
    st = torch.cuda.Stream()
    g, _ = F.grid_from_board(b, hip_stream=st.cuda_stream)
    h, _ = F.grid_from_board(b)
    try:
        F.fdtd_step_n(g, 4)                     # set-up done, two launches
        F.fdtd_step_n(h, 4)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=st):
            F.fdtd_step_n(g, n)
        for _ in range(replays):                # an odd number: the host's field copy agrees again
            with torch.cuda.stream(st):
                graph.replay()
            torch.cuda.synchronize()
        F.fdtd_step_n(h, replays * n)
        want = images(F, h, b)
        assert np.abs(want[2]).max() > 0
        for c, (x, y) in enumerate(zip(images(F, g, b), want)):
            assert np.array_equal(x, y), c
        # and the board steps on from there outside a graph
        F.fdtd_step_n(g, n)
        F.fdtd_step_n(h, n)
        for c, (x, y) in enumerate(zip(images(F, g, b), images(F, h, b))):
            assert np.array_equal(x, y), c
    finally:
        F.fdtd_destroy_grid(g)
        F.fdtd_destroy_grid(h)

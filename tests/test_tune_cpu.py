"""What the tuner times, without a GPU: a modelled library whose shapes differ in what
their steps take, in what the time inside their kernels takes and in what building a
batched call's plan takes.  The tuner keeps the shape whose steps are fastest."""
import types

import pytest

from paper_1008_2602_amd import fdtd, tune

SHAPES = [(64, 15, 1), (64, 9, 2), (64, 14, 2)]
#        per step, per step inside kernels, per plan (seconds)
COST = {(64, 15, 1): (9e-6, 5e-6, 1e-3), (64, 9, 2): (6e-6, 3e-6, 1e-3), (64, 14, 2): (5e-6, 4e-6, 6e-3)}


@pytest.fixture
def model(monkeypatch):
    state = types.SimpleNamespace(now=0.0, shape=SHAPES[0], plans=set(), kernel=0.0, steps=0, cap=0)

    def work(n):
        state.steps += n
        assert state.steps < state.cap, "more steps than the scratch handles have"
        state.now += n * COST[state.shape][0] + 12e-6
        state.kernel += n * COST[state.shape][1]

    def step_many(gs, ns):
        if (state.shape, tuple(ns)) not in state.plans:
            state.plans.add((state.shape, tuple(ns)))
            state.now += COST[state.shape][2]
        work(ns[0])

    def scratch(F, board, steps):
        state.cap = steps
        return object()

    monkeypatch.setattr(fdtd, "fdtd_tile_shapes", lambda: list(SHAPES))
    monkeypatch.setattr(fdtd, "fdtd_set_tile", lambda g, *s: setattr(state, "shape", s))
    monkeypatch.setattr(fdtd, "fdtd_step_n", lambda g, n: work(n))
    monkeypatch.setattr(fdtd, "fdtd_step_many", step_many)
    monkeypatch.setattr(fdtd, "fdtd_synchronize", lambda g: None)
    monkeypatch.setattr(fdtd, "fdtd_set_timing", lambda g, on: None)

    def get_timing(g):
        ms, state.kernel = state.kernel * 1e3, 0.0
        return ms, 1
    monkeypatch.setattr(fdtd, "fdtd_get_timing", get_timing)
    monkeypatch.setattr(fdtd, "fdtd_destroy_grid", lambda g: None)
    monkeypatch.setattr(tune, "_scratch", scratch)
    monkeypatch.setattr(tune.time, "perf_counter", lambda: state.now)
    return state


def board(n=40):
    return types.SimpleNamespace(nx=n, ny=n, nz=n, npml=(8,) * 6, plane_dft=None)


@pytest.mark.parametrize("n", [40, 400])
def test_board_tuner_keeps_the_fastest_steps(model, tmp_path, n):
    assert tune.tune_board(board(n), path=str(tmp_path / "t.json")) == (64, 14, 2)


@pytest.mark.parametrize("n", [40, 400])
def test_batch_tuner_leaves_the_plan_out(model, tmp_path, n):
    path = str(tmp_path / "t.json")
    assert tune.tune_batch([board(n)] * 4, path=path) == (64, 14, 2)
    # kept: the next call times nothing
    now = model.now
    assert tune.tune_batch([board(n)] * 4, path=path) == (64, 14, 2) and model.now == now

"""The probe FFT at every transform size up to 2^18 and three larger ones (one-column
blocks, spectra longer than the pinned buffer), against numpy in FP64: within 30
rounding errors of the largest bin, and no further off than the conditioning of an
FFT of that length (a radix-2 FFT's error grows with log2 n: eps log2(n) of the
2-norm)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    import torch
    assert torch.cuda.is_available()
    torch.cuda.set_device(0)
    from paper_1008_2602_amd import fdtd
    return fdtd


def test_every_transform_size(F):
    nx, ny, nz = 16, 14, 10
    g = F.fdtd_create_grid(nx, ny, nz, 1e-3, 1e-3, 1e-3, npml=(3,) * 6, max_steps=700)
    try:
        F.fdtd_set_materials(g, np.ones((nz, ny, nx), np.float32))
        F.fdtd_add_source(g, 7, 6, 4, F.FDTD_WAVE_GAUSS, 1e6, 1e-11, 3e-12)
        p = F.fdtd_add_probe(g, 9, 7, 5)
        done = 0
        for steps, sizes in ((2, [2]), (3, [4, 8]), (13, [16, 64]), (700, [1 << l for l in range(10, 19)] +
                                                             [1 << 20, 1 << 23, 1 << 25])):
            F.fdtd_step_n(g, steps - done)
            done = steps
            e = F.fdtd_get_probe(g, p, steps).astype(np.float64)
            for n in sizes:
                print(f"[gpu] fft {n}", flush=True)
                got = F.fdtd_probe_fft(g, p, n)
                ref = np.fft.rfft(e, n)
                eps = np.finfo(np.float64).eps
                assert got.shape == ref.shape
                assert np.linalg.norm(got - ref) <= 2 * eps * np.log2(2 * n) * max(np.linalg.norm(ref), 1e-300), n
                assert np.abs(got - ref).max() <= 30 * eps * max(np.abs(e).sum(), 1e-300), n
                if n <= 1 << 20:
                    assert np.array_equal(F.fdtd_probe_fft_noalloc(g, p, n), got), n
        assert np.abs(e).max() > 0
    finally:
        F.fdtd_destroy_grid(g)


def test_small_transforms_and_the_largest(F):
    """2 to 512 points, each with a full series and a padded one, and 2^26, the one size
    whose rows are one to a block: with the bounds above."""
    nx, ny, nz = 16, 14, 10
    g = F.fdtd_create_grid(nx, ny, nz, 1e-3, 1e-3, 1e-3, npml=(3,) * 6, max_steps=600)
    try:
        F.fdtd_set_materials(g, np.ones((nz, ny, nx), np.float32))
        F.fdtd_add_source(g, 7, 6, 4, F.FDTD_WAVE_GAUSS, 1e6, 3e-12, 2e-12)
        p = F.fdtd_add_probe(g, 8, 6, 4)
        eps = np.finfo(np.float64).eps
        done = 0
        for steps, n in [(s, 1 << l) for l in range(1, 10) for s in ((1 << l) - (1 << l) // 4, 1 << l)] + [(600, 1 << 26)]:
            print(f"[gpu] fft {n} of {steps} samples", flush=True)
            F.fdtd_step_n(g, steps - done)
            done = steps
            e = F.fdtd_get_probe(g, p, steps).astype(np.float64)
            assert np.abs(e).max() > 0
            got = F.fdtd_probe_fft(g, p, n)
            ref = np.fft.rfft(e, n)
            assert got.shape == ref.shape
            assert np.linalg.norm(got - ref) <= 2 * eps * np.log2(2 * n) * np.linalg.norm(ref), n
            assert np.abs(got - ref).max() <= 30 * eps * np.abs(e).sum(), n
            if n <= 1 << 20:
                assert np.array_equal(F.fdtd_probe_fft_noalloc(g, p, n), got), n
    finally:
        F.fdtd_destroy_grid(g)

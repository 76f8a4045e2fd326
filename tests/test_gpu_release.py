"""A handle whose memory comes from the caller's allocator is released without waiting
for other work on the device (a server releases finished boards while others step)."""
import numpy as np
import pytest

import boardgen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    import torch
    assert torch.cuda.is_available()
    torch.cuda.set_device(0)
    from paper_1008_2602_amd import fdtd
    return fdtd


def test_release_does_not_wait_for_other_work(F):
    import torch
    b = boardgen.small_board(steps=16)
    alloc = F.TorchAllocator()
    other = torch.cuda.Stream()
    x = torch.zeros(1 << 28, device="cuda")            # 1 GiB: about 0.4 ms per pass
    x.add_(1.0)
    F.fdtd_destroy_grid(F.grid_from_board(b, allocator=alloc)[0])   # first uses of everything
    for _ in range(2):
        g, ids = F.grid_from_board(b, allocator=alloc)
        F.fdtd_step_n(g, b.steps)
        assert np.isfinite(F.fdtd_get_probe(g, ids[0], b.steps)).all()
        torch.cuda.synchronize()
        with torch.cuda.stream(other):
            for _ in range(800):                       # 0.3 s of work
                x.add_(1.0)
        F.fdtd_destroy_grid(g)
        assert not other.query(), "the release waited for another stream's work"
        torch.cuda.synchronize()

"""Positions and species read back in one copy: every bit of what the box was built from, for boxes with room
left and for an empty one, on the default stream and on another."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [0, 1, 63, 1000])
@pytest.mark.parametrize("other_stream", [False, True])
def test_read(n, other_stream):
    from paper_1408_3764_amd.box import Box
    rng = np.random.default_rng(n)
    pos = rng.uniform(0.0, 20.0, (n, 3))
    sp = rng.integers(0, 2, n).astype(np.int32)
    s = torch.cuda.Stream() if other_stream else None
    b = Box(pos, 20.0, 2.5, eps=np.ones((2, 2)), sigma=np.full((2, 2), 0.1), species=sp, max_n=n + 37, cell_cap=64,
            stream=s)
    for got in (b.particles(), b.export_state()[:2]):
        assert got[0].shape == (n, 3) and got[0].dtype == np.float64 and got[0].flags["C_CONTIGUOUS"]
        assert got[0].tobytes() == pos.tobytes()
        assert got[1].dtype == np.int32 and (got[1] == sp).all()
        got[0][:] = 0.0      # the caller's own arrays
    assert b.export_state()[2]["n"] == n

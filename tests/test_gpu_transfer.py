"""The library's small transfers: every size around the limits of the fast ways
(4 KB read, 2 KB written), odd bytes and odd addresses, behind queued work, and
from more threads than there are slots.  Bytes are compared exactly."""
import threading

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _keeper():
    from paper_1408_3764_amd.box import Box
    return Box(np.array([[1.0, 2.0, 3.0]]), [8.0] * 3, 2.5, max_n=2)


@pytest.mark.parametrize("n", [0, 1, 3, 4, 8, 2044, 2047, 2048, 2052, 4092, 4096, 4097, 4100, 70000])
@pytest.mark.parametrize("off", [0, 1, 4])
def test_bytes_come_and_go(n, off):
    from paper_1408_3764_amd import _lib
    box = _keeper()
    want = np.random.default_rng(n + off).integers(0, 256, n, dtype=np.uint8)
    d = torch.zeros(n + 8, dtype=torch.uint8, device="cuda")
    _lib.gcmc_write(d[off:off + n], want)
    assert np.array_equal(d.cpu().numpy(), np.concatenate([np.zeros(off, np.uint8), want, np.zeros(8 - off, np.uint8)]))
    got = np.empty(n, np.uint8)
    for _ in range(3):
        got[:] = 0
        _lib.gcmc_read(got, d[off:off + n])
        assert np.array_equal(got, want)
    box.close()


def test_read_is_behind_the_streams_work():
    from paper_1408_3764_amd import _lib
    box = _keeper()
    s = torch.cuda.Stream()
    d = torch.zeros(512, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    got = np.empty(512)
    for k in range(1, 6):
        with torch.cuda.stream(s):
            for _ in range(50 * k):           # up to 250 launches ahead of the read
                d.add_(1.0)
            big = torch.full((1 << 27,), 1.0, dtype=torch.float64, device="cuda")   # past the polled time
            d.add_(big[:512])
        _lib.gcmc_read(got, d, s)
        assert (got == sum(50 * j + 1 for j in range(1, k + 1))).all()
        del big
    box.close()


def test_more_threads_than_slots():
    from paper_1408_3764_amd import _lib
    box = _keeper()
    bad = []

    def work(t):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            d = torch.full((100,), float(t), dtype=torch.float64, device="cuda")
            got = np.empty(100)
            for k in range(20):
                _lib.gcmc_write(d, np.full(100, t + 1000.0 * k), s)
                _lib.gcmc_read(got, d, s)
                if not (got == t + 1000.0 * k).all():
                    bad.append((t, k))

    threads = [threading.Thread(target=work, args=(t,)) for t in range(24)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
    box.close()


def test_wrong_positions_are_still_named():
    """A tensor of the wrong N is refused as a value, also on a box that holds an error."""
    from paper_1408_3764_amd import _lib
    box = _keeper()
    for shape in ((2, 3), (1, 4), (3,), (0, 3)):
        with pytest.raises(ValueError):
            box.set_positions_device(torch.zeros(shape, dtype=torch.float64, device="cuda"))
    with pytest.raises(TypeError):
        box.set_positions_device(torch.zeros((1, 3), dtype=torch.float32, device="cuda"))
    with pytest.raises(ValueError):
        box.set_positions_device(torch.zeros((2, 3), dtype=torch.float32, device="cuda"))
    with pytest.raises(_lib.GcmcError):
        box.set_positions_device(torch.full((1, 3), 9.0, dtype=torch.float64, device="cuda"))
    with pytest.raises(ValueError):
        box.set_positions_device(torch.zeros((2, 3), dtype=torch.float64, device="cuda"))
    box.close()

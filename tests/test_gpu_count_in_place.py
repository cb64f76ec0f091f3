"""Counts whose prefix offsets overwrite the offsets they are counted by:
every event must be counted by the offsets as they came in."""
import numpy as np
import pytest

from paper_1906_06242_amd import hepk as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("shift", [0, 3, -3])
@pytest.mark.parametrize("n", [0, 1, 255, 256, 257, 4097, 1048577, 2100000])
def test_count_in_place(n, shift, masked):
    """offsets_out = offsets, and the two arrays three entries apart."""
    import torch
    print("count in place", n, shift, masked, flush=True)
    rng = np.random.default_rng(n + 2)
    off = np.concatenate([[0], np.cumsum(rng.poisson(3.0, n))]).astype(np.int64)
    om = rng.integers(0, 2, max(1, int(off[-1]))).astype(np.uint8)
    c = np.concatenate([[0], np.cumsum(om[:int(off[-1])], dtype=np.int64)])
    want = (c[off[1:]] - c[off[:-1]]) if masked else np.diff(off)
    buf = torch.zeros(n + 8, dtype=torch.int64, device="cuda")
    src, dst = buf[3:n + 4], buf[3 + shift:n + 4 + shift]
    src.copy_(torch.from_numpy(off))
    out = torch.empty(max(1, n), dtype=torch.int32, device="cuda")
    mask = torch.from_numpy(om).cuda() if masked else None
    H._call("hepk_reduce", H.COUNT, H._ptr(src), n, None, H.F32, H._ptr(mask), None, H._ptr(out), None, H._ptr(dst),
            H._stream())
    assert np.array_equal(out.cpu().numpy()[:n], want)
    assert np.array_equal(dst.cpu().numpy(), np.concatenate([[0], np.cumsum(want, dtype=np.int64)]))


def test_count_over_event_mask():
    """offsets_out in the event mask's own memory."""
    import torch
    n = 300000
    rng = np.random.default_rng(9)
    off = np.concatenate([[0], np.cumsum(rng.poisson(3.0, n))]).astype(np.int64)
    em = rng.integers(0, 2, n).astype(np.uint8)
    want = np.diff(off) * em
    buf = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    mask = buf.view(torch.uint8)[4 * n:5 * n]
    mask.copy_(torch.from_numpy(em))
    src, out = torch.from_numpy(off).cuda(), torch.empty(n, dtype=torch.int32, device="cuda")
    H._call("hepk_reduce", H.COUNT, H._ptr(src), n, None, H.F32, None, H._ptr(mask),
            H._ptr(out), None, H._ptr(buf), H._stream())
    assert np.array_equal(out.cpu().numpy(), want)
    assert np.array_equal(buf.cpu().numpy(), np.concatenate([[0], np.cumsum(want, dtype=np.int64)]))

"""Counts with prefix offsets at the edges of their spans: exact against numpy."""
import numpy as np
import pytest

from paper_1906_06242_amd import hepk as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("n", [0, 1, 63, 64, 65, 255, 256, 257, 1023, 1025, 4097, 524289, 1048575, 1048576, 1048577,
                               2100000])
def test_count_offsets(n, shift, masked):
    """1048576 = 4096 spans of 256 events: one event more doubles the span."""
    import torch
    print("count offsets", n, shift, masked, flush=True)
    rng = np.random.default_rng(n + 1)
    off = np.concatenate([[0], np.cumsum(rng.poisson(3.0, n))]).astype(np.int64)
    m = int(off[-1])
    om = rng.integers(0, 2, m).astype(np.uint8) if masked else np.ones(m, np.uint8)
    em = rng.integers(0, 4, n).astype(np.uint8) if masked else np.ones(n, np.uint8)
    c = np.concatenate([[0], np.cumsum(om, dtype=np.int64)])
    want = ((c[off[1:]] - c[off[:-1]]) * (em != 0)).astype(np.int32)
    dev = lambda a: torch.from_numpy(a).cuda() if a.size else None  # noqa: E731
    out = torch.full((n + shift + 8,), -7, dtype=torch.int32, device="cuda")
    got, offs = H.reduce(H.COUNT, torch.from_numpy(off).cuda(), obj_mask=dev(om) if masked else None,
                         evt_mask=dev(em) if masked else None, want_offsets=True, out=out[shift:shift + n])
    assert np.array_equal(got.cpu().numpy(), want)
    assert np.array_equal(offs.cpu().numpy(), np.concatenate([[0], np.cumsum(want, dtype=np.int64)]))
    rest = out.cpu().numpy()
    assert np.all(rest[:shift] == -7) and np.all(rest[shift + n:] == -7)

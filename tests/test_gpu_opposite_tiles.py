"""Opposite-sign selection at the edges of its staged tiles: the mask bytes
must equal the oracle's (pT order with ties, NaN and charge 0)."""
import numpy as np
import pytest

from oracle import ref
from paper_1906_06242_amd import hepk as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("name", ["eight", "nine", "long", "ragged", "one event"])
def test_opposite_sign_tiles(name, dtype, masked):
    """512 objects of a tile are staged: 64 events of 8 fill it, of 9 run in
    two parts, events of 511 to 700 objects stand at and beyond it."""
    import torch
    print("opposite sign tiles", name, dtype, masked, flush=True)
    rng = np.random.default_rng(11)
    n = 1 if name == "one event" else 1000
    counts = {"eight": np.full(n, 8), "nine": np.full(n, 9), "long": rng.poisson(2.0, n), "ragged": rng.poisson(6.0, n),
              "one event": np.array([256])}[name]
    if name == "long":
        counts[[5, 70, 71, 200, 999]] = [511, 512, 513, 700, 512]
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    m = int(off[-1])
    pt = rng.choice(np.array([20, 25, 25, 30.5, 41, np.nan, np.inf, -1], np.float32), m)
    pt = pt.astype(np.float16 if dtype == "f16" else np.float32)
    q = rng.integers(-1, 2, m).astype(np.int32)
    om = rng.integers(0, 2, m).astype(np.uint8) * 3 if masked else None
    dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    got = H.select_opposite_sign(dev(off), dev(pt), dev(q), dev(om) if masked else None)
    assert np.array_equal(got.cpu().numpy(), ref.select_opposite_sign(off, pt, q, om))

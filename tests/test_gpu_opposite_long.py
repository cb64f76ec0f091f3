"""Opposite-sign pairs of events with many objects, which the wavefront takes
one by one: ties and signed zeros across lanes, NaN and infinities, events with
one sign only, against the oracle; also with the mask written over itself."""
import numpy as np
import pytest

from oracle import ref
from paper_1906_06242_amd import hepk as H

pytestmark = pytest.mark.gpu

COUNTS = {"63 to 65": [63, 64, 65] * 40, "hundreds": [100, 127, 128, 129, 256, 300, 0, 511, 512] * 9,
          "beyond staging": [513, 1, 600, 0, 1000, 4097, 2, 2] * 4, "eight": [512] + [64] * 8 + [63] * 57,
          "few events": [3, 1, 0, 2, 5], "mixed": [1] * 60 + [700] + [2] * 70 + [200, 200, 0]}
POOLS = {"ties": [20, 25, 30], "zeros": [0.0, -0.0], "special": [np.nan, np.inf, -np.inf, -1, 1e-8, 40], "nan": [np.nan]}


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("pool", list(POOLS))
@pytest.mark.parametrize("name", list(COUNTS))
def test_opposite_sign_long(name, pool, dtype):
    import torch
    print("opposite sign long", name, pool, dtype, flush=True)
    rng = np.random.default_rng(12)
    off = np.concatenate([[0], np.cumsum(COUNTS[name])]).astype(np.int64)
    m = int(off[-1])
    pt = rng.choice(np.array(POOLS[pool], np.float32), m).astype(np.float16 if dtype == "f16" else np.float32)
    q = rng.integers(-1, 2, m).astype(np.int32)
    q[off[1]:off[2]] = np.abs(q[off[1]:off[2]])  # an event of one sign
    om = (rng.random(m) < 0.3).astype(np.uint8) * 2
    dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    o, p, c, k = dev(off), dev(pt), dev(q), dev(om)
    want = ref.select_opposite_sign(off, pt, q, om)
    assert np.array_equal(H.select_opposite_sign(o, p, c).cpu().numpy(), ref.select_opposite_sign(off, pt, q, None))
    assert np.array_equal(H.select_opposite_sign(o, p, c, k).cpu().numpy(), want)
    assert np.array_equal(H.select_opposite_sign(o, p, c, k, out=k).cpu().numpy(), want)

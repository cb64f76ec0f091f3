"""Triplet search at the edges of its staged tiles: masses and indices equal to
the oracle's, bit for bit (the same float32 arithmetic and choice)."""
import numpy as np
import pytest

from oracle import ref
from paper_1906_06242_amd import hepk as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["one event of 384", "one event of 385", "six each", "seven each", "mixed", "pairs"])
def test_triplet_tiles(name):
    """384 objects of a 64-event tile are staged; one event of 384 has 9.3
    million triplets, events of two have none."""
    import torch
    print("triplet tiles", name, flush=True)
    rng = np.random.default_rng(31)
    counts = {"one event of 384": [384], "one event of 385": [385], "six each": [6] * 200, "seven each": [7] * 200,
              "mixed": [0, 1, 2, 3, 60, 0, 0, 2] * 40, "pairs": [2] * 100}[name]
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    m = int(off[-1])
    v = [rng.normal(0, 40, m).astype(np.float32) for _ in range(3)]
    # few distinct energies: ties in the distance to the target
    en = (np.sqrt(v[0] ** 2 + v[1] ** 2 + v[2] ** 2) + rng.integers(0, 3, m)).astype(np.float32)
    if m > 20:
        v[0][::53] = np.inf
        v[0][10:16], v[1][10:16], v[2][10:16], en[10:16] = v[0][10], v[1][10], v[2][10], en[10]
    dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    wm, wi = ref.best_triplet(off, *v, en, None, 172.0)
    gm, gi = H.best_triplet(dev(off), *(dev(a) for a in v), dev(en), None, 172.0)
    gm, gi = gm.cpu().numpy(), gi.cpu().numpy()
    assert np.array_equal(gi, wi)
    assert np.array_equal(np.isnan(gm), np.isnan(wm))
    ok = ~np.isnan(wm)
    assert np.array_equal(gm[ok].view(np.uint32), wm[ok].view(np.uint32))

"""The clean mask of hepk_match_dr when nothing else is asked for: equal to the
oracle's, over tile edges, masks, cones and non-finite content."""
import numpy as np
import pytest

from oracle import ref
from paper_1906_06242_amd import hepk as H

pytestmark = pytest.mark.gpu


def draw(rng, counts, dtype, bad):
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    m = int(off[-1])
    eta, phi = rng.uniform(-2.5, 2.5, m), rng.uniform(-np.pi, np.pi, m)
    if bad and m:
        at = rng.integers(0, m, max(1, m // 50))
        eta[at] = rng.choice([np.nan, np.inf, -np.inf], at.size)
    dt = np.float16 if dtype == "f16" else np.float32
    return off, eta.astype(dt), phi.astype(dt), rng.integers(0, 3, m).astype(np.uint8)


@pytest.mark.parametrize("dr", [0.0, 0.4, 3.0, float("inf")])
@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("name", ["usual", "full", "beyond", "long", "one event", "no b"])
def test_match_clean(name, dtype, dr):
    """512 a and 256 b objects of a 64-event tile are staged."""
    import torch
    print("match clean", name, dtype, dr, flush=True)
    rng = np.random.default_rng(21)
    n = 1 if name == "one event" else 700
    ca, cb = {"usual": (rng.poisson(5.0, n), rng.poisson(1.5, n)), "full": (np.full(n, 8), np.full(n, 4)),
              "beyond": (np.full(n, 9), np.full(n, 3)), "long": (rng.poisson(5.0, n), rng.poisson(1.5, n)),
              "one event": (np.array([300]), np.array([200])), "no b": (rng.poisson(5.0, n), np.zeros(n, int))}[name]
    if name == "long":
        ca[[3, 200]], cb[[3, 400]] = [400, 600], [100, 300]
    off_a, ea, pa, ma = draw(rng, ca, dtype, True)
    off_b, eb, pb, mb = draw(rng, cb, dtype, True)
    if eb.size == 0:  # a valid pointer for a column of no objects
        eb = pb = np.zeros(1, ea.dtype)
        mb = np.zeros(1, np.uint8)
    dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    for use_a in (False, True):
        for use_b in (False, True):
            got = H.match_dr(dev(off_a), dev(ea), dev(pa), dev(off_b), dev(eb), dev(pb), dr,
                             mask_a=dev(ma) if use_a else None, mask_b=dev(mb) if use_b else None, want=("clean",))[2]
            want = ref.match_dr(off_a, ea, pa, off_b, eb, pb, dr, mask_a=ma if use_a else None,
                                mask_b=mb if use_b else None)[2]
            assert np.array_equal(got.cpu().numpy(), want), (use_a, use_b)

"""NaN depths in the sort-last composite: a layer is inserted behind every layer before
it that is not later than it, and no depth compares as later than NaN or NaN as later
than any; as many layers are composited as have a depth below +inf.  Against that
rule written out per pixel."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def reference(rgba, depth):
    n, (h, w) = len(depth), depth[0].shape
    out = np.zeros((h, w, 4), np.float32)
    for y in range(h):
        for x in range(w):
            order = []
            for l in range(n):
                at = len(order)
                while at > 0 and depth[order[at - 1]][y, x] > depth[l][y, x]:
                    at -= 1
                order.insert(at, l)
            c = np.zeros(4, np.float32)
            for l in order[:sum(bool(d[y, x] < np.inf) for d in depth)]:
                t = np.float64(np.float32(1) - c[3])
                c = (t * rgba[l][y, x].astype(np.float64) + c.astype(np.float64)).astype(np.float32)
            out[y, x] = c
    return out


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 8, 9, 16])
def test_nan_depths(n):
    import torch
    from paper_1611_09048_amd import Context
    w, h = 37, 19
    rng = np.random.default_rng(n)
    # 64 levels; every step rounds once on both sides (the product is exact in 64 bits)
    rgba = [(rng.integers(0, 64, size=(h, w, 4)) / 64).astype(np.float32) for _ in range(n)]
    values = np.array([0.5, 1.0, 2.0, 3.5, np.inf, -np.inf, np.nan, np.nan], dtype=np.float32)
    depth = [rng.choice(values, size=(h, w)) for _ in range(n)]
    for d in depth:
        d[0, 0] = np.nan                                      # nothing below +inf: not covered
    r = [torch.from_numpy(x).cuda() for x in rgba]
    d = [torch.from_numpy(x).cuda() for x in depth]
    out = torch.full((h, w, 4), float("nan"), device="cuda")
    torch.cuda.synchronize()
    with Context(device=0) as ctx:
        ctx.composite([t.data_ptr() for t in r], [t.data_ptr() for t in d], w, h, out.data_ptr())
    got, want = out.cpu().numpy(), reference(rgba, depth)
    assert np.abs(got - want).max() <= 2.0 ** -22 and (got[0, 0] == 0).all()

"""tet_locate on both sides of the rule for its two descents (coordinates that
are 0 or at least 2^-29, and smaller ones), against the oracle."""
import numpy as np
import pytest

import oracle
import synthetic

pytestmark = pytest.mark.gpu
TINY = synthetic.scene("tiny")


@pytest.mark.parametrize("depth", [0, 1, 2, 9, 16])
def test_small_coordinates(depth):
    import torch
    assert torch.cuda.is_available(), "no GPU"
    import paper_2506_11510_amd as tv
    print("case small coordinates, depth", depth, flush=True)
    opts = dict(TINY["build"], uniform_depth=depth)
    if depth > 2:
        opts = dict(TINY["build"], want_mode=2, max_depth=depth, rand_seed=3, rand_thresh=50000)
    density = np.ascontiguousarray(TINY["density_fn"]())
    g = tv.leb_build(torch.from_numpy(density).cuda(), 64, TINY["camera"], build=opts)
    o = oracle.leb_build(density, 64, TINY["camera"], opts)
    rng = np.random.default_rng(depth)
    pts = rng.random((4096, 3)).astype(np.float32)
    small = np.float32(2.0) ** rng.integers(-149, -20, 4096).astype(np.float32)
    small[::7] = np.float32(2.0 ** -29)
    small[1::7] = np.nextafter(np.float32(2.0 ** -29), np.float32(0))
    small[2::7] = 0
    pts[np.arange(4096), rng.integers(0, 3, 4096)] = small
    pts[::5, 1] = np.float32(1) - pts[::5, 0]
    pts[::11] = np.sort(pts[::11], axis=1)
    pts[3::11, 2] = pts[3::11, 1]
    assert np.array_equal(g.locate(pts), o.locate(pts))

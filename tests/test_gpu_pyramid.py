"""Builds at the volume sizes where the pyramid's launches change (no level,
one, the small levels alone, the first size with a level above them), dense
and sparse, against the oracle."""
import numpy as np
import pytest

import oracle
import synthetic
from parity import assert_grids_equal

pytestmark = pytest.mark.gpu
TINY = synthetic.scene("tiny")


@pytest.mark.parametrize("n, sparse", [(1, 0), (2, 0), (4, 0), (8, 0), (16, 0), (32, 0), (64, 0),
                                       (8, 1), (16, 1), (32, 1), (64, 1)])  # (bricks are 8^3)
def test_sizes(n, sparse):
    import torch
    assert torch.cuda.is_available(), "no GPU"
    import paper_2506_11510_amd as tv
    print("case pyramid, n", n, "sparse", sparse, flush=True)
    rng = np.random.default_rng(n)
    d = rng.random((n, n, n)).astype(np.float32)  # z, y, x
    if sparse:
        d[: n // 2] = 0
    opts = dict(TINY["build"], want_mode=0, max_depth=12, variation_tau=0.05)
    if sparse:
        nb = n // 8
        v = d.reshape(nb, 8, nb, 8, nb, 8).transpose(0, 2, 4, 1, 3, 5).reshape(nb ** 3, 512)
        at = np.flatnonzero(v.any(axis=1))
        coords = np.stack([at % nb, at // nb % nb, at // nb ** 2], axis=1).astype(np.int32)
        g = tv.leb_build_sparse(torch.from_numpy(coords).cuda(), torch.from_numpy(np.ascontiguousarray(v[at])).cuda(),
                                n, TINY["camera"], build=opts)
    else:
        g = tv.leb_build(torch.from_numpy(d.reshape(-1)).cuda(), n, TINY["camera"], build=opts)
    o = oracle.leb_build(d.reshape(-1), n, TINY["camera"], opts)
    assert_grids_equal(g.export(), o.export(), f"n {n}")

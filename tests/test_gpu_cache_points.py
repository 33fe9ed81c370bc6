"""The radiance cache's query kernel at the edges of its 64-sample waves and
16-sample column blocks, and of its encoding (positions where the waves
vanish or peak)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cache():
    import torch
    assert torch.cuda.is_available(), "no GPU"
    import paper_2506_11510_amd as tv
    n = tv.Nrc(dict(sigma_ref=20.0, ema=0.0, seed=5))
    return n, n.export()


def points(count, seed):
    rng = np.random.default_rng(seed)
    d = rng.normal(size=(count, 3))
    d /= np.linalg.norm(d, axis=1)[:, None]
    return rng.random((count, 3)).astype(np.float32), d.astype(np.float32), (30 * rng.random(count)).astype(np.float32)


@pytest.mark.parametrize("count", [1, 15, 16, 17, 63, 64, 65, 4097])
def test_a_point_does_not_depend_on_its_place(cache, count):
    """Every sample is computed by itself: the first `count` of a larger
    query, and the same points in reverse, give the same bits."""
    n, _ = cache
    print("case", count, flush=True)
    pos, d, s = points(5000, 1)
    whole = n.infer(pos, d, s).cpu().numpy()
    part = n.infer(pos[:count], d[:count], s[:count]).cpu().numpy()
    back = n.infer(pos[:count][::-1].copy(), d[:count][::-1].copy(), s[:count][::-1].copy()).cpu().numpy()
    assert part.tobytes() == whole[:count].tobytes()
    assert back[::-1].tobytes() == part.tobytes()


def test_encoding_edges(cache):
    """Positions at 0, 1, powers of two and their neighbours, against the
    oracle's FP64 encoding and BF16-operand network: equal but where an
    operand sits on a bfloat16 boundary (2^-6 of the scale at most, 1e-4 on
    at least 95 % of outputs)."""
    n, P = cache
    v = np.float32([0, 1, 0.5, 0.25, 0.75, 1 / 3, 2.0 ** -12, 1 - 2.0 ** -12, 2.0 ** -24, 1 - 2.0 ** -24, 0.1])
    pos = np.stack(np.meshgrid(v, v, v), axis=-1).reshape(-1, 3).astype(np.float32)
    _, d, s = points(len(pos), 2)
    s[::7] = 0.0
    y = n.infer(pos, d, s).cpu().numpy().astype(np.float64)
    ref = oracle.mlp_forward(P.astype(np.float64), oracle.nrc_encode(pos, d, s, 20.0).astype(np.float64), bf16=True)
    e = np.abs(y - ref) / np.sqrt((ref ** 2).mean())
    assert e.max() <= 2.0 ** -6 and (e <= 1e-4).mean() >= 0.95

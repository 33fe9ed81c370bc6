"""The tracer's stages at the sizes where they can go wrong: the lists of
colliding samples (partial waves, blocks, chunks, fewer chunks than lists),
queued light rays of every transmittance and of training paths, and face
tests that leave the common path (near ties, directions with components that
vanish or nearly do)."""
import numpy as np
import pytest

import oracle
import synthetic
from parity import assert_image_parity

pytestmark = pytest.mark.gpu
QUEUED, OWN = (1 << 31) - 1, 1 << 20  # step guards: light rays queued / walked by their lanes
TINY = synthetic.scene("tiny")


def say(*a):
    print(*a, flush=True)


@pytest.fixture(scope="module")
def tv():
    import torch
    assert torch.cuda.is_available(), "no GPU"
    import paper_2506_11510_amd as tv
    tv.lib()
    return tv


@pytest.fixture(scope="module")
def tiny(tv):
    import torch
    d = TINY["density_fn"]()
    return tv.leb_build(torch.from_numpy(d).cuda(), 64, TINY["camera"], build=TINY["build"]), d


@pytest.mark.parametrize("w,h,spp", [(8, 8, 1), (8, 8, 3), (8, 8, 4), (9, 8, 4), (24, 40, 5), (257, 129, 3),
                                     (512, 264, 17), (1024, 512, 9)])
@pytest.mark.parametrize("transmittance", [0, 1])
def test_queued_image_equals_own_walks(tv, tiny, w, h, spp, transmittance):
    """The image with queued light rays against the one whose lanes walk
    their own: the same paths and steps, FP32 sums of at most 8 terms per
    sample in another order.  Sums of k positive terms in two orders differ
    by at most 2 k 2^-24 relative: k = 8 spp <= 136 gives 1.7e-5."""
    g, _ = tiny
    say(f"case {w}x{h} spp {spp} transmittance {transmittance}")
    cam = dict(TINY["camera"], width=w, height=h)
    got = {}
    for guard in (QUEUED, OWN):
        r = dict(max_bounces=8, transmittance=transmittance, max_steps_per_path=guard)
        img, st = tv.render(g, cam, TINY["medium"], TINY["light"], spp, 5, r)
        got[guard] = img.cpu().numpy().astype(np.float64), st
    (a, sa), (b, sb) = got[QUEUED], got[OWN]
    for k in ("tet_steps", "real_collisions", "null_collisions", "escapes", "truncated"):
        assert sa[k] == sb[k], k
    assert sa["light_rays_queued"] > 0 and sb["light_rays_queued"] == 0
    assert (np.abs(a - b) <= 1.7e-5 * np.abs(b)).all()


@pytest.mark.parametrize("channels", [False, True])
@pytest.mark.parametrize("paths,bounces", [(1, 1), (63, 8), (1000, 5)])
def test_training_records_queued_equal_own_walks(tv, channels, paths, bounces):
    """Training records do not depend on who walks the light rays: the terms
    of a path are summed in path order either way, so the records are the
    same bits."""
    import torch
    sc = synthetic.scene("blobs_adaptive")
    d = sc["density_fn"]()
    g = tv.leb_build(torch.from_numpy(d).cuda(), 32, sc["camera"], build=sc["build"])
    r = dict(max_bounces=bounces)
    if channels:
        g.set_channels(32, **synthetic.channels(4, 32))
        r.update(channels=1, emission=[0.3, 0.2, 0.1])
    n = tv.Nrc(dict(sigma_ref=5.0, train_paths=paths))
    say(f"case training records, {paths} paths, {bounces} bounces, channels {channels}")
    a, b = (n.collect(g, sc["camera"], sc["medium"], sc["light"], 9, dict(r, max_steps_per_path=guard))
            for guard in (QUEUED, OWN))
    assert len(a["tag"]) == len(b["tag"]) and (paths == 1 or len(a["tag"]) > 0)
    for k in a:
        assert a[k].tobytes() == b[k].tobytes(), k


@pytest.mark.parametrize("sun", [(0.0, 1.0, 0.0), (1e-20, 1.0, 0.0), (1e-38, 1e-30, -1.0), (0.0, 0.0, 0.0), (0.7071067, 0.7071068, 0.0),
                                 (0.57735026, 0.57735026, 0.57735026)])
@pytest.mark.parametrize("layout", [32, 48])
def test_degenerate_light_directions(tv, tiny, sun, layout):
    """Light rays along axes, diagonals and edges of the tets (ties between
    faces) and with components too small for reciprocals, from a camera at a
    lattice point, against the oracle at the image bar."""
    g, d = tiny
    say(f"case light along {sun}, {layout}-byte records")
    o = oracle.leb_build(d, 64, TINY["camera"], TINY["build"])
    cam = dict(TINY["camera"], pos=[0.5, 0.5, 0.5], look_at=[0.5, 0.5, 1.0], up=[0, 1, 0], fov_y_deg=90.0, width=24, height=24)
    light = dict(TINY["light"], sun_dir=list(sun))
    r = dict(TINY["render"], record_layout=layout)
    img, _ = tv.render(g, cam, TINY["medium"], light, 4, 3, r)
    ref, _ = o.render(cam, TINY["medium"], light, 4, 3, r, threads=8)
    assert_image_parity(img.cpu().numpy().reshape(-1, 3), ref, f"light {sun}")

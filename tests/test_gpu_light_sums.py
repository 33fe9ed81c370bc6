"""Light terms are summed with their samples, in path order, whoever walks the
light rays: wherever light rays are queued to be summed so (voxels, density
models, ratio and delta tracking, batches, renders without allocation), the
image has the bits of the one whose lanes walk their own, also where the queue
is full and the paths wait for a second launch, and two calls agree."""
import numpy as np
import pytest

import synthetic

pytestmark = pytest.mark.gpu
QUEUED, OWN = (1 << 31) - 1, 1 << 30  # step guards: light rays queued / walked by their lanes
SC = synthetic.scene("tiny")
NEAR = dict(SC["camera"], pos=[0.5, 0.5, 0.2])  # inside: nearly every sample collides
EMIT = dict(channels=1, emission=[0.3, 0.2, 0.1])


def say(*a):
    print(*a, flush=True)


@pytest.fixture(scope="module")
def tv():
    import torch
    assert torch.cuda.is_available(), "no GPU"
    import paper_2506_11510_amd as tv
    tv.lib()
    return tv


def grid_of(tv, channels=False, model=0, scale=1.0):
    import torch
    d = SC["density_fn"]()
    g = tv.leb_build(torch.from_numpy(d).cuda(), 64, SC["camera"], build=dict(SC["build"], density_scale=scale))
    if channels:
        g.set_channels(32, **synthetic.channels(4, 32))
    if model:
        g.set_density_model(model, torch.from_numpy(d).cuda(), 64, scale=scale)
    return g


def same_bits(a, b, what):
    assert a.tobytes() == b.tobytes(), f"{what}: {int((a.view(np.uint32) != b.view(np.uint32)).sum())} of {a.size} differ"


# scale 1: about one collision a path; 30 with albedo 1: tens, more than the queue holds
@pytest.mark.parametrize("w,h,spp,scale,bounces", [(8, 8, 1, 1.0, 8), (33, 17, 5, 1.0, 8), (64, 48, 9, 30.0, 64), (251, 187, 24, 30.0, 40)])
@pytest.mark.parametrize("kind,opts", [("voxels", {}), ("voxels", dict(transmittance=1)), ("tets", dict(transmittance=1)),
                                       ("tets", dict(transmittance=2, **EMIT)), ("linear", {}), ("linear", EMIT),
                                       ("lookup", dict(transmittance=1)), ("tets", dict(transmittance=1, record_layout=48))])
def test_image_bits(tv, kind, opts, w, h, spp, scale, bounces):
    say(f"case {kind} {opts} {w}x{h} spp {spp}, density x {scale}")
    import torch
    cam = dict(NEAR if scale > 1 else SC["camera"], width=w, height=h)
    med = dict(albedo=1.0 if scale > 1 else 0.9, g=0.3)
    got = []
    if kind == "voxels":
        vol = torch.from_numpy(SC["density_fn"]()).cuda()
        call = lambda r: tv.dda_render(vol, 64, scale, cam, med, SC["light"], spp, 5, render=r)
    else:
        g = grid_of(tv, "channels" in opts, {"linear": 1, "lookup": 2}.get(kind, 0), scale)
        call = lambda r: tv.render(g, cam, med, SC["light"], spp, 5, render=r)
    for guard in (QUEUED, QUEUED, OWN):
        img, st = call(dict(opts, max_bounces=bounces, max_steps_per_path=guard))
        got.append((img.cpu().numpy(), st))
    (a, sa), (b, sb), (c, sc) = got
    say(f"  {sa['real_collisions']} collisions, {sa['light_rays_queued']} queued")
    assert 0 < sa["light_rays_queued"] <= sa["real_collisions"] and sc["light_rays_queued"] == 0
    assert scale == 1.0 or "channels" in opts or sa["light_rays_queued"] < sa["real_collisions"]  # the queue was full
    for k in ("tet_steps", "real_collisions", "null_collisions", "escapes", "truncated"):
        assert sa[k] == sb[k] == sc[k], k
    same_bits(a, b, "two calls")
    same_bits(a, c, "queued and own walks")


def test_several_passes(tv):
    """More samples than a pass holds (2^25 entry records)."""
    import torch
    say("case voxels, two passes")
    cam = dict(SC["camera"], width=1024, height=1024)
    vol = torch.from_numpy(SC["density_fn"]()).cuda()
    a, b = (tv.dda_render(vol, 64, 1.0, cam, SC["medium"], SC["light"], 33, 5,
                          render=dict(max_bounces=8, max_steps_per_path=guard))[0].cpu().numpy() for guard in (QUEUED, OWN))
    same_bits(a, b, "queued and own walks")


@pytest.mark.parametrize("w,h,spp,scale", [(64, 48, 3, 1.0), (64, 48, 9, 30.0), (251, 187, 30, 30.0), (1280, 720, 1, 4.0),
                                           (2048, 1024, 1, 4.0)])  # (room for 1.4 light rays a sample, for no queue)
@pytest.mark.parametrize("opts", [{}, EMIT])
def test_noalloc_bits(tv, opts, w, h, spp, scale):
    """One pass each but 251 x 187 at 30 samples, whose passes end elsewhere
    with a queue than without: there two calls are compared."""
    import torch
    say(f"case noalloc {w}x{h} spp {spp}, density x {scale}, {opts}")
    cam = dict(NEAR, width=w, height=h)
    g = grid_of(tv, bool(opts), 0, scale)
    got = []
    for guard in (QUEUED, QUEUED, OWN):
        out = torch.full((h, w, 3), -1.0, device="cuda")
        tv.render_noalloc(g, cam, dict(albedo=1.0, g=0.3), SC["light"], spp, 5,
                          render=dict(opts, max_bounces=24, max_steps_per_path=guard), out=out)
        got.append(out.cpu().numpy())
    same_bits(got[0], got[1], "two calls")
    if spp < 30:
        same_bits(got[0], got[2], "queued and own walks")


@pytest.mark.parametrize("scale", [1.0, 30.0])
@pytest.mark.parametrize("opts", [{}, dict(transmittance=1), EMIT])
def test_batch_bits(tv, opts, scale):
    say(f"case batch, density x {scale}, {opts}")
    grids = [grid_of(tv, bool(opts.get("channels")), m, scale) for m in (0, 1)]
    cams = [dict(NEAR, width=w, height=h) for w, h in ((33, 17), (64, 48))]
    args = (grids, cams, [dict(albedo=1.0, g=0.3)] * 2, [SC["light"]] * 2, [5, 9])
    got = {}
    for guard in (QUEUED, OWN):
        b = tv.Batch(*args, dict(opts, max_bounces=40, max_steps_per_path=guard))
        for rep in range(3):
            st = b.render([7, 8])
            got[guard, rep] = [o.cpu().numpy().copy() for o in b.outs], st
    for (guard, rep), (imgs, st) in got.items():
        for i in range(2):
            same_bits(imgs[i], got[OWN, 0][0][i], f"scene {i}, guard {guard}, frame {rep}")
            one, _ = tv.render(grids[i], cams[i], args[2][i], SC["light"], args[4][i], 7 + i,
                               render=dict(opts, max_bounces=40, max_steps_per_path=OWN))
            same_bits(imgs[i], one.cpu().numpy(), f"scene {i} and its own render")
        assert st["tet_steps"] == got[OWN, 0][1]["tet_steps"]


@pytest.mark.parametrize("guard", [QUEUED, OWN])
def test_batch_counts_its_queued_light_rays(tv, guard):
    """Every light ray of two small scenes is queued, or none (a ray per collision)."""
    say(f"case batch statistics, guard {guard}")
    g = grid_of(tv)
    r = dict(max_bounces=4, max_steps_per_path=guard)
    cams = [dict(SC["camera"], width=w, height=h) for w, h in ((33, 17), (64, 48))]
    _, st = tv.render_batch([g, g], cams, [SC["medium"]] * 2, [SC["light"]] * 2, [3, 2], [7, 8], r)
    assert st["real_collisions"] > 0
    assert st["light_rays_queued"] == (st["real_collisions"] if guard == QUEUED else 0)


def test_cached_image_bits(tv):
    """With a radiance cache and one sample a pixel (one query at most, so its
    atomic addition has one order): image paths with tracked light rays."""
    say("case cache, ratio tracking")
    g = grid_of(tv, scale=30.0)
    n = tv.Nrc(dict(sigma_ref=50.0, truncate_bounce=12))
    cam = dict(NEAR, width=96, height=80)
    a, b = (tv.render(g, cam, dict(albedo=1.0, g=0.3), SC["light"], 1, 5,
                      render=dict(max_bounces=24, transmittance=1, nrc=n, max_steps_per_path=guard)) for guard in (QUEUED, OWN))
    assert 0 < a[1]["light_rays_queued"] < a[1]["real_collisions"] and a[1]["cache_queries"] == b[1]["cache_queries"] > 0
    same_bits(a[0].cpu().numpy(), b[0].cpu().numpy(), "queued and own walks")

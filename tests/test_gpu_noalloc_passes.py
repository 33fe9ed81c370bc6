"""tet_render_noalloc in several passes whose last is one sample shorter, with
nearly every sample colliding: the fullest lists that such a call can have."""
import pytest

import synthetic
from parity import assert_image_parity

pytestmark = pytest.mark.gpu


# passes of 244 + 243, 43 + 42 and 27 + 26 samples, and others
@pytest.mark.parametrize("w,h,spp", [(64, 64, 487), (192, 120, 85), (192, 192, 53), (64, 64, 543), (192, 120, 95), (192, 192, 59)])
def test_short_last_pass_of_a_dense_view(w, h, spp):
    import torch
    assert torch.cuda.is_available(), "no GPU"
    import paper_2506_11510_amd as tv
    print(f"case noalloc {w}x{h} spp {spp}, dense", flush=True)
    sc = synthetic.scene("tiny")
    cam = dict(sc["camera"], pos=[0.5, 0.5, 0.5], look_at=[0.6, 0.5, 1.0], width=w, height=h)
    d = torch.full((64 ** 3,), 40.0, device="cuda")
    g = tv.leb_build(d, 64, cam, build=sc["build"])
    r = dict(sc["render"], max_bounces=3)
    ref, st = tv.render(g, cam, dict(albedo=0.9, g=0.3), sc["light"], spp, 5, r)
    assert st["escapes"] < 0.1 * w * h * spp  # (two thirds colliding would do)
    out = torch.full((h, w, 3), -1.0, device="cuda")
    for _ in range(2):
        tv.render_noalloc(g, cam, dict(albedo=0.9, g=0.3), sc["light"], spp, 5, render=r, out=out)
        torch.cuda.synchronize()
        assert_image_parity(out.cpu().numpy(), ref.cpu().numpy(), f"noalloc {w}x{h}")


@pytest.mark.parametrize("w,h,spp", [(64, 48, 9), (251, 187, 30)])  # one pass, two
def test_captured_render_replays(w, h, spp):
    """A captured call, replayed with the program's own work between the
    replays, gives the eager call's bits every time (dense: the queue fills
    and paths wait for the second launch)."""
    import torch
    assert torch.cuda.is_available(), "no GPU"
    import paper_2506_11510_amd as tv
    print(f"case noalloc captured, {w}x{h} spp {spp}", flush=True)
    sc = synthetic.scene("tiny")
    cam = dict(sc["camera"], pos=[0.5, 0.5, 0.2], width=w, height=h)
    g = tv.leb_build(torch.from_numpy(sc["density_fn"]()).cuda(), 64, cam, build=dict(sc["build"], density_scale=30.0))
    out = torch.full((h, w, 3), -1.0, device="cuda")
    call = lambda: tv.render_noalloc(g, cam, dict(albedo=1.0, g=0.3), sc["light"], spp, 5, render=dict(max_bounces=24), out=out)
    call()
    torch.cuda.synchronize()
    want = out.clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for rep in range(4):
        out.fill_(-1.0)
        tv.render(g, cam, sc["medium"], sc["light"], 2, rep)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want), rep

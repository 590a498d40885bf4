"""Views whose tiles are all long (a dense cloud of small splats over an image of
thousands of tiles): they are blended by a wave per 8x8 quarter, with the
backward's segments started from the states those waves leave.  Image and
gradients against the kernels with two pixels per lane (the image bit for bit),
and the forward blend's time for each instance."""
import numpy as np
import pytest

import scenegen
from scenegen import configs

pytestmark = pytest.mark.gpu


def view(leaves, width, height):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2507_01110_amd.lodgs import Scene
    spec = configs.tiny_spec(n=leaves, seed=5, sh_degree=0)
    spec.half_extent = ext = 10.0 * (leaves / 16384.0) ** (1.0 / 3.0)
    S = Scene(scenegen.build_tree(spec))
    return S, scenegen.camera_look_at((0.0, 0.0, 2.2 * ext), (0.0, 0.0, 0.0), (0.0, 1.0, 0.0), width, height)


@pytest.mark.parametrize("leaves,width,height", [(600_000, 816, 800), (1_500_000, 1027, 1005)])
def test_long_tiles_by_quarters(monkeypatch, leaves, width, height):
    import torch
    from paper_2507_01110_amd.lodgs import Frame, grads_like
    S, cam = view(leaves, width, height)
    dL = torch.from_numpy(np.random.default_rng(leaves).standard_normal((height, width, 3)).astype(np.float32)).cuda()
    out = {}
    for px in (1, 2):
        monkeypatch.setenv("LODGS_BLEND_PX_FWD", str(px))
        monkeypatch.setenv("LODGS_BLEND_PX_BWD", str(px))
        f = Frame(S, S.n_nodes, 1 << 22, width, height)
        f.lod_select(cam, 0.0)
        for _ in range(2):  # the second pass starts from the first one's state
            img = f.render(cam)
            sel = grads_like(S, S.n_nodes, zero=False)
            f.backward(dL, sel=sel)
        assert f.stats()["status"] == 0
        tile, _ = f.instances()
        lengths = torch.bincount(tile.long())
        n = int(f.stats()["n_instances"])
        long = int(((lengths > 256) & (lengths < n // 2048)).sum())
        print("dense", leaves, width, height, px, "instances", n, "tiles by quarters with segments", long, flush=True)
        assert long >= 500
        rows = int(f.count.item())  # the others are not written
        out[px] = img.clone(), {k: t[:rows].double() for k, t in sel.items()}
        del f
    assert torch.equal(out[1][0], out[2][0])
    for k, t in out[1][1].items():
        d = float((t - out[2][1][k]).norm() / out[2][1][k].norm())
        assert d <= 1e-4, (k, d)


def test_time_of_the_forward_blend_of_a_dense_view():
    import torch
    from paper_2507_01110_amd.lodgs import Frame
    S, cam = view(2_000_000, 1920, 1080)
    f = Frame(S, S.n_nodes, 1 << 23, 1920, 1080)
    f.lod_select(cam, 0.0)
    f.render(cam)
    f.set_timing(True)
    best = float("inf")
    for _ in range(5):
        f.render(cam)
        torch.cuda.synchronize()
        best = min(best, 1e3 * f.timings()["blend"][0])
    n = f.stats()["n_instances"]
    print("us", best, "instances", n, flush=True)
    assert best <= 1e-4 * n, (best, n)  # 0.1 ns an instance: 0.06 by quarters, 0.14 by blocks

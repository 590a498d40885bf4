"""The blend kernels against the oracle at the sizes where they change form:
pixels with the path's 1e-4 bar, node gradients with its 1e-3 relative L2 per
parameter group."""
import numpy as np
import pytest

import oracle
import scenegen
from scenegen import configs

pytestmark = pytest.mark.gpu

GROUPS = {"means": slice(0, 3), "log_scales": slice(3, 6), "quats": slice(6, 10), "opacity_logits": slice(10, 11),
          "sh": slice(11, None)}


@pytest.fixture(scope="module")
def scene():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2507_01110_amd.lodgs import Scene
    tree = scenegen.build_tree(configs.tiny_spec(n=20000, seed=11, sh_degree=1))
    return tree, Scene(tree)


def check(tree, S, n, width, height, distance=300.0):
    """Render and backward of n nodes spread over the layout."""
    import torch
    from paper_2507_01110_amd.lodgs import Frame, grads_like
    cam = scenegen.camera_look_at((0.0, 0.0, distance), (0.0, 0.0, 0.0), (0.0, 1.0, 0.0), width, height)
    positions = np.arange(n) * (S.n_nodes // n)
    print("blend", n, width, height, distance, flush=True)
    f = Frame(S, n, 1 << 20, width, height)
    F = oracle.OracleFrame(tree, S.perm[positions].astype(np.int32), cam)
    dL = np.random.default_rng(n).standard_normal((height, width, 3)).astype(np.float32)
    _, g_o = F.backward(dL.astype(np.float64))
    idx = torch.from_numpy(np.ascontiguousarray(positions, np.int32)).cuda()
    cnt = torch.tensor([n], dtype=torch.int32, device="cuda")
    sel = grads_like(S, n, zero=False)
    for _ in range(2):  # the second pass starts from the first one's state
        img = f.render(cam, idx=idx, count=cnt)
        assert f.stats()["status"] == 0
        assert float(np.abs(img.cpu().numpy().astype(np.float64) - F.image).max()) <= 1e-4
        f.backward(torch.from_numpy(dL).cuda(), sel=sel)
        got = np.concatenate([sel[k].reshape(n, -1).cpu().numpy().astype(np.float64) for k in GROUPS], axis=1)
        for k, s in GROUPS.items():
            err = np.linalg.norm(got[:, s] - g_o[:, s])
            assert err <= 1e-3 * max(np.linalg.norm(g_o[:, s]), 1e-12), (k, err)


@pytest.mark.parametrize("px", [1, 2, 4])
@pytest.mark.parametrize("n", [60, 130, 300])
def test_pixels_per_lane(scene, monkeypatch, px, n):
    # rows that replay more than 64 of a batch's instances
    monkeypatch.setenv("LODGS_BLEND_PX_FWD", str(px))
    monkeypatch.setenv("LODGS_BLEND_PX_BWD", str(px))
    check(*scene, n, 16, 16)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 127, 128, 129, 255, 256, 257, 320, 1025])
@pytest.mark.parametrize("size", [(16, 16), (13, 11)])
def test_one_tile(scene, n, size):
    # partial batches, and the tiles' forms on both sides of 256 instances
    check(*scene, n, *size)


@pytest.mark.parametrize("n,distance", [(255, 60.0), (600, 60.0), (2500, 90.0), (6000, 300.0)])
def test_pixels_that_stop(scene, n, distance):
    # pixels that stop early, in tiles of both forms; images of partial tiles
    check(*scene, n, 40, 23, distance)


@pytest.mark.parametrize("n", [511, 512, 513, 769])
def test_segments(scene, n):
    # lists that end at, before and behind the backward's segments of 256
    check(*scene, n, 16, 16)


@pytest.mark.parametrize("width,height", [(96, 80), (128, 72), (512, 496), (608, 560), (640, 640)])
def test_splats_over_many_tiles(scene, width, height):
    # one splat's instances around a thread's (32), a wave's (1024) and a
    # workgroup's share, its neighbours with few
    check(*scene, 40, width, height, 8.0)


@pytest.mark.parametrize("degree", [0, 1, 2, 3])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 700])
def test_rows_of_splats_that_were_not_drawn(degree, n):
    # selection-indexed gradients: rows hold whatever they held before, some of
    # the splats lie behind the camera
    import torch
    from paper_2507_01110_amd.lodgs import Frame, Scene, grads_like
    tree = scenegen.build_tree(configs.tiny_spec(n=2000, seed=3, sh_degree=degree))
    S = Scene(tree)
    cam = scenegen.camera_look_at((0.5, 0.2, 0.3), (4.0, 1.0, 2.0), (0.0, 0.0, 1.0), 64, 48)
    positions = np.arange(n) * (S.n_nodes // n)
    F = oracle.OracleFrame(tree, S.perm[positions].astype(np.int32), cam)
    dL = np.random.default_rng(n).standard_normal((48, 64, 3)).astype(np.float32)
    _, g_o = F.backward(dL.astype(np.float64))
    f = Frame(S, n, 1 << 20, 64, 48)
    print("rows", degree, n, F.info()["n_visible"], flush=True)
    f.render(cam, idx=torch.from_numpy(np.ascontiguousarray(positions, np.int32)).cuda(),
             count=torch.tensor([n], dtype=torch.int32, device="cuda"))
    sel = grads_like(S, n, zero=False)
    for t in sel.values():
        t.fill_(float("nan"))
    f.backward(torch.from_numpy(dL).cuda(), sel=sel)
    got = np.concatenate([sel[k].reshape(n, -1).cpu().numpy().astype(np.float64) for k in GROUPS], axis=1)
    none = ~np.any(g_o, axis=1)
    assert not np.any(got[none])
    for k, s in GROUPS.items():
        assert np.linalg.norm(got[:, s] - g_o[:, s]) <= 1e-3 * max(np.linalg.norm(g_o[:, s]), 1e-12), k

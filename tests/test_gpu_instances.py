"""The instance list (drawn-splat scan, instance emission, bucketing by tile,
per-tile depth sort) against the oracle's order, at the sizes where its
kernels change form: tiles of a sort run, a workgroup's sort and several
chunks; selections around the scan's tiles and thresholds; images of one tile,
of several chunks of the tile order and of more tiles than the LDS counters
hold; depth ties (broken by selection position).  The order is compared
exactly; pixels with the path's 1e-4 bar."""
import numpy as np
import pytest

import oracle
import scenegen
from scenegen import configs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def scene():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2507_01110_amd.lodgs import Scene
    tree = scenegen.build_tree(configs.tiny_spec(n=20000, seed=11, sh_degree=1))
    return tree, Scene(tree)


def check(tree, S, cam, positions, max_instances=1 << 22):
    """Renders the nodes at the given layout positions (repeats allowed)."""
    import torch
    from paper_2507_01110_amd.lodgs import Frame
    n = len(positions)
    print("instances", n, cam.width, cam.height, flush=True)
    f = Frame(S, max(n, 1), max_instances, cam.width, cam.height)
    idx = torch.from_numpy(np.ascontiguousarray(positions, np.int32)).cuda()
    cnt = torch.tensor([n], dtype=torch.int32, device="cuda")
    F = oracle.OracleFrame(tree, S.perm[positions].astype(np.int32), cam)
    ot, op = F.instances()
    for _ in range(2):  # the second render starts from the first one's state
        img = f.render(cam, idx=idx, count=cnt)
        st = f.stats()
        assert st["status"] == 0 and st["n_instances"] == len(ot)
        t, p = f.instances()
        assert np.array_equal(t.cpu().numpy(), ot)
        assert np.array_equal(p.cpu().numpy(), op)
        assert float(np.abs(img.cpu().numpy().astype(np.float64) - F.image).max()) <= 1e-4


@pytest.mark.parametrize("n", [1, 63, 64, 65, 255, 256, 257, 512, 513, 1024, 1025, 2047, 2048, 2049, 4096, 4097, 9000,
                               39999])
def test_one_tile(scene, n):
    tree, S = scene
    cam = scenegen.camera_look_at((0.0, 0.0, 300.0), (0.0, 0.0, 0.0), (0.0, 1.0, 0.0), 16, 16)
    check(tree, S, cam, np.arange(n) * (S.n_nodes // n))


@pytest.mark.parametrize("n", [2048, 2049, 65536, 65537, 524288, 524289, 600000])
def test_selection_sizes_with_repeated_nodes(scene, n):
    # repeats of a node tie in depth: their order is the selection's
    tree, S = scene
    cam = configs.tiny_camera(96, 80)
    check(tree, S, cam, np.arange(n) % 4099 + 30000, max_instances=1 << 23)


@pytest.mark.parametrize("size", [(1, 1), (512, 512), (768, 720), (1920, 1088), (4112, 2064)])
def test_image_sizes(scene, size):
    tree, S = scene
    check(tree, S, configs.tiny_camera(*size), np.arange(20000, 39999, 3), max_instances=1 << 24)


def test_ties_in_depth():
    # every splat at one depth: the whole list is in selection order per tile
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2507_01110_amd.lodgs import Scene
    tree = scenegen.build_tree(configs.tiny_spec(n=6000, seed=12, sh_degree=0))
    tree.means[:, 2] = 0.0
    S = Scene(tree)
    check(tree, S, configs.tiny_camera(64, 48), np.arange(S.n_nodes))


def test_overflow_keeps_within_the_frame(scene):
    # more instances than the frame holds: reported, then a fitting view is right
    import torch
    from paper_2507_01110_amd._lib import E_CAPACITY
    from paper_2507_01110_amd.lodgs import Frame
    tree, S = scene
    f = Frame(S, S.n_nodes, 5000, 4112, 2064)
    idx = torch.arange(S.n_nodes, dtype=torch.int32, device="cuda")
    cnt = torch.tensor([S.n_nodes], dtype=torch.int32, device="cuda")
    f.render(configs.tiny_camera(4112, 2064), idx=idx, count=cnt)
    st = f.stats()
    assert st["status"] == E_CAPACITY and st["n_instances"] > 5000
    f.clear_status()
    cam = configs.tiny_camera(64, 48)
    cnt.fill_(500)
    img = f.render(cam, idx=idx, count=cnt)
    assert f.stats()["status"] == 0
    F = oracle.OracleFrame(tree, S.perm[:500].astype(np.int32), cam)
    assert float(np.abs(img.cpu().numpy().astype(np.float64) - F.image).max()) <= 1e-4

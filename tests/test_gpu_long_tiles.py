"""Tiles of many sort chunks (2048 instances each): both sides of the 24 chunks
up to which the sorted chunks are put together by counting, tiles of more
chunks than a split keeps windows for (2048), equal depths over whole tiles,
several such tiles at once; and the time of the instance sort, which grows with
the tile's list and not with its square."""
import numpy as np
import pytest

import oracle
import scenegen
from scenegen import configs

pytestmark = pytest.mark.gpu

CHUNK = 2048


@pytest.fixture(scope="module")
def scene():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2507_01110_amd.lodgs import Scene
    tree = scenegen.build_tree(configs.tiny_spec(n=20000, seed=11, sh_degree=0))
    S = Scene(tree)
    # a camera that sees every node in its one tile, and the nodes' depths (FP32 bits)
    cam = scenegen.camera_look_at((0.0, 0.0, 300.0), (0.0, 0.0, 0.0), (0.0, 1.0, 0.0), 16, 16)
    F = oracle.OracleFrame(tree, S.perm.astype(np.int32), cam)
    assert F.info()["n_inst"] == S.n_nodes
    return tree, S, cam, F.splats()["depth_bits"]


def render(S, cam, positions, max_instances):
    import torch
    from paper_2507_01110_amd.lodgs import Frame
    n = len(positions)
    f = Frame(S, n, max_instances, cam.width, cam.height)
    idx = torch.from_numpy(np.ascontiguousarray(positions, np.int32)).cuda()
    cnt = torch.tensor([n], dtype=torch.int32, device="cuda")
    f.render(cam, idx=idx, count=cnt)
    st = f.stats()
    assert st["status"] == 0
    return f, idx, cnt


@pytest.mark.parametrize("n", [24 * CHUNK - 1, 24 * CHUNK, 24 * CHUNK + 1, 25 * CHUNK, 25 * CHUNK + 1, 100 * CHUNK - 7,
                               257 * CHUNK + 1, 2048 * CHUNK, 2048 * CHUNK + 5, 2300 * CHUNK + 1])
def test_order_in_a_long_tile(scene, n):
    # selections in a scattered order with repeats, which tie in depth: by depth,
    # then by place in the selection
    import torch
    tree, S, cam, depth = scene
    print("long tile", n, flush=True)
    positions = (np.arange(n, dtype=np.int64) * 7919 + 13) % S.n_nodes
    f, _, _ = render(S, cam, positions, n)
    t, p = f.instances()
    assert f.stats()["n_instances"] == n and not bool(t[:n].any())
    want = np.argsort(depth[positions], kind="stable")
    assert np.array_equal(p[:n].cpu().numpy(), want)


@pytest.mark.parametrize("nodes", [1, 2, 30])
def test_few_depths_in_a_long_tile(scene, nodes):
    tree, S, cam, depth = scene
    n = 40 * CHUNK + 77
    print("few depths", nodes, flush=True)
    positions = np.arange(n, dtype=np.int64) % nodes * 1000
    f, _, _ = render(S, cam, positions, n)
    _, p = f.instances()
    assert np.array_equal(p[:n].cpu().numpy(), np.argsort(depth[positions], kind="stable"))


def test_several_long_tiles(scene):
    tree, S, _, _ = scene
    positions = np.tile(np.arange(S.n_nodes), 8)
    cam = scenegen.camera_look_at((0.0, 0.0, 60.0), (0.0, 0.0, 0.0), (0.0, 1.0, 0.0), 40, 24)
    F = oracle.OracleFrame(tree, S.perm[positions].astype(np.int32), cam)
    ot, op = F.instances()
    assert np.bincount(ot).max() > 24 * CHUNK
    f, _, _ = render(S, cam, positions, 1 << 22)
    t, p = f.instances()
    assert np.array_equal(t.cpu().numpy(), ot) and np.array_equal(p.cpu().numpy(), op)


def test_time_of_the_sort_grows_with_the_list(scene):
    import torch
    tree, S, cam, depth = scene
    us = []
    for n in (64 * CHUNK, 512 * CHUNK):
        positions = (np.arange(n, dtype=np.int64) * 7919 + 13) % S.n_nodes
        f, idx, cnt = render(S, cam, positions, n)
        f.set_timing(True)
        best = float("inf")
        for _ in range(5):
            f.render(cam, idx=idx, count=cnt)
            torch.cuda.synchronize()
            t = f.timings()
            best = min(best, 1e3 * t["depth_sort"][0])
        us.append(best)
        f.set_timing(False)
    print("us", us, flush=True)
    # 8 times the list, on a chip that the shorter one leaves half idle at least
    assert us[1] <= 4.0 * us[0], us


def test_time_of_the_tile_scan_hardly_grows_with_one_list(scene):
    # the segments and sort chunks of a long tile are listed by many threads
    import torch
    tree, S, cam, depth = scene
    us = []
    for n in (CHUNK, 512 * CHUNK):
        positions = (np.arange(n, dtype=np.int64) * 7919 + 13) % S.n_nodes
        f, idx, cnt = render(S, cam, positions, n)
        f.set_timing(True)
        best = float("inf")
        for _ in range(5):
            f.render(cam, idx=idx, count=cnt)
            torch.cuda.synchronize()
            best = min(best, 1e3 * f.timings()["ranges"][0])
        us.append(best)
        f.set_timing(False)
    print("us", us, flush=True)
    assert us[1] <= 4.0 * us[0], us

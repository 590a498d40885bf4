"""Counts of the blend: the evaluations and contributions of Frame.blend_work
and the contributing pixels that the backward adds to an attached pruning
statistic, exact, at the sizes where the kernels change form."""
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
    tree = scenegen.build_tree(configs.tiny_spec(n=20000, seed=11, sh_degree=0))
    return tree, Scene(tree)


def rendered(tree, S, n, width, height, distance, positions=None):
    import torch
    from paper_2507_01110_amd.lodgs import Frame
    cam = scenegen.camera_look_at((0.0, 0.0, distance), (0.0, 0.0, 0.0), (0.0, 1.0, 0.0), width, height)
    positions = np.arange(n) * (S.n_nodes // n) if positions is None else positions
    f = Frame(S, n, 1 << 20, width, height)
    f.render(cam, idx=torch.from_numpy(np.ascontiguousarray(positions, np.int32)).cuda(),
             count=torch.tensor([n], dtype=torch.int32, device="cuda"))
    assert f.stats()["status"] == 0
    return f, oracle.OracleFrame(tree, S.perm[positions].astype(np.int32), cam), positions


def evaluations(F, width, height):
    """Splats of its tile that each pixel evaluates: up to the one that stops it."""
    tile, pos = F.instances()
    m = F.splats()["f32"].astype(np.float64)
    mean = np.stack([m[:, 0] + m[:, 1], m[:, 2] + m[:, 3]], axis=1)
    tx = (width + 15) // 16
    total = 0
    for t in range(tx * ((height + 15) // 16)):
        g = pos[tile == t]
        if not len(g):
            continue
        x, y = np.meshgrid(np.arange(16 * (t % tx), min(16 * (t % tx) + 16, width)) + 0.5,
                           np.arange(16 * (t // tx), min(16 * (t // tx) + 16, height)) + 0.5)
        dx, dy = x.reshape(-1, 1) - mean[g, 0], y.reshape(-1, 1) - mean[g, 1]
        ce, se, h1, h2, o = m[g, 4], m[g, 5], m[g, 6], m[g, 7], m[g, 8]
        alpha = np.minimum(0.99, o * np.exp(h1 * (ce * dx + se * dy) ** 2 + h2 * (ce * dy - se * dx) ** 2))
        T = np.cumprod(np.where(alpha >= 1.0 / 255.0, 1.0 - alpha, 1.0), axis=1)
        stop = (T < 1e-4).argmax(axis=1)
        total += int(np.where((T < 1e-4).any(axis=1), stop + 1, len(g)).sum())
    return total


@pytest.mark.parametrize("px", [1, 2, 4])
@pytest.mark.parametrize("n,width,height,distance", [(60, 16, 16, 300.0), (65, 16, 16, 300.0), (130, 16, 16, 300.0),
                                                     (257, 13, 11, 300.0), (1025, 16, 16, 300.0), (600, 40, 23, 60.0),
                                                     (3000, 40, 23, 40.0)])
def test_work_of_the_forward_blend(scene, monkeypatch, px, n, width, height, distance):
    monkeypatch.setenv("LODGS_BLEND_PX_FWD", str(px))
    f, F, _ = rendered(*scene, n, width, height, distance)
    e, c = f.blend_work()
    print("work", px, n, width, height, e, c, flush=True)
    assert c == F.info()["n_contrib"]
    assert e == evaluations(F, width, height)


@pytest.mark.parametrize("px", [1, 2, 4])
@pytest.mark.parametrize("n,width,height,distance", [(1, 16, 16, 300.0), (64, 16, 16, 300.0), (65, 16, 16, 300.0),
                                                     (257, 16, 16, 300.0), (513, 13, 11, 300.0), (2500, 40, 23, 90.0),
                                                     (40, 96, 80, 8.0), (40, 512, 496, 8.0), (40, 608, 560, 8.0)])
def test_contributing_pixels_of_the_backward(scene, monkeypatch, px, n, width, height, distance):
    # lists of several segments; splats whose partials a thread, a wave and a
    # workgroup add up
    import torch
    monkeypatch.setenv("LODGS_BLEND_PX_FWD", str(px))
    monkeypatch.setenv("LODGS_BLEND_PX_BWD", str(px))
    tree, S = scene
    f, F, positions = rendered(tree, S, n, width, height, distance)
    last = torch.zeros(S.n_nodes, dtype=torch.int32, device="cuda")
    count = torch.zeros(S.n_nodes, dtype=torch.int32, device="cuda")
    iteration = torch.tensor([7], dtype=torch.int32, device="cuda")
    f.set_contrib_stats(last, count, iteration)
    dL = np.random.default_rng(n).standard_normal((height, width, 3)).astype(np.float32)
    print("contributing", px, n, width, height, flush=True)
    for k in (1, 2):  # the second pass adds the same again
        f.backward(torch.from_numpy(dL).cuda())
        want = np.zeros(S.n_nodes, np.int64)
        want[positions] = k * F.splat_contrib()
        assert np.array_equal(count.cpu().numpy(), want)
        assert np.array_equal(last.cpu().numpy(), np.where(want > 0, 7, 0))
    f.set_contrib_stats()

"""Values that are not finite in the image's derivative: they reach the splats
that contribute to a pixel of the block they lie in, and no others."""
import numpy as np
import pytest

import oracle
import scenegen
from scenegen import configs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("px", [1, 2, 4])
@pytest.mark.parametrize("layers,width,height", [(2, 4, 4), (3, 16, 16), (70, 16, 16), (300, 16, 16)])
def test_derivative_that_is_not_finite(monkeypatch, value, px, layers, width, height):
    # opaque splats behind each other, each over the whole image: the first
    # leaves 0.01 of the light, the second would leave less than 1e-4 and stops
    # every pixel, so that it and the ones behind it contribute nowhere
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2507_01110_amd.lodgs import Frame, Scene, grads_like
    monkeypatch.setenv("LODGS_BLEND_PX_FWD", str(px))
    monkeypatch.setenv("LODGS_BLEND_PX_BWD", str(px))
    tree = scenegen.build_tree(configs.tiny_spec(n=layers, seed=3, sh_degree=1))
    tree.means[:] = 0.0
    tree.means[:, 2] = -np.arange(tree.n_nodes)
    tree.log_scales[:] = 8.0
    tree.opacity_logits[:] = 12.0
    S = Scene(tree)
    cam = scenegen.camera_look_at((0.0, 0.0, 20.0), (0.0, 0.0, 0.0), (0.0, 1.0, 0.0), width, height)
    ids = np.arange(layers, dtype=np.int32)
    pos = np.empty(S.n_nodes, np.int32)
    pos[S.perm] = np.arange(S.n_nodes, dtype=np.int32)
    F = oracle.OracleFrame(tree, ids, cam)
    contrib = F.splat_contrib()
    assert contrib[0] == width * height and not contrib[1:].any()
    f = Frame(S, layers, 1 << 16, width, height)
    print("derivative", value, px, layers, width, height, flush=True)
    f.render(cam, idx=torch.from_numpy(pos[ids]).cuda(), count=torch.tensor([layers], dtype=torch.int32, device="cuda"))
    dL = np.random.default_rng(layers).standard_normal((height, width, 3)).astype(np.float32)
    dL[1, 2, 0] = value
    sel = grads_like(S, layers, zero=False)
    f.backward(torch.from_numpy(dL).cuda(), sel=sel)
    assert f.stats()["status"] == 0
    assert not bool(torch.isfinite(sel["sh"][0]).all())
    for k, t in sel.items():
        assert not bool((t[1:] != 0).any()), (k, t[1])  # (a NaN is not 0)

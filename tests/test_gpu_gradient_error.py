"""The geometry gradients' distance from 64 bits on splats that cover whole
4x4 blocks with weights of one sign, where the order of the sums over a
block's 16 pixels shows: no larger than with FP32 sums by a tree of adds (four
levels), which measured the bounds below on these 24 scenes."""
import numpy as np
import pytest

import oracle
import scenegen
from scenegen import configs

pytestmark = pytest.mark.gpu

# group: (columns of the oracle's gradients, root mean square of the relative L2 errors with a tree of adds)
TREE = {"means": (slice(0, 3), 6.37116e-07), "log_scales": (slice(3, 6), 1.15336e-07),
        "quats": (slice(6, 10), 6.69397e-07)}


def test_geometry_gradients_of_splats_over_whole_blocks():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2507_01110_amd.lodgs import Frame, Scene, grads_like
    total = dict.fromkeys(TREE, 0.0)
    for seed in range(24):
        tree = scenegen.build_tree(configs.tiny_spec(n=64, seed=seed, sh_degree=0))
        tree.log_scales[:] += 2.0
        tree.opacity_logits[:] -= 2.5
        S = Scene(tree)
        n = S.n_nodes
        cam = scenegen.camera_look_at((0.0, 0.0, 30.0), (0.0, 0.0, 0.0), (0.0, 1.0, 0.0), 64, 48)
        F = oracle.OracleFrame(tree, S.perm.astype(np.int32), cam)
        dL = np.abs(np.random.default_rng(seed).standard_normal((48, 64, 3)).astype(np.float32))
        _, want = F.backward(dL.astype(np.float64))
        f = Frame(S, n, 1 << 16, 64, 48)
        f.render(cam, idx=torch.arange(n, dtype=torch.int32, device="cuda"),
                 count=torch.tensor([n], dtype=torch.int32, device="cuda"))
        sel = grads_like(S, n, zero=False)
        f.backward(torch.from_numpy(dL).cuda(), sel=sel)
        for k, (cols, _) in TREE.items():
            got = sel[k].reshape(n, -1).cpu().numpy().astype(np.float64)
            total[k] += ((got - want[:, cols]) ** 2).sum() / (want[:, cols] ** 2).sum()
    for k, (_, bound) in TREE.items():
        err = (total[k] / 24) ** 0.5
        print(k, err, bound, flush=True)
        assert err <= bound, (k, err, bound)

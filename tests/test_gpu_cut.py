"""The HSPT cut (candidate chunks listed by visible tile, counted and written a
wave per chunk) against the oracle's, where its kernels change form: one SPT
holding the whole hierarchy (many chunks of one SPT), every node in the upper
hierarchy (SPTs of one node, several tiles of both kinds), and mixtures; with
and without culling, plain and CONSERVATIVE, through the frame and through the
allocation-free call.  Selected sets are compared exactly."""
import numpy as np
import pytest

import oracle
import scenegen
from scenegen import configs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("leaves,quantile", [(1, 0.5), (2, 1.0), (300, 0.0), (300, 1.0), (9000, 0.0), (9000, 0.5),
                                             (9000, 0.97), (30000, 1.0)])
def test_cut_over_volume_thresholds(leaves, quantile):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2507_01110_amd.lodgs import Frame, Scene
    print("cut", leaves, quantile, flush=True)
    tree = scenegen.build_tree(configs.tiny_spec(n=leaves, seed=21, sh_degree=0))
    lv = np.sort(tree.log_scales.astype(np.float64).sum(axis=1))
    # SPT roots are leaves or nodes below the threshold: the lowest volume puts
    # every interior node in the upper hierarchy, above the highest none
    tree.log_volume_threshold = float(lv[0] - 1.0 if quantile == 0.0 else lv[-1] + 1.0 if quantile == 1.0
                                      else lv[int(quantile * len(lv))])
    O = oracle.OracleScene(tree)
    S = Scene(tree)
    f = Frame(S, S.n_nodes, 1 << 20, 64, 64)
    idx = torch.empty(S.n_nodes, dtype=torch.int32, device="cuda")
    cnt = torch.empty(1, dtype=torch.int32, device="cuda")
    cams = [configs.tiny_camera(64, 64), scenegen.camera_look_at((3, 2, 1), (9, -4, 2), (0, 0, 1), 64, 48)]
    for cam in cams:
        for tau in (0.0, 0.5, 3.0, 1e4):
            for cull, conservative in ((True, False), (False, False), (True, True)):
                ids, _ = O.select(cam, tau, cull=cull, conservative=conservative)
                want = O.pos_of[ids]
                f.lod_select(cam, tau, cull=cull, conservative=conservative)
                S.lod_select_noalloc(cam, tau, idx, cnt, cull=cull, conservative=conservative)
                n = int(f.count.item())
                assert n == len(want) and int(cnt.item()) == n
                assert np.array_equal(f.idx[:n].cpu().numpy(), want)
                assert torch.equal(idx[:n], f.idx[:n])
                st = f.stats()
                assert st["status"] == 0 and st["n_selected"] == n
                assert st["n_upper_selected"] == int((want < S.n_upper).sum())

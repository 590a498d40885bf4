"""Device memory of a frame with many tiles and few instances: what is kept per
tile is its range, counters and place in the order, 32 bytes; nothing else
grows with the image."""
import pytest

import scenegen
from scenegen import configs

pytestmark = pytest.mark.gpu


def test_frame_of_a_large_image_and_few_instances():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2507_01110_amd.lodgs import Frame, Scene
    S = Scene(scenegen.build_tree(configs.tiny_spec(n=2000, seed=3, sh_degree=0)))
    first = Frame(S, 4096, 1 << 14, 16, 16)  # whatever a first frame loads
    torch.cuda.synchronize()
    free0, _ = torch.cuda.mem_get_info()
    f = Frame(S, 4096, 1 << 14, 16384, 16384)
    free1, _ = torch.cuda.mem_get_info()
    used = free0 - free1
    print("bytes", used, flush=True)
    # 2^20 tiles of 32 bytes, at most 256 bytes for each instance and selected
    # node, and 32 MiB for the allocator's granularity (some fifty arrays)
    assert used <= 32 * (1 << 20) + 256 * ((1 << 14) + 4096) + (32 << 20), used
    del f, first

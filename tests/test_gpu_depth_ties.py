"""Equal depths in the core (needs an MI355X): entries of one depth follow the
list, in front of the camera and, where a negative z_near lets splats through,
behind it."""
import numpy as np
import pytest
import torch

from paper_2410_08129_amd import htgs, scenes

pytestmark = pytest.mark.gpu

W, H, COPIES = 40, 24, 5


@pytest.mark.parametrize("z", [3.0, -3.0])
@pytest.mark.parametrize("K", [1, 2, 3, 4, 5, 8, 16])
def test_equal_depths_follow_the_list(z, K):
    # two groups of equal splats at different depths, dealt alternately
    n = 2 * COPIES
    depth = np.where(np.arange(n) % 2 == 0, z, z + 0.5)
    means = np.stack([np.zeros(n), np.zeros(n), depth], 1)
    ls = np.full((n, 3), np.log(0.4))
    q = np.tile([1.0, 0.0, 0.0, 0.0], (n, 1))
    sc = scenes._pack(means, ls, q, np.full(n, -1.0), np.zeros((n, 1, 3)), 0)
    w2c = np.concatenate([np.eye(3), np.zeros((3, 1))], 1).astype(np.float32)
    cam = scenes.Camera(w2c, 60.0, 60.0, W / 2, H / 2, W, H, z_near=-100.0)
    st = scenes.RenderSettings(K=K, tau_core=0.01, tile_w=8, tile_h=8)
    params = [torch.tensor(a, device="cuda") for a in sc.arrays()]
    print(f"z={z} K={K}", flush=True)
    frame = htgs.forward(params, 0, [cam], st)
    planes = htgs.state_planes(frame)
    ids, pos = planes["core_ids"].cpu().numpy(), planes["core_pos"].cpu().numpy()
    order = (list(range(0, n, 2)) + list(range(1, n, 2)))[:K]
    order += [-1] * (K - len(order))
    mid = (slice(None), slice(H // 2 - 1, H // 2 + 1), slice(W // 2 - 1, W // 2 + 1))
    for got in (ids[mid], pos[mid]):
        assert (got == np.array(order)[:, None, None]).all(), got[:, 0, 0]

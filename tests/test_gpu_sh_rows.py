"""Degree-3 SH gradients of sorted blending, stored a wave's rows at a time
(needs an MI355X): adding to given tensors gives their values plus the new
gradients bit for bit, rows of Gaussians that the view does not see stay as they
are, and nothing is written past the last Gaussian, at counts around a wave and
a workgroup."""
import numpy as np
import pytest
import torch

from paper_2410_08129_amd import htgs, scenes

pytestmark = pytest.mark.gpu

CAM = scenes.look_at((0, 0, -4), (0, 0, 0), (0, -1, 0), 45.0, 70, 50)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 257, 1000])
def test_rows_added_and_written(n):
    rng = np.random.default_rng(n)
    means = rng.uniform(-1.5, 1.5, (n, 3))
    means[1::3] += (0.0, 0.0, -20.0)          # behind the camera
    sc = scenes._pack(means, rng.normal(-2.0, 0.5, (n, 3)), scenes._quats(rng, n),
                      rng.normal(0.0, 1.0, n), rng.normal(0.0, 0.3, (n, 16, 3)), 3)
    st = scenes.RenderSettings(tile_w=8, tile_h=8, sorted_blend=True)
    params = [torch.tensor(a, device="cuda") for a in sc.arrays()]
    frame = htgs.forward(params, 3, [CAM], st)
    G = [torch.tensor(rng.normal(0, 1, (3, CAM.height, CAM.width)), dtype=torch.float32,
                      device="cuda")]
    print(f"n={n}", flush=True)
    new = htgs.backward(params, frame, G)
    base = [torch.randn_like(p) for p in params]
    room = torch.full((n * 48 + 48,), 7.0, device="cuda")     # one row of guard
    room[:n * 48] = base[4].reshape(-1)
    given = [b.clone() for b in base[:4]] + [room[:n * 48].view(n, 16, 3)]
    htgs.backward(params, frame, G, grads=given)
    for b, x, y in zip(base, new, given):
        assert torch.equal(b + x, y)
    assert torch.all(room[n * 48:] == 7.0)
    assert torch.all(new[4][1::3] == 0) and torch.any(new[4] != 0)

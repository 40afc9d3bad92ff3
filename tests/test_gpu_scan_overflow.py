"""Partials that are finite while their sum is not (needs an MI355X). One
Gaussian's loss gradients add up past the largest float32 over its tiles; it
alone gets gradients that are not finite, and its neighbours, whose partials
share its 64-slot chunks, get bit for bit what they get without its loss."""
import numpy as np
import pytest
import torch

from paper_2410_08129_amd import htgs, scenes

pytestmark = pytest.mark.gpu

N, BIG = 40, 20


@pytest.mark.parametrize("sorted_blend,views", [(False, 1), (False, 2), (True, 1)])
def test_overflow_stays_with_its_gaussian(sorted_blend, views):
    W, H = 128, 48
    cam = scenes.look_at((0, 0, -4), (0, 0, 0), (0, -1, 0), 45.0, W, H)
    rng = np.random.default_rng(2)
    # small splats in the right half, one that covers most of the left half
    px, py = rng.uniform(76, 124, N), rng.uniform(4, 44, N)
    px[BIG], py[BIG] = 28.0, 24.0
    depth = rng.uniform(3.8, 4.2, N)
    # (sorted blending emits in depth order: the big one in its middle)
    depth[BIG] = np.median(depth)
    means = np.stack([(px - cam.cx) / cam.fx * depth, (py - cam.cy) / cam.fy * depth,
                      depth - 4.0], 1)
    ls = np.log(np.full((N, 3), 0.8) * (depth / cam.fx)[:, None])
    ls[BIG] = np.log(8.0 * depth[BIG] / cam.fx)
    # grey 1/2 over a black background, and a loss gradient (c, -c, 0): the
    # geometry's terms cancel, the colours' are c alpha
    sh = np.zeros((N, 1, 3))
    sc = scenes._pack(means, ls, scenes._quats(rng, N), np.full(N, 2.0), sh, 0)
    st = scenes.RenderSettings(K=4, tile_w=8, tile_h=8, sorted_blend=sorted_blend)
    params = [torch.tensor(a, device="cuda") for a in sc.arrays()]
    frame = htgs.forward(params, 0, [cam] * views, st)
    G = rng.normal(0.0, 1.0, (3, H, W)).astype(np.float32)
    G[:, :, :64] = 0.0
    clean = htgs.backward(params, frame, [torch.tensor(G, device="cuda")] * views)
    # at most 64 pixels of alpha < 1 per tile: every partial is below 1.3e38
    G[0, :, :64], G[1, :, :64] = 2.0e36, -2.0e36
    print(f"sorted={sorted_blend} views={views}", flush=True)
    dirty = htgs.backward(params, frame, [torch.tensor(G, device="cuda")] * views)
    keep = torch.arange(N, device="cuda") != BIG
    assert not torch.isfinite(dirty[4][BIG]).all()
    for name, a, b in zip(("means", "log_scales", "quats", "logits", "sh"), clean, dirty):
        assert torch.isfinite(a).all(), name
        assert torch.equal(a[keep], b[keep]), name

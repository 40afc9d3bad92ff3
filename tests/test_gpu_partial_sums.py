"""Sums of the backward's instance partials with infinite and NaN values (needs
an MI355X). One pixel's loss gradient is not finite: the Gaussians with a
fragment there get gradients that are not finite, and every other Gaussian,
also those whose partials share a 64-slot chunk with them, gets bit for bit
the gradient of a loss that leaves the pixel out."""
import numpy as np
import pytest
import torch

import oracle
from paper_2410_08129_amd import htgs, scenes

pytestmark = pytest.mark.gpu

W, H, N = 60, 44, 500
CAM = scenes.look_at((0, 0, -4), (0, 0, 0), (0, -1, 0), 45.0, W, H)


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("sorted_blend", [False, True])
def test_one_pixel_without_a_finite_gradient(value, sorted_blend):
    rng = np.random.default_rng(11)
    means = rng.uniform(-1.3, 1.3, (N, 3))
    sc = scenes._pack(means, rng.normal(-2.6, 0.5, (N, 3)), scenes._quats(rng, N),
                      rng.normal(-1.0, 1.0, N), rng.uniform(0.2, 1.0, (N, 1, 3)), 0)
    st = scenes.RenderSettings(K=4, tile_w=8, tile_h=8, sorted_blend=sorted_blend)
    x, y = 31, 22
    G = rng.normal(0.0, 1.0, (3, H, W)).astype(np.float32)
    G[:, y, x] = 0.0
    params = [torch.tensor(a, device="cuda") for a in sc.arrays()]
    frame = htgs.forward(params, 0, [CAM], st)
    print(f"value={value} sorted={sorted_blend}", flush=True)
    clean = htgs.backward(params, frame, [torch.tensor(G, device="cuda")])
    G[:, y, x] = value
    dirty = htgs.backward(params, frame, [torch.tensor(G, device="cuda")])
    torch.cuda.synchronize()
    _, info = oracle.render.render_scene(sc, CAM, st, info=True)
    f, p = info["frags"], y * W + x
    rows = slice(f["ptr"][p], f["ptr"][p + 1])
    hit = set(f["gid"][rows][f["frag"][rows]].tolist())
    assert 3 <= len(hit) < N // 2
    for name, a, b in zip(("means", "log_scales", "quats", "logits", "sh"), clean, dirty):
        a, b = a.reshape(N, -1), b.reshape(N, -1)
        bad = set(torch.nonzero(~torch.isfinite(b).all(1))[:, 0].tolist())
        assert torch.isfinite(a).all() and bad and bad <= hit, (name, bad, hit)
        keep = torch.tensor([g not in hit for g in range(N)], device="cuda")
        assert torch.equal(a[keep], b[keep]), name

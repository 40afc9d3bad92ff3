"""The forward's depth test by the splats' means (needs an MI355X).

A splat's depth at a pixel is not evaluated when its mean lies further behind
the last core entry than any splat of the staged batch reaches in front of its
mean. Here needles up to 3 units long, most of them nearly along the view
axis, cross flat splats without any extent in depth, so means are far out of
the order of the depths at the pixels, in batches whose reach is long and in
batches whose reach is zero. One splat that fills the image lies behind the
others with an extent that passes through them.

Bounds: images and cores as in tests/parity.py (1e-4, near ties by their
branch)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2410_08129_amd import htgs, scenes
from tests import parity

pytestmark = pytest.mark.gpu

W, H, N = 45, 38, 600
CAM = scenes.look_at((0, 0, -5), (0, 0, 0), (0, -1, 0), 45.0, W, H)


def _scene(flat_first):
    rng = np.random.default_rng(7)
    z = rng.uniform(-1.5, 1.5, N)
    depth = z + 5.0
    px, py = rng.uniform(0.0, W, N), rng.uniform(0.0, H, N)
    means = np.stack([(px - CAM.cx) / CAM.fx * depth, (py - CAM.cy) / CAM.fy * depth, z], 1)
    side = rng.uniform(1.0, 4.0, N) * depth / CAM.fx
    ls = np.log(np.stack([side, side, 10.0 ** rng.uniform(-1.5, 0.0, N)], 1))
    tilt = rng.normal(0.0, 0.08, (N, 2))
    q = np.stack([np.ones(N), tilt[:, 0], tilt[:, 1], np.zeros(N)], 1)
    flat = np.arange(N) < N // 2 if flat_first else rng.random(N) < 0.5
    ls[flat, 2] = -np.inf
    q[flat] = (1.0, 0.0, 0.0, 0.0)
    means[-1], ls[-1], q[-1] = (0.0, 0.0, 1.6), np.log((3.0, 3.0, 1.0)), (1.0, 0.0, 0.0, 0.0)
    return scenes._pack(means, ls, q, rng.normal(0.0, 1.0, N),
                        rng.uniform(-1.5, 1.5, (N, 1, 3)), 0)


@pytest.mark.parametrize("flat_first", [False, True])
@pytest.mark.parametrize("K,tile,mult", [(1, (8, 8), 1), (4, (8, 8), 2), (16, (8, 8), 1),
                                         (3, (16, 8), 1), (8, (16, 16), 1)])
def test_cores_against_the_oracle(K, tile, mult, flat_first):
    sc = _scene(flat_first)
    st = scenes.RenderSettings(K=K, tile_w=tile[0], tile_h=tile[1],
                               lds_batch=mult * tile[0] * tile[1] if mult > 1 else 0)
    print(f"K={K} tile={tile} flat_first={flat_first}", flush=True)
    params = [torch.tensor(x, device="cuda") for x in sc.arrays()]
    frame = htgs.forward(params, 0, [CAM], st)
    torch.cuda.synchronize()
    assert htgs.read_status(frame.ws)[0] == 0
    ref, info = oracle.render.render_scene(sc, CAM, st, info=True)
    core = htgs.state_planes(frame, 0)["core_ids"].cpu().numpy()
    print(parity.check_image(frame.images[0].cpu().numpy(), core, ref.numpy(), info, st), flush=True)
    assert (core >= 0).mean() > 0.9

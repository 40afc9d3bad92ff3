"""The backward of frames of few tiles (needs an MI355X): eight waves per tile.

A crop of a large frame has few tiles, the frame has many. The crop's gradients
equal those of the frame with a loss on the crop's pixels, to the rounding of
sums that the tiles outside regroup (1e-3 of each gradient's norm, as between
tile sizes), and both differentiate every fragment of their forward. Lists of
up to about 3000 splats per tile give every wave of the wide form several
chunks; the crop at the frame's corner has tiles that are cut off."""
import numpy as np
import pytest
import torch

from paper_2410_08129_amd import htgs, scenes

pytestmark = pytest.mark.gpu

W, H = 1290, 772
CAM = scenes.look_at((0, 0, -4), (0, 0, 0), (0, -1, 0), 45.0, W, H)


@pytest.mark.parametrize("tile,K", [((8, 8), 8), ((8, 8), 32), ((16, 8), 3), ((16, 8), 16),
                                    ((16, 8), 32), ((16, 16), 16), ((32, 8), 16)])
@pytest.mark.parametrize("x,y", [(608, 384), (1248, 752)])
def test_crop_equals_the_frame(tile, K, x, y):
    rng = np.random.default_rng(K)
    n = 3000
    cw, ch = min(40, W - x), min(24, H - y)
    depth = rng.uniform(3.0, 5.0, n)
    px, py = rng.uniform(x - 4, x + cw + 4, n), rng.uniform(y - 4, y + ch + 4, n)
    means = np.stack([(px - CAM.cx) / CAM.fx * depth, (py - CAM.cy) / CAM.fy * depth,
                      depth - 4.0], 1)
    ls = np.log(rng.uniform(1.0, 6.0, (n, 3)) * (depth / CAM.fx)[:, None])
    sc = scenes._pack(means, ls, scenes._quats(rng, n), rng.normal(-2.0, 1.0, n),
                      rng.uniform(-1.0, 1.0, (n, 1, 3)), 0)
    st = scenes.RenderSettings(K=K, tile_w=tile[0], tile_h=tile[1])
    params = [torch.tensor(a, device="cuda") for a in sc.arrays()]
    print(f"K={K} tile={tile} crop at {x}, {y}", flush=True)
    G = torch.zeros((3, H, W), device="cuda")
    G[:, y:y + ch, x:x + cw] = torch.tensor(rng.normal(0, 1, (3, ch, cw)), device="cuda")
    grads = []
    for cam, g in ((CAM, G), (CAM.crop(x, y, cw, ch), G[:, y:y + ch, x:x + cw].contiguous())):
        frame = htgs.forward(params, 0, [cam], st)
        grads.append(htgs.backward(params, frame, [g]))
        fwd, bwd = htgs.fragment_counts(frame.ws)
        assert fwd == bwd > 0
    for a, b in zip(*grads):
        assert float((a - b).norm()) <= 1e-3 * float(a.norm())

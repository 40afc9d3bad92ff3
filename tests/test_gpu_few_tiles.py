"""Both forms of the backward raster on the same frame (needs an MI355X): eight
waves per tile where there are few tiles and room for many instances, two or
four otherwise. The gradients are the same bits on either side of the rule, at
the tile counts where it changes, for core sizes and tiles that hold one or two
such workgroups per CU."""
import numpy as np
import pytest
import torch

from paper_2410_08129_amd import htgs, scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile,K", [((8, 8), 8), ((8, 8), 24), ((16, 8), 16), ((16, 8), 24),
                                    ((16, 8), 32), ((16, 16), 12), ((32, 8), 12)])
@pytest.mark.parametrize("nx,ny", [(16, 16), (257, 1), (24, 16), (35, 11), (32, 16), (27, 19)])
def test_room_leaves_the_gradients_alone(tile, K, nx, ny):
    rng = np.random.default_rng(K)
    n = 400
    W, H = nx * tile[0] - 3, ny * tile[1] - 2
    cam = scenes.look_at((0, 0, -4), (0, 0, 0), (0, -1, 0), 45.0, W, H)
    # lists of up to a few hundred splats, in few tiles
    depth = rng.uniform(3.0, 5.0, n)
    px, py = rng.uniform(0, min(W, 20), n), rng.uniform(0, min(H, 20), n)
    means = np.stack([(px - cam.cx) / cam.fx * depth, (py - cam.cy) / cam.fy * depth,
                      depth - 4.0], 1)
    ls = np.log(rng.uniform(1.0, 4.0, (n, 3)) * (depth / cam.fx)[:, None])
    sc = scenes._pack(means, ls, scenes._quats(rng, n), rng.normal(-1.0, 1.0, n),
                      rng.uniform(-1.0, 1.0, (n, 1, 3)), 0)
    st = scenes.RenderSettings(K=K, tile_w=tile[0], tile_h=tile[1])
    params = [torch.tensor(a, device="cuda") for a in sc.arrays()]
    G = torch.tensor(rng.normal(0, 1, (3, H, W)), dtype=torch.float32, device="cuda")
    count = htgs.count_instances(params, 0, [cam], st)
    assert n // 2 < count < 60 * nx * ny
    print(f"K={K} tile={tile} tiles={nx * ny} instances={count}", flush=True)
    grads = []
    for room in (count, 1100 * nx * ny):
        ws = htgs.alloc_workspace(n, [cam], st, room, torch.device("cuda"))
        frame = htgs.forward(params, 0, [cam], st, ws=ws)
        grads.append(htgs.backward(params, frame, [G]))
        fwd, bwd = htgs.fragment_counts(frame.ws)
        assert fwd == bwd > 0
    for a, b in zip(*grads):
        assert torch.equal(a, b) and torch.any(a != 0)

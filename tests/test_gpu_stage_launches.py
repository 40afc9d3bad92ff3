"""The stage timer's launch counts (needs an MI355X) against the launch rules:
two launches per sort pass with room for at most 64 chunks of 4096 and three
beyond, and as many passes as the benchmark charges for the key's bits."""
import numpy as np
import pytest
import torch

import bench
from paper_2410_08129_amd import htgs, scenes

pytestmark = pytest.mark.gpu


SIZES = [(16, 16, 8), (32, 16, 9), (27, 19, 10), (256, 256, 16), (257, 256, 17), (512, 512, 18),
         (513, 512, 19)]
MANY = 1024 * 256 + 1   # Gaussians of 1025 preprocess workgroups


@pytest.mark.parametrize("tiles_x,tiles_y,bits,n", [s + (300,) for s in SIZES]
                         + [s + (MANY,) for s in SIZES[::5]])
@pytest.mark.parametrize("room", [64 * 4096, 64 * 4096 + 4096])
@pytest.mark.parametrize("sorted_blend", [False, True])
def test_launches(tiles_x, tiles_y, bits, n, room, sorted_blend):
    W, H = 8 * tiles_x, 8 * tiles_y
    cam = scenes.look_at((0, 0, -4), (0, 0, 0), (0, -1, 0), 45.0, W, H)
    rng = np.random.default_rng(n)
    means = rng.uniform(-0.5, 0.5, (n, 3))
    means[300:, 2] = -9.0   # (behind the camera)
    sc = scenes._pack(means, np.full((n, 3), -5.0), scenes._quats(rng, n),
                      rng.normal(0, 1, n), np.zeros((n, 1, 3)), 0)
    params = [torch.tensor(a, device="cuda") for a in sc.arrays()]
    G = torch.zeros((3, H, W), device="cuda")
    for cost_order in (False, True):
        st = scenes.RenderSettings(K=4, tile_w=8, tile_h=8, sorted_blend=sorted_blend,
                                   cost_order=cost_order)
        ws = torch.empty(htgs.workspace_bytes(n, [cam], st, room), dtype=torch.uint8,
                         device="cuda")
        print(f"bits={bits} room={room} n={n} sorted={sorted_blend}", flush=True)
        htgs.profile_enable(True)
        htgs.profile_read()
        frame = htgs.forward(params, 0, [cam], st, ws=ws)
        htgs.backward(params, frame, [G])
        got = {k: v[1] for k, v in htgs.profile_read().items()}
        htgs.profile_enable(False)
        assert htgs.read_status(ws)[0] == 0
        assert max(1, (tiles_x * tiles_y - 1).bit_length()) == bits
        # (a workspace's room is rounded up by less than 64 instances)
        assert got["sort"] == bench.sort_passes(bits) * (2 if bench.instance_room(
            n, [cam], st, ws.numel()) <= 64 * 4096 else 3)
        assert got["depth_sort"] == (0 if not sorted_blend else 9 if n <= 64 * 4096 else 13)
        assert got["preprocess"] == 2 + sorted_blend + (n == MANY)
        assert got["ranges"] == (3 if cost_order else 1)
        assert got["raster_fwd"] == got["raster_bwd"] == 1
        assert got["preprocess_bwd"] == 1 + sorted_blend

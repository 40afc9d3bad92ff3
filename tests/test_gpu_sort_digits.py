"""Tile sort at the edges of its digit widths (needs an MI355X): tile counts
on both sides of a change in passes or table size, lists bit-exact against
the float64 oracle's, with fewer instances than one 4,096-key chunk and with
several chunks, the last one partial."""
import numpy as np
import pytest
import torch

import oracle
from paper_2410_08129_amd import htgs, scenes
from tests import parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h,bits", [
    (128, 128, 8), (256, 128, 9), (264, 128, 10), (2048, 2048, 16), (2056, 2048, 17),
    (4096, 4096, 18), (4104, 4096, 19),
])
@pytest.mark.parametrize("n", [40, 3000])
def test_tile_lists_at_digit_edges(w, h, bits, n):
    tiles = -(-w // 8) * -(-h // 8)
    assert (tiles - 1).bit_length() == bits
    rng = np.random.default_rng(bits * 100 + n)
    cam = scenes.look_at((0, 0, -3), (0, 0, 0), (0, -1, 0), 50.0, w, h)
    aspect = h / w
    means = rng.uniform(-1.0, 1.0, (n, 3)) * np.array([1.2, 1.2 * aspect, 0.5])
    # a few tiles to a few dozen each, whatever the image size
    ls = np.log(np.exp(rng.uniform(1.0, 3.0, (n, 1))) * 3.0 / cam.fx) + rng.normal(0, 0.3, (n, 3))
    sc = scenes._pack(means, ls, scenes._quats(rng, n), rng.normal(1.0, 1.0, n),
                      rng.uniform(-1.0, 1.0, (n, 1, 3)), 0)
    st = scenes.RenderSettings(K=1, tile_w=8, tile_h=8)
    print(f"{w}x{h}, {bits} key bits, {n} Gaussians", flush=True)
    params = [torch.tensor(a, device="cuda") for a in sc.arrays()]
    frame = htgs.forward(params, 0, [cam], st, with_state=False)
    torch.cuda.synchronize()
    keys, vals, rects, flags = htgs.export_bins(params, 0, [cam], st, frame.ws)
    assert flags == 0
    ref = oracle.bins.tile_lists(sc.means, sc.log_scales, sc.quats, sc.opacity_logits, cam, st)
    ties = parity.compare_bins(keys, vals, rects, ref)
    print(f"  {len(keys)} instances, round-off ties {ties}", flush=True)
    assert len(keys) > n // 2

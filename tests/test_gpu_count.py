"""htgs_count_instances (needs an MI355X): the counting launch writes none of
the preprocess' outputs, and its count is the exact number of instances that
the forward then bins: with and without tile culling, for one and several
views, both blending modes, every SH degree, and Gaussian counts at the edges
of a workgroup."""
import numpy as np
import pytest
import torch

from paper_2410_08129_amd import htgs, scenes

pytestmark = pytest.mark.gpu

VIEWS = [scenes.look_at((0, 0, -4), (0, 0, 0), (0, -1, 0), 45.0, 301, 187),
         scenes.look_at((2.5, 1.0, -2.0), (0, 0, 0), (0, -1, 0), 60.0, 64, 40),
         scenes.look_at((0, 0, -4), (0, 0, -8), (0, -1, 0), 45.0, 33, 17)]   # sees nothing


@pytest.mark.parametrize("n", [0, 1, 255, 257, 60001])
@pytest.mark.parametrize("tile_cull", [False, True])
def test_count_equals_the_forward(n, tile_cull):
    rng = np.random.default_rng(n)
    for degree, views, sorted_blend in ((0, VIEWS[:1], False), (3, VIEWS[:1], True),
                                        (1, VIEWS, False), (2, VIEWS[2:], False)):
        if sorted_blend and n == 0:
            continue
        sc = scenes._pack(rng.uniform(-2.0, 2.0, (n, 3)), rng.normal(-3.5, 1.0, (n, 3)),
                          scenes._quats(rng, n), rng.normal(0.0, 2.0, n),
                          rng.normal(0.0, 0.3, (n, (degree + 1) ** 2, 3)), degree)
        st = scenes.RenderSettings(K=4, tile_w=16, tile_h=16, tile_cull=tile_cull,
                                   sorted_blend=sorted_blend)
        params = [torch.tensor(a, device="cuda") for a in sc.arrays()]
        print(f"n={n} cull={tile_cull} degree={degree} views={len(views)}", flush=True)
        counted = htgs.count_instances(params, degree, views, st)
        ws = htgs.alloc_workspace(n, views, st, 2 * counted + 1000, torch.device("cuda"))
        htgs.forward(params, degree, views, st, ws=ws)
        flags, binned = htgs.read_status(ws)
        assert flags == 0 and binned == counted
        assert n < 255 or views[0] is VIEWS[2] or counted > n // 4

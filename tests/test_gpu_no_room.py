"""A workspace with room for no instance (needs an MI355X): with and without the
cost order, every pixel is background, whether the views see nothing or their
instances do not fit (which the status reports); memory around the images stays
as it was."""
import numpy as np
import pytest
import torch

from paper_2410_08129_amd import htgs, scenes

pytestmark = pytest.mark.gpu

W, H = 77, 45
TOWARDS = scenes.look_at((0, 0, -4), (0, 0, 0), (0, -1, 0), 45.0, W, H)
AWAY = scenes.look_at((0, 0, -4), (0, 0, -8), (0, -1, 0), 45.0, W, H)


@pytest.mark.parametrize("cost_order", [False, True])
@pytest.mark.parametrize("cams,sorted_blend", [([AWAY], False), ([TOWARDS], False),
                                               ([AWAY, TOWARDS], False), ([TOWARDS], True)])
def test_background_everywhere(cost_order, cams, sorted_blend):
    rng = np.random.default_rng(3)
    n = 300
    sc = scenes._pack(rng.uniform(-1, 1, (n, 3)), rng.normal(-3.0, 0.3, (n, 3)),
                      scenes._quats(rng, n), rng.normal(0, 1, n), rng.uniform(0, 1, (n, 1, 3)), 0)
    st = scenes.RenderSettings(K=4, tile_w=8, tile_h=8, cost_order=cost_order,
                               sorted_blend=sorted_blend, bg=(0.25, 0.5, 0.75))
    params = [torch.tensor(a, device="cuda") for a in sc.arrays()]
    ws = torch.zeros(htgs.workspace_bytes(n, cams, st, 0), dtype=torch.uint8, device="cuda")
    around = torch.full((len(cams) + 2, 3, H, W), -1.0, device="cuda")
    print(f"cost={cost_order} views={len(cams)} sorted={sorted_blend}", flush=True)
    htgs.forward(params, 0, cams, st, ws=ws, images=list(around[1:-1]))
    flags, count = htgs.read_status(ws)
    sees = any(c is TOWARDS for c in cams)
    assert (flags != 0) == sees and (count > 0) == sees
    bg = torch.tensor(st.bg, device="cuda").reshape(3, 1, 1).expand(3, H, W)
    assert all(torch.equal(im, bg) for im in around[1:-1])
    assert torch.all(around[0] == -1.0) and torch.all(around[-1] == -1.0)

"""htgs.backward without ``grads`` (needs an MI355X): the new tensors hold what
adding to zeros gives, for Gaussians that no view sees, for frames without any
instance and for a frame whose instances did not fit its workspace (no
gradients), whatever their memory held before."""
import numpy as np
import pytest
import torch

from paper_2410_08129_amd import htgs, scenes

pytestmark = pytest.mark.gpu

HERE = scenes.look_at((0, 0, -4), (0, 0, 0), (0, -1, 0), 45.0, 97, 61)
AWAY = scenes.look_at((0, 0, -4), (0, 0, -8), (0, -1, 0), 45.0, 33, 17)


@pytest.mark.parametrize("views", [[HERE], [HERE, AWAY], [AWAY]])
@pytest.mark.parametrize("fits", [True, False])
@pytest.mark.parametrize("sorted_blend", [False, True])
def test_new_gradients_equal_added_ones(views, fits, sorted_blend):
    if sorted_blend and len(views) > 1:
        pytest.skip("sorted blending renders one view")
    n, degree = 700, 1
    rng = np.random.default_rng(3)
    sc = scenes._pack(rng.uniform(-4.0, 4.0, (n, 3)), rng.normal(-2.5, 0.5, (n, 3)),
                      scenes._quats(rng, n), rng.normal(0.0, 1.0, n),
                      rng.normal(0.0, 0.3, (n, 4, 3)), degree)
    st = scenes.RenderSettings(K=4, tile_w=8, tile_h=8, sorted_blend=sorted_blend)
    params = [torch.tensor(a, device="cuda") for a in sc.arrays()]
    count = htgs.count_instances(params, degree, views, st)
    ws = htgs.alloc_workspace(n, views, st, count if fits else count // 2, torch.device("cuda"))
    frame = htgs.forward(params, degree, views, st, ws=ws)
    # (16 spare instances: a frame with none always fits)
    assert (htgs.read_status(ws)[0] == 0) == (fits or count == 0)
    gimgs = [torch.tensor(rng.normal(0.0, 1.0, (3, v.height, v.width)).astype(np.float32),
                          device="cuda") for v in views]
    added = htgs.backward(params, frame, gimgs, grads=[torch.zeros_like(p) for p in params])
    torch.cuda.synchronize()
    stale = [torch.full_like(p, float("nan")) for p in params]
    del stale   # (the allocator hands this memory to the new gradients)
    new = htgs.backward(params, frame, gimgs)
    for a, b in zip(added, new):
        assert torch.equal(a, b)
        assert bool(torch.any(a != 0)) == (fits and count > 0)

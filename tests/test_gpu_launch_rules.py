"""The front end's launch rules (needs an MI355X): the preprocess clears the
workspace or a fill does, the emit launch adds up the workgroups' totals (up to
1024 of them) or reads their scan, and the tile sort's scatter adds up the
chunk counts (up to 64 chunks of room, 262,144 instances) or reads theirs. The
same frame on both sides of each rule, in workspaces that hold ones or zeros
before, gives the same bits; so does a Gaussian more that no view sees."""
import numpy as np
import pytest
import torch

from paper_2410_08129_amd import htgs, scenes

pytestmark = pytest.mark.gpu

EDGE = 1024 * 256        # Gaussians of 1024 preprocess workgroups
CHUNKS = 64 * 4096       # instances of 64 sort chunks
CAM = scenes.look_at((0, 0, -4), (0, 0, 0), (0, -1, 0), 45.0, 333, 211)


def _frame(arrays, st, cap, fill):
    params = [torch.tensor(a, device="cuda") for a in arrays]
    size = htgs.workspace_bytes(len(arrays[0]), [CAM], st, cap)
    ws = torch.full((size,), fill, dtype=torch.uint8, device="cuda")
    frame = htgs.forward(params, 0, [CAM], st, ws=ws)
    flags, count = htgs.read_status(ws)
    G = torch.tensor(np.random.default_rng(1).normal(0, 1, (3, CAM.height, CAM.width)),
                     dtype=torch.float32, device="cuda")
    grads = htgs.backward(params, frame, [G])
    return flags, count, frame.images[0].clone(), [g.clone() for g in grads]


@pytest.mark.parametrize("n", [3, 300, EDGE - 1, EDGE])
@pytest.mark.parametrize("tile,sorted_blend", [((8, 8), False), ((16, 16), False), ((8, 8), True)])
def test_both_sides_of_each_rule(n, tile, sorted_blend):
    rng = np.random.default_rng(n)
    wide = 2.0 if n <= 300 else 60.0      # (few of many are in view)
    sc = scenes._pack(rng.uniform(-wide, wide, (n, 3)), rng.normal(-2.5, 0.5, (n, 3)),
                      scenes._quats(rng, n), rng.normal(0.0, 1.0, n),
                      rng.uniform(-1.0, 1.0, (n, 1, 3)), 0)
    arrays = list(sc.arrays())
    st = scenes.RenderSettings(K=4, tile_w=tile[0], tile_h=tile[1], sorted_blend=sorted_blend,
                               tile_cull=True)
    print(f"n={n} tile={tile} sorted={sorted_blend}", flush=True)
    flags, count, img, grads = _frame(arrays, st, CHUNKS, 255)
    assert flags == 0 and 0 < count < CHUNKS
    aside = [np.concatenate([a, a[-1:]]) for a in arrays]
    aside[0][-1] = (1000.0, 0.0, 100.0)   # (last in index and in depth order)
    for arr, cap, fill in ((arrays, CHUNKS + 1, 0), (arrays, CHUNKS, 0), (arrays, count, 255),
                           (aside, CHUNKS, 255), (aside, CHUNKS + 1, 255)):
        f2, c2, img2, g2 = _frame(arr, st, cap, fill)
        assert (f2, c2) == (0, count)
        assert torch.equal(img, img2)
        for a, b in zip(grads, g2):
            assert torch.equal(a, b[:n])
            assert not torch.any(b[n:] != 0)
    # too little room is reported as before (a few hundred instances' room
    # rounds up to more of them)
    if count > 1000:
        assert _frame(arrays, st, count // 2, 255)[0] & htgs.HTGS_STATUS_OVERFLOW

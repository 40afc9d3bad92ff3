"""The backward's fragment codes and its two walks (needs an MI355X).

A chunk whose splats all stay below the alpha clamp walks its pixels without
the clamp and the smallest-|d|^2 test; the fragment codes are bytes whose
unit depends on the core size. Gradients against the float64 oracle's
autograd, with the bar of the other gradient tests (1e-3 relative, norm and
element-wise, near-tie pixels left out), over core sizes on both sides of
each table shape, ragged tiles and several chunks per tile, with no opaque
splat and with every second one above the clamp."""
import numpy as np
import pytest
import torch

import oracle
from paper_2410_08129_amd import htgs, scenes
from tests import parity, window_grads

pytestmark = pytest.mark.gpu

W, H, N = 45, 29, 600
CAM = scenes.look_at((0, 0, -4), (0, 0, 0), (0, -1, 0), 40.0, W, H)
NAMES = ("means", "log_scales", "quats", "opacity_logits", "sh")


def _scene(opaque):
    rng = np.random.default_rng(3)
    means = rng.uniform(-1.0, 1.0, (N, 3)) * np.array([1.5, 1.0, 1.0])
    ls = rng.normal(-2.2, 0.5, (N, 3))
    logit = rng.normal(-1.0, 1.0, N)
    if opaque:
        logit[::2] = rng.uniform(5.0, 8.0, logit[::2].size)     # sigmoid above 0.99
    sh = np.zeros((N, 1, 3))
    sh[:, 0, :] = rng.uniform(-1.0, 1.0, (N, 3))
    return scenes._pack(means, ls, scenes._quats(rng, N), logit, sh, 0)


@pytest.mark.parametrize("opaque", [False, True])
@pytest.mark.parametrize("K,tile", [(1, (8, 8)), (8, (8, 8)), (9, (8, 8)), (16, (8, 8)),
                                    (32, (8, 8)), (8, (16, 8)), (16, (16, 8)), (24, (16, 8)),
                                    (8, (16, 16)), (16, (32, 8))])
def test_gradients_of_both_walks(K, tile, opaque):
    sc = _scene(opaque)
    st = scenes.RenderSettings(K=K, tile_w=tile[0], tile_h=tile[1], bg=(0.3, 0.5, 0.1))
    print(f"K={K} tile={tile} opaque={opaque}", flush=True)
    pre = oracle.splat.prepare(sc.means, sc.log_scales, sc.quats, sc.opacity_logits, CAM,
                               st.tau_alpha)
    G = np.random.default_rng(5).normal(0.0, 1.0, (3, H, W)) / (3 * H * W)
    win = window_grads.oracle_window(sc, CAM, st, 0, 0, W, H, G, pre["p"].numpy(),
                                     pre["h"].numpy(), pre["visible"].numpy(), piece=32)
    params = [torch.tensor(a, device="cuda") for a in sc.arrays()]
    frame = htgs.forward(params, 0, [CAM], st)
    grads = htgs.backward(params, frame, [torch.tensor(G, dtype=torch.float32, device="cuda")])
    fwd, bwd = htgs.fragment_counts(frame.ws)
    assert fwd == bwd > 0
    ref, _ = window_grads.accumulate(sc.n, [a.shape[1:] for a in sc.arrays()], [win])
    errs = parity.grad_errors([g.cpu().numpy().astype(np.float64) for g in grads], ref)
    for name, (den, rel, elem) in zip(NAMES, errs):
        print(f"  {name}: |g| {den:.3e}, rel {rel:.2e}, elem {elem:.2e}", flush=True)
        assert rel <= 1e-3 and elem <= 1e-3, name

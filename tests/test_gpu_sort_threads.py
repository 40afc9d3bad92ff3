"""The tile sort's launch shapes (needs an MI355X): 1024 threads per chunk of
4096 keys with room for up to 512 chunks (whose counts the scatter adds up with
room for up to 64), 512 threads beyond. The same frame with room on both sides
of each line gives the same lists bit for bit, for 16-bit and 32-bit keys, and
lists longer than either line are in tile order and, inside a tile, in index
order."""
import numpy as np
import pytest
import torch

from paper_2410_08129_amd import htgs, scenes

pytestmark = pytest.mark.gpu

CHUNK = 4096


def _bins(arrays, cam, st, cap):
    params = [torch.tensor(a, device="cuda") for a in arrays]
    ws = torch.full((htgs.workspace_bytes(len(arrays[0]), [cam], st, cap),), 255,
                    dtype=torch.uint8, device="cuda")
    htgs.forward(params, 0, [cam], st, ws=ws, with_state=False)
    keys, vals, rects, flags = htgs.export_bins(params, 0, [cam], st, ws)
    assert flags == 0
    return keys, vals, rects


@pytest.mark.parametrize("n,size,pixels", [(700, (401, 303), 6.0), (30000, (2200, 2000), 4.0),
                                           (30000, (900, 700), 30.0), (30000, (2200, 2000), 40.0)])
def test_lists_do_not_depend_on_the_launch_shape(n, size, pixels):
    cam = scenes.look_at((0, 0, -4), (0, 0, 0), (0, -1, 0), 45.0, *size)
    rng = np.random.default_rng(n + size[0])
    z = rng.uniform(-0.5, 0.5, n)
    px, py = rng.uniform(0, size[0], n), rng.uniform(0, size[1], n)
    means = np.stack([(px - cam.cx) / cam.fx * (z + 4), (py - cam.cy) / cam.fy * (z + 4), z], 1)
    ls = np.log(rng.uniform(0.3, 1.0, (n, 3)) * pixels * 4.0 / cam.fx)
    arrays = list(scenes._pack(means, ls, scenes._quats(rng, n), rng.normal(2.0, 1.0, n),
                               rng.uniform(-1.0, 1.0, (n, 1, 3)), 0).arrays())
    st = scenes.RenderSettings(K=1, tile_w=8, tile_h=8)
    params = [torch.tensor(a, device="cuda") for a in arrays]
    count = htgs.count_instances(params, 0, [cam], st)
    print(f"n={n} {size}: {count / CHUNK:.1f} chunks", flush=True)
    first = None
    for cap in (count, 64 * CHUNK, 64 * CHUNK + 1, 512 * CHUNK, 512 * CHUNK + 1):
        if cap < count:
            continue
        keys, vals, rects = _bins(arrays, cam, st, cap)
        if first is None:
            first = keys, vals
            assert len(keys) == count
            assert int(((rects[:, 2] - rects[:, 0] + 1).clip(0) *
                        (rects[:, 3] - rects[:, 1] + 1).clip(0)).sum()) == count
            step = np.diff(keys.astype(np.int64))
            assert (step >= 0).all()
            assert (np.diff(vals.astype(np.int64))[step == 0] > 0).all()
        assert np.array_equal(keys, first[0]) and np.array_equal(vals, first[1])

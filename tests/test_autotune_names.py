"""The autotuner's candidates: no two run the same launches, and every name that
reports have carried still resolves."""
import pytest

from paper_2410_08129_amd import autotune, htgs, scenes

QUEUED = [f"tile{t}_batch1x_{order}_cull_queue" for t in ("8x8", "16x8", "16x16")
          for order in ("xcd", "cost")]


def test_candidates_differ_in_more_than_the_queue():
    configs = set()
    for cand in autotune.CANDIDATES:
        c = htgs.config_struct(autotune.apply(scenes.RenderSettings(), cand))
        configs.add((c.tile_w, c.tile_h, c.lds_batch, c.flags & ~htgs.HTGS_FLAG_PERSISTENT))
    assert len(configs) == len(autotune.CANDIDATES) == 16


@pytest.mark.parametrize("name", QUEUED)
def test_queue_names_stay_known(name):
    cand = autotune.by_name(name)
    assert cand == autotune.by_name(name[:-len("_queue")])
    assert not autotune.apply(scenes.RenderSettings(), cand).persistent


def test_names_resolve_and_others_are_refused():
    for cand in autotune.CANDIDATES:
        assert autotune.by_name(autotune.candidate_name(cand)) == cand
    for name in ("tile32x8_batch1x_xcd_cull_queue", "tile8x8_batch2x_xcd_queue", "tile4x4"):
        with pytest.raises(KeyError):
            autotune.by_name(name)

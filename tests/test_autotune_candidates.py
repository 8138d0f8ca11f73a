"""The autotuner searches what changes a detection's launch and nothing else: no
rows per tile (they would reach hs_sum and the statistic, which are not timed),
no configuration under two names, no cache entry of other kernels."""
import pytest
import torch

import paper_1805_12258_amd as hs
from paper_1805_12258_amd import autotune as at


@pytest.mark.parametrize("T,H,dtype", [(85, 8, "f32"), (85, 16, "f32"), (85, 8, "f16"), (85, 16, "bf16"), (1, 8, "f32"),
                                       (2000, 8, "f16")])
@pytest.mark.parametrize("n_chans", [None, [3000, 5000]])
def test_candidates_change_the_detection_only(T, H, dtype, n_chans):
    default = hs.Plan(T, 4096, H, dtype=dtype, n_chans=n_chans)
    for cfg in at.candidates(n_chans is None):
        p = hs.Plan(T, 4096, H, dtype=dtype, n_chans=n_chans, **cfg)
        for k in ("tile_rows", "row_blocks", "lds_bytes", "tiles_total", "src_rows", "staged_words"):
            assert p.info[k] == default.info[k], (cfg, k)


def test_cache_key_names_the_kernels():
    key = at.cache_key(85, 1 << 21, 8, "f32", None, "gfx950")
    assert key != "gfx950|T85|N%d|H8|f32" % (1 << 21)      # entries of the kernels before the row walk


@pytest.mark.gpu
@pytest.mark.parametrize("T,H,dtype,distinct", [(85, 8, "f32", 12), (85, 8, "f16", 12), (1, 8, "f32", 4)])
def test_no_launch_is_timed_twice(T, H, dtype, distinct):
    """Twelve launches: three strip widths, two orders, two grids; the defaults
    are one of them.  A plane of one row has one width."""
    _, _, tried = at.tune(T, 20000, H, dtype=dtype, input_scale=1.0 if dtype == "f32" else 0.125, reps=1, cache=None)
    timed = [t["config"] for t in tried if t["ms"] is not None]
    assert tried[0]["ms"] is not None
    keys = [at.launch_key(hs.Plan(T, 20000, H, dtype=dtype, input_scale=1.0 if dtype == "f32" else 0.125, **c).info, c)
            for c in timed]
    assert len(set(keys)) == len(keys) == distinct

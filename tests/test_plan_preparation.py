"""What a plan costs before its first call.  A batch of FOPs that are all of
another length costs about what one of equal FOPs does (host only), and the
tables of a single-FOP plan go to the device in one piece: an upload with a
tile schedule takes about as long as one without.  Times are the best of many,
bounds twice what the code needs."""
import time

import pytest
import torch

import paper_1805_12258_amd as hs


def create_s(lens, reps=7):
    best = float("inf")
    for _ in range(reps):
        t0 = time.perf_counter()
        h = hs.hs_plan_create(9, n_hp=4, n_chans=lens)
        best = min(best, time.perf_counter() - t0)
        hs.hs_plan_destroy(h)
    return best


def test_batches_of_distinct_lengths():
    distinct, equal = create_s(list(range(20000, 40000))), create_s([30000] * 20000)
    assert distinct <= 8 * equal, (distinct, equal)


@pytest.mark.parametrize("lens", [[100, 300, 100, 511, 512, 513, 257], [1], [70000, 256, 65281, 65280]])
def test_lengths_of_as_many_strips_share_a_list(lens):
    """Every FOP is still covered by the batch's tiles."""
    p = hs.Plan(85, 0, 8, n_chans=lens)
    assert p.info["tiles_total"] == p.info["row_blocks"] * sum((n + 255) // 256 for n in lens)


@pytest.mark.gpu
def test_tables_are_uploaded_in_one_piece():
    def upload_s(schedule):
        best = float("inf")
        for _ in range(60):
            h = hs.hs_plan_create(21, 1 << 16, 8, schedule=schedule)
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            hs.hs_plan_upload(h)
            best = min(best, time.perf_counter() - t0)
            hs.hs_plan_destroy(h)
        return best
    upload_s(0)
    both, one = upload_s(0), upload_s(3)       # schedule 3: contiguous tiles, no tile schedule
    assert both <= 1.5 * one, (both, one)

"""The transpose's loads in the last strip of a ragged plane (the row's last
four elements for the lanes across and past the end): rows of one to nine bins
and strips of one to five past a full one, at every alignment of the rows,
against the fp64 oracle within the bound of a fp32 sum of so many non-negative
terms; values past a row's end (the next row's, NaN) must not reach it.  And
planes of less than a strip take no longer than full ones."""
import numpy as np
import pytest
import torch

import oracle
import paper_1805_12258_amd as hs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 6, 7, 9, 255, 257, 258, 259, 260, 261, 515])
@pytest.mark.parametrize("T,H", [(7, 16), (33, 4), (18, 1)])
def test_ragged_rows(T, N, H):
    print("case", T, N, H, flush=True)
    g = np.random.default_rng(N).random((H, T, N), dtype=np.float32)
    buf = torch.full((H * T * N + 8,), float("nan"), device="cuda")
    for shift in (0, 1, 2, 3):
        gd = buf[shift:shift + H * T * N].view(H, T, N)
        gd.copy_(torch.from_numpy(g))
        got = hs.Plan(T, N, H).backward(gd).cpu().numpy().astype(np.float64)
        want = oracle.vjp_f64(g)
        assert np.all(np.abs(got - want) <= (3 * H + 40) * 2.0 ** -24 * want)


def test_special_values_stay_in_their_row():
    """A NaN and an infinity at a row's first and last bins reach the targets of
    that row's boxes alone."""
    T, N, H = 12, 261, 5
    g = np.zeros((H, T, N), dtype=np.float32)
    g[2, 6, N - 1], g[4, 9, 0] = np.nan, np.inf
    got = hs.Plan(T, N, H).backward(torch.from_numpy(g).cuda()).cpu().numpy()
    want = np.zeros((T, N), dtype=np.float64)
    c = T // 2
    for k, r, j in ((2, 6, N - 1), (4, 9, 0)):
        for m in range(1, k + 2):
            want[(r - c) // m + c, j // m] += g[k, r, j]
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isinf(got), np.isinf(want))
    assert np.all(got[np.isfinite(want)] == 0)


def backward_us(T, N, H):
    plan = hs.Plan(T, N, H)
    g = torch.rand((H, T, N), device="cuda")
    d = torch.empty((T, N), device="cuda")
    w = torch.empty(max(1, hs.hs_backward_workspace_bytes(plan.handle)), dtype=torch.uint8, device="cuda")
    best = float("inf")
    for _ in range(10):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        hs.hs_sum_backward(plan.handle, g, d, w)
        e1.record()
        e1.synchronize()
        best = min(best, 1e3 * e0.elapsed_time(e1))
    return best


def test_a_ragged_strip_takes_no_longer():
    ragged, full = backward_us(65536, 100, 16), backward_us(65536, 256, 16)
    print("case us", round(ragged, 1), round(full, 1), flush=True)
    assert ragged <= 1.5 * full

"""The canonical sort on lists as searches have them and worse: half of the
entries in plane 1, half-empty bin fields, low bins only, one row with
interference, a far outlier, words that repeat, and a list made so that the
samples which the buckets are chosen by miss most of it.  Bitwise against
numpy's stable sort, at the sizes named; and no such list may take more than
four times as long as one of evenly spread words."""
import numpy as np
import pytest
import torch

import paper_1805_12258_amd as hs

pytestmark = pytest.mark.gpu


def fields(n, rng, rows=85, n_bins=(1 << 20) + 77, planes=8):
    """Words row << 24 | plane << 21 | bin at the plane rates of k + 6 sqrt(k)."""
    rate = np.array([0.52, 0.2, 0.1, 0.06, 0.045, 0.03, 0.025, 0.02])[:planes]
    k = rng.choice(planes, n, p=rate / rate.sum()).astype(np.uint32)
    return (rng.integers(0, rows, n).astype(np.uint32) << 24) | (k << 21) | rng.integers(0, n_bins, n).astype(np.uint32)


def missed(n, _):
    """Small words at the places the samples are taken from, large elsewhere."""
    bins = 64
    while bins < 1024 and bins * 1024 < n:
        bins *= 2
    S = 4 * bins
    i = np.arange(S, dtype=np.uint64)
    a, b = i * n // S, (i + 1) * n // S
    h = ((i + 1) * 0x9E3779B1) & 0xFFFFFFFF
    h ^= h >> 15
    h = (h * 0x85EBCA77) & 0xFFFFFFFF
    h ^= h >> 13
    w = (5000 + np.arange(n, 0, -1)).astype(np.uint32)
    w[(a + (h * (b - a) >> 32)).astype(np.int64)] = np.arange(S)
    return w


def far(n, rng):
    w = rng.permutation(1 << 21)[:n].astype(np.uint32)
    w[n // 2] = 0xFFFFFFF0
    return w


def row(n, rng):
    w = fields(n, rng)
    m = 9 * n // 10
    w[:m] = (40 << 24) | rng.permutation(1 << 21)[:m]
    return rng.permutation(w)


KINDS = {
    "spread": lambda n, rng: (rng.permutation(n).astype(np.uint64) * (((1 << 31) - 1) // n)).astype(np.uint32),
    "fields": fields,
    "lowbins": lambda n, rng: fields(n, rng, n_bins=1 << 18),
    "rednoise": lambda n, rng: (fields(n, rng, n_bins=1) | np.exp(rng.uniform(0, np.log(1 << 21), n)).astype(np.uint32)),
    "row": row,
    "far": far,
    "equal": lambda n, rng: np.full(n, 0xFFFFFFFF, dtype=np.uint32),
    "few": lambda n, rng: np.where(rng.random(n) < 0.999, rng.integers(0, 7, n), 0xFFFFFFF0).astype(np.uint32),
    "missed": missed,
}


def entries(kind, n):
    w = KINDS[kind](n, np.random.default_rng(n))
    return w, np.stack([w, np.arange(n, dtype=np.uint32)], axis=1).view(np.int32)


@pytest.mark.parametrize("n", [3, 1000, 1025, 2049, 4097, 8193, 16384, 16385, 20000, 65537, 305000, 128 * 4096 + 1, 1 << 20])
@pytest.mark.parametrize("kind", sorted(KINDS))
def test_order_of_crowded_lists(kind, n):
    if kind == "missed" and not 16384 < n <= 20000:
        n = 17000 + n % 1000                   # one bucket takes all but the samples
    print("case", kind, n, flush=True)
    w, a = entries(kind, n)
    dev = torch.from_numpy(a.copy()).cuda()
    hs.sort_candidates(dev, n)
    assert np.array_equal(dev.cpu().numpy(), a[np.argsort(w, kind="stable")])


def sort_us(kind, n):
    _, a = entries(kind, n)
    src = torch.from_numpy(a.copy()).cuda()
    dev = torch.empty_like(src)
    work = torch.empty(hs.hs_sort_workspace_bytes(n), dtype=torch.uint8, device="cuda")
    best = float("inf")
    for _ in range(8):
        dev.copy_(src)
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        hs.hs_sort_candidates(dev, n, work)
        e1.record()
        e1.synchronize()
        best = min(best, 1e3 * e0.elapsed_time(e1))
    return best


@pytest.mark.parametrize("n", [5000, 50000, 305000])
def test_time_does_not_depend_on_the_words(n):
    us = {k: sort_us(k, n) for k in ("spread", "fields", "lowbins", "rednoise", "row", "far", "equal")}
    print("case", n, {k: round(v, 1) for k, v in us.items()}, flush=True)
    assert max(us.values()) <= 4 * us["spread"]


def test_time_of_crowded_bins_in_a_short_list():
    """9000 different entries at log-uniform bins against evenly spread bins: 1.14
    times the time where entries are ranked inside bins, 1.0 against all others.
    The two in turn (a clock that rises favours neither), the smallest of each."""
    n, src, us = 9000, {}, {}
    for k in ("rednoise", "fields"):
        rng = np.random.default_rng(n)
        w = rng.permutation(np.unique(np.concatenate([KINDS[k](2 * n, rng), KINDS[k](2 * n, rng)])))[:n]
        src[k] = torch.from_numpy(np.stack([w, np.arange(n, dtype=np.uint32)], axis=1).view(np.int32)).cuda()
        us[k] = float("inf")
    dev = torch.empty_like(src["fields"])
    work = torch.empty(hs.hs_sort_workspace_bytes(n), dtype=torch.uint8, device="cuda")
    for i in range(300):
        for k in src:
            dev.copy_(src[k])
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            hs.hs_sort_candidates(dev, n, work)
            e1.record()
            e1.synchronize()
            if i >= 50:
                us[k] = min(us[k], 1e3 * e0.elapsed_time(e1))
    print("case", us, flush=True)
    assert us["rednoise"] <= 1.08 * us["fields"], us


@pytest.mark.parametrize("n", [40, 64, 65, 127, 200, 250, 254, 255, 256])
@pytest.mark.parametrize("equal", [False, True])
def test_buckets_at_the_limit(n, equal):
    """64 buckets of about n entries, compared with all others up to 256; and with one
    pair of equal words in each."""
    rng = np.random.default_rng(n)
    w = (np.arange(64 * n, dtype=np.uint64) * (((1 << 31) - 1) // (64 * n))).astype(np.uint32)
    if equal:
        w[5::n] = w[6::n]
    w = rng.permutation(w)
    a = np.stack([w, np.arange(len(w), dtype=np.uint32)], axis=1).view(np.int32)
    dev = torch.from_numpy(a.copy()).cuda()
    hs.sort_candidates(dev, len(w))
    assert np.array_equal(dev.cpu().numpy(), a[np.argsort(w, kind="stable")])


@pytest.mark.parametrize("n", [1500, 9000, 60000])
def test_replays_of_a_captured_sort(n):
    """The passes of every length in a graph, replayed on new lists with eager
    work between the replays."""
    _, a = entries("fields", n)
    dev = torch.from_numpy(a.copy()).cuda()
    work = torch.empty(hs.hs_sort_workspace_bytes(n), dtype=torch.uint8, device="cuda")
    hs.hs_sort_candidates(dev, n, work)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        hs.hs_sort_candidates(dev, n, work)
    for kind in ("row", "fields", "few", "spread"):
        w, a = entries(kind, n)
        dev.copy_(torch.from_numpy(a.copy()))
        graph.replay()
        got = dev.cpu().numpy()
        assert np.array_equal(got, a[np.argsort(w, kind="stable")]), kind
        work.random_()
        torch.cuda.synchronize()

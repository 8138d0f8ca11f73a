"""Batches of many short FOPs: more than 64 and more than 4096 segments on a
list (the search for a unit's FOP takes one, two and three steps), waves that
take runs of units across FOPs, rejected FOPs among them; each list bitwise
against the oracle's.  And 5000 FOPs take no longer than four times what 50 take
that hold as many points."""
import numpy as np
import pytest
import torch

import oracle
import paper_1805_12258_amd as hs
from tests.helpers import padded_device, random_thresholds

pytestmark = pytest.mark.gpu


def make(lens, T, seed, dtype):
    """FOPs of the given lengths as rows of one buffer (distinct contents)."""
    kind, scale = {"f32": (torch.float32, 1.0), "f16": (torch.float16, 0.125)}[dtype]
    g = torch.Generator().manual_seed(seed)
    pool = torch.empty((T, max(lens) + 4096)).exponential_(1.0, generator=g)
    stores = [pool[:, (37 * f) % 4096:][:, :n] for f, n in enumerate(lens)]
    return [padded_device(s, dtype=kind, scale=scale) for s in stores], scale


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("lens,T,H", [([300] * 700, 9, 4), ([17, 900, 1, 256, 257] * 240, 5, 8), ([3] * 40000, 1, 1),
                                      ([2000] * 90, 21, 4)])
def test_many_short_fops(lens, T, H, dtype):
    print("case", len(lens), T, H, dtype, flush=True)
    pairs, scale = make(lens[:975], T, T + H, dtype)
    ta = random_thresholds(H, T, T * H)
    plan = hs.Plan(T, 0, H, n_chans=lens, dtype=dtype, input_scale=scale)
    sr, sb = plan.info["s_row"], plan.info["s_bin"]
    want = []
    for _, store in pairs:
        idx, pw, cnt = oracle.detect_f32(store.to(torch.float32).numpy(), H, ta, scale=scale, nthreads=1)
        _, k, b = oracle.field_bits(T, store.shape[1], H)
        row, low = (idx.astype(np.uint64) >> np.uint64(k + b)), idx & np.uint32((1 << b) - 1)
        pl = (idx >> np.uint32(b)) & np.uint32((1 << k) - 1)
        word = (row << np.uint64(sr)).astype(np.uint32) | (pl << np.uint32(sb)) | low
        o = np.argsort(word)
        want.append((word[o], pw[o].view(np.uint32), cnt))
    n, m = len(lens), len(pairs)
    caps = np.array([len(want[f % m][0]) for f in range(n)], dtype=np.int64)
    offs = np.concatenate([[0], np.cumsum(caps)[:-1]])
    lds = [pairs[f % m][0].stride(0) for f in range(n)]
    bad = n // 2
    lds[bad] += 1                              # breaks the pitch rule: skipped
    dev = lambda a: torch.tensor(np.asarray(a, dtype=np.int64)).cuda()
    out = torch.empty((int(caps.sum()) + 1, 2), dtype=torch.int32, device="cuda")
    counts = torch.empty((n, H + 1), dtype=torch.int64, device="cuda")
    hs.hs_detect_batched(plan.handle, dev([pairs[f % m][0].data_ptr() for f in range(n)]), dev(lds),
                         torch.from_numpy(np.ascontiguousarray(ta)).cuda(), out, dev(offs), dev(caps), counts)
    c, o = counts.cpu().numpy(), out.cpu().numpy().view(np.uint32)
    assert c[bad, -1] == -1
    for f in range(n):
        if f == bad:
            continue
        word, power, cnt = want[f % m]
        assert np.array_equal(c[f], cnt), f
        got = o[offs[f]:offs[f] + caps[f]]
        got = got[np.argsort(got[:, 0])]
        assert np.array_equal(got[:, 0], word) and np.array_equal(got[:, 1], power), f


def batch_us(n, bins, T=9, H=4):
    x = torch.empty((n * T, bins), device="cuda").exponential_()
    plan = hs.Plan(T, 0, H, n_chans=[bins] * n)
    dev = lambda a: torch.tensor(a, dtype=torch.int64).cuda()
    ptrs = dev([x.data_ptr() + f * T * bins * 4 for f in range(n)])
    out = torch.empty((n, 2), dtype=torch.int32, device="cuda")
    counts = torch.empty((n, H + 1), dtype=torch.int64, device="cuda")
    args = (ptrs, dev([bins] * n), torch.full((H, T), 1e9, device="cuda"), out, dev(list(range(n))), dev([1] * n), counts)
    best = float("inf")
    for _ in range(10):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        hs.hs_detect_batched(plan.handle, *args)
        e1.record()
        e1.synchronize()
        best = min(best, 1e3 * e0.elapsed_time(e1))
    return best


def test_many_fops_cost_what_their_points_cost():
    many, few = batch_us(5000, 256), batch_us(50, 25600)
    print("case us", round(many, 1), round(few, 1), flush=True)
    assert many <= 4 * few

"""The canonical sort (hs_sort_candidates) against numpy's stable sort on the
CL1 word: bitwise, at the sizes where its passes change (one block, several,
the bucket and list limits) and on words that fill one bucket, repeat, or
span the whole 32 bits."""
import numpy as np
import pytest
import torch

import paper_1805_12258_amd as hs

pytestmark = pytest.mark.gpu


def words(kind, n, rng):
    if kind == "spread":                       # as a detection gives them: unique, any order
        return rng.choice(1 << 31, size=n, replace=False).astype(np.uint32) if n <= 4096 else \
            (rng.permutation(n).astype(np.uint64) * (((1 << 32) - 1) // n)).astype(np.uint32)
    if kind == "equal":                        # one bucket, order by place in the input
        return np.full(n, 0xFFFFFFFF, dtype=np.uint32)
    if kind == "crowded":                      # most entries in a few words, one far away
        w = rng.integers(0, 7, size=n).astype(np.uint32)
        w[-1] = 0xFFFFFFF0
        return w
    return np.arange(n, 0, -1).astype(np.uint32)   # descending


@pytest.mark.parametrize("kind", ["spread", "equal", "crowded", "descending"])
@pytest.mark.parametrize("n", [2, 63, 65, 1024, 1025, 2048, 16384, 16385, 128 * 4096 + 1, 1 << 20, (1 << 20) + 1])
def test_sort_matches_stable_sort(kind, n):
    if kind in ("equal", "crowded") and n > 16385:
        n = 40000                              # a bucket ordered in global memory
    print("case", kind, n, flush=True)
    rng = np.random.default_rng(n)
    w = words(kind, n, rng)
    p = np.arange(n, dtype=np.uint32)          # tells equal words apart
    a = np.stack([w, p], axis=1).view(np.int32)
    dev = torch.from_numpy(a.copy()).cuda()
    hs.sort_candidates(dev, n)
    want = a[np.argsort(w, kind="stable")]
    assert np.array_equal(dev.cpu().numpy(), want)


def test_scratch_of_a_longer_list_holds_a_shorter():
    sizes = [2, 16384, 16385, 1 << 20, (1 << 20) + 1, 1 << 21, 1 << 22]
    need = [hs.hs_sort_workspace_bytes(n) for n in sizes]
    assert all(a > 0 for a in need) and need == sorted(need)

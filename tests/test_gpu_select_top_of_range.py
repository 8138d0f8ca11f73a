"""Capped lists whose last entries all lie in the uppermost bin of their keys'
range: crowded last bins of the spectrum, a crowded last row, powers at the top
of the total order.  The uppermost bin ends past 2^64 unless the range starts
at 0.  Exact against numpy."""
import numpy as np
import pytest
import torch

import paper_1805_12258_amd as hs

pytestmark = pytest.mark.gpu

T, N, H = 256, 1 << 16, 4          # word: row << 18 | plane << 16 | bin; rows and bins use all their bits


def ordered(bits):
    """The IEEE total order of fp32 bits as unsigned integers."""
    return np.where(bits >> 31, ~bits, bits | np.uint32(1 << 31))


def expect(word, bits, plane, policy, n_cand):
    at = np.nonzero((word >> 16 & 3) == plane)[0]
    j, r = (word[at] & (N - 1)).astype(np.uint64), (word[at] >> 18).astype(np.uint64)
    if policy == "top":
        at = at[np.lexsort((word[at], ~ordered(bits[at])))][:n_cand]
    else:
        key = j << np.uint64(8) | r if policy == "last_alg2" else r << np.uint64(16) | j
        at = at[np.argsort(key)][-n_cand:]
    return np.stack([word[at], bits[at]], axis=1)


# crowd: entries of plane 0 in the uppermost 64 bins / last row / with the largest NaN's bits; above 2048 the bin
# is split again.
@pytest.mark.parametrize("crowd", [300, 2048, 9000])
@pytest.mark.parametrize("policy", ["last_alg2", "last_alg1", "top"])
def test_cut_in_the_uppermost_bin(policy, crowd):
    rng = np.random.default_rng(crowd)
    r, j = rng.integers(1, T, 30000), rng.integers(N // 4, N, 30000)
    word = r << 18 | rng.integers(0, H, 30000) << 16 | j
    if policy == "last_alg2":      # (bin, row): the uppermost 64 bins hold 16 K words
        c = rng.choice(T * 64, crowd, replace=False)
        edge = (c % T) << 18 | (N - 64 + c // T)
    else:                          # (row, bin): the last row holds 64 K words
        edge = (T - 1) << 18 | rng.choice(N, crowd, replace=False)
    word = np.setdiff1d(np.unique(word), edge)
    word = np.concatenate([word, edge]).astype(np.uint32)
    bits = rng.standard_normal(len(word)).astype(np.float32).view(np.uint32).copy()
    if policy == "top":
        bits[-crowd:] = 0x7FFFFFFF
        bits[:50] = 0xFF800000
    mix = rng.permutation(len(word))
    word, bits = word[mix], bits[mix]
    cand = torch.from_numpy(np.stack([word, bits], axis=1).view(np.int32).copy()).cuda()
    plan = hs.Plan(T, N, H)
    for n_cand in (1, 200):
        kept, counts = plan.select(cand, len(word), n_cand, policy)
        kept, counts = kept.cpu().numpy().view(np.uint32), counts.cpu().tolist()
        for plane in range(H):
            want = expect(word, bits, plane, policy, n_cand)
            assert counts[plane] == len(want)
            assert np.array_equal(kept[plane][:len(want)], want), (policy, plane, n_cand)

"""Workspaces smaller than the size queries give, down to the least that the overlap scan
and the matrix can do with: one sized for one text serves any smaller one, and what
does not fit is refused."""
import sys

import numpy as np
import pytest

from paper_1404_3448_amd import lor, synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def least_overlap(n):   # a summary of 48 bytes for each 16 tiles of 4,096 ranks, and one
    return 256 + 512 + ((n + 65535) // 65536 + 1) * 48 + 1024


def text(k, n, seed):
    rng = np.random.default_rng(seed)
    seqs = [synth.noncoding_like(rng, n + j) for j in range(k)]
    seqs[-1][-700:] = seqs[0][100:800]
    offs = np.concatenate([[0], np.cumsum([s.size for s in seqs])]).astype(np.int64)
    r = lor.longest_overlap_region(torch.from_numpy(np.concatenate(seqs)).cuda(), offs)
    return r["sa"], r["lcp"], offs, r["overlap"]


def scratch(nbytes):
    return torch.empty(nbytes, dtype=torch.uint8, device="cuda")


@pytest.mark.parametrize("n", [70_000, 1_000_000, 8_388_000, 8_500_000])
def test_overlap_scan_in_little_scratch(n):
    """Two texts around 2^24 ranks and smaller ones: the first takes twice the summaries of
    the others with one tile per workgroup."""
    print("scratch, overlap", n, flush=True, file=sys.stderr)
    sa, lcp, offs, want = text(2, n, n)
    N = sa.numel()
    full, least = lor.lor_longest_overlap_workspace(N, 2), least_overlap(N)
    assert least <= full
    for size in (least, (least + full) // 2, full):
        assert lor.lor_longest_overlap(sa, lcp, offs, ws=scratch(size)) == want, size
    with pytest.raises(ValueError):
        lor.lor_longest_overlap(sa, lcp, offs, ws=scratch(least - 1))
    assert want[0] >= 700


def test_matrix_in_little_scratch():
    """26 sequences of 160,000 bases, whose ranks are dropped first where the workspace
    holds what that needs."""
    print("scratch, matrix", flush=True, file=sys.stderr)
    k = 26
    sa, lcp, offs, _ = text(k, 160_000, 26)
    N = sa.numel()
    full = lor.lor_overlap_matrix_workspace(N, k)
    small = lor.lor_overlap_matrix_workspace(3_800_000, k)   # no ranks are dropped there: n x k below 10^8
    assert small < full - N
    want = lor.records_to_tuples(lor.lor_overlap_matrix(sa, lcp, offs))
    for size in (small * N // 3_800_000 + 65536, full - 1, full):
        assert lor.records_to_tuples(lor.lor_overlap_matrix(sa, lcp, offs, ws=scratch(size))) == want, size
    with pytest.raises(ValueError):
        lor.lor_overlap_matrix(sa, lcp, offs, ws=scratch(small // 2))

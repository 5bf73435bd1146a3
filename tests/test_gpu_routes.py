"""Which kernels build a call's suffix array, by the event timing of every
launch, next to the oracle's results: DC3 gives the same array wherever the
prefix sort declines, so results alone do not tell the two apart."""
import sys

import numpy as np
import pytest

import oracle
from paper_1404_3448_amd import lor, synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def say(*a):
    print(*a, flush=True, file=sys.stderr)


def launches(call):
    """(result of `call`, launches of every kernel it made)"""
    try:
        lor.lor_timing_only(None)
        lor.lor_timing_reset()
        lor.lor_timing_enable(True)
        out = call()
        torch.cuda.synchronize()
        return out, {k: v["launches"] for k, v in lor.lor_timing_read().items()}
    finally:
        lor.lor_timing_enable(False)
        lor.lor_timing_reset()


def used_dc3(k):
    return "k_records" in k or "k_sample_keys" in k


def flat(seqs):
    seqs = [np.asarray(s, dtype=np.uint8) for s in seqs]
    offs = np.concatenate([[0], np.cumsum([s.size for s in seqs])]).astype(np.int64)
    cat = np.concatenate(seqs) if offs[-1] else np.zeros(1, np.uint8)
    return cat, torch.from_numpy(np.ascontiguousarray(cat)).cuda(), offs


@pytest.mark.parametrize("n", [(1 << 22) - 1, 1 << 22, (1 << 22) + 1])
def test_one_pair_of_a_batch(n):
    """A batch of one pair on both sides of 2^22 tagged symbols, from where its
    keys hold 16 symbols (32 bits): the prefix sort builds it."""
    say("route, one pair", n)
    rng = np.random.default_rng(n)
    la = n // 2
    a, b = synth.noncoding_like(rng, la), synth.noncoding_like(rng, n - 2 - la)
    b[1000:5000] = a[70_000:74_000]
    a[-40:] = 3
    b[-25:] = 3
    cat, d, offs = flat([a, b])
    (rec, lcp, isa), k = launches(lambda: lor.lor_longest_overlap_batched_state(d, offs))
    assert not used_dc3(k) and "k_resolve" in k, k
    joined = oracle.join(cat, offs)
    sa = oracle.suffix_array(joined)
    want = oracle.lcp(joined, sa)
    assert np.array_equal(lcp.cpu().numpy(), want)
    assert np.array_equal(isa.cpu().numpy(), oracle.isa(sa))
    assert lor.records_to_tuples(rec)[0] == oracle.overlap(sa, want, offs)

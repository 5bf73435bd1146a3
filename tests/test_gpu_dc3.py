"""DC3 on byte texts against the oracle, called as such: it builds the suffix
arrays that the prefix sort leaves to it."""
import os
import subprocess
import sys

import numpy as np
import pytest

import oracle
from paper_1404_3448_amd import lor, synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def say(*a):
    print(*a, flush=True, file=sys.stderr)


def check(seqs):
    seqs = [np.asarray(s, dtype=np.uint8) for s in seqs]
    offs = np.concatenate([[0], np.cumsum([s.size for s in seqs])]).astype(np.int64)
    cat = np.concatenate(seqs) if offs[-1] else np.zeros(1, np.uint8)
    sa, joined = lor.lor_build_sa_dc3(torch.from_numpy(cat).cuda(), offs)
    want = oracle.join(cat[:offs[-1]], offs)
    assert np.array_equal(joined.cpu().numpy(), want)
    got, expect = sa.cpu().numpy(), oracle.suffix_array(want)
    bad = np.flatnonzero(got != expect)
    assert bad.size == 0, (bad.size, bad[:5], got[bad[:5]], expect[bad[:5]])


@pytest.mark.parametrize("seed", [31, 32])
def test_noncoding_text_with_deep_levels(seed):
    """2 x 2^21 noncoding-like bases: deep levels take their order from the parent's."""
    say("dc3 noncoding", seed)
    w = synth.long_text(seed=seed, num_seqs=2, seq_len=1 << 21, num_queries=1)
    check([w.concat[:1 << 21], w.concat[1 << 21:]])


def test_noncoding_pair_8m():
    say("dc3 8M + 8M")
    w = synth.noncoding_pair()
    a = int(w.offsets[1])
    check([w.concat[:a], w.concat[a:]])


@pytest.mark.parametrize("text", ["equal", "period 2", "period 40", "period 171", "identical", "random", "many", "tiny"])
def test_texts(text):
    say("dc3", text)
    rng = np.random.default_rng(11)
    a = synth.gc40_bases(rng, 300_000)
    if text == "equal":
        check([np.zeros(200_001, np.uint8), np.zeros(100_000, np.uint8)])
    elif text.startswith("period"):
        p = int(text.split()[1])
        check([np.resize(a[:p], 250_000), a[:90_000], np.resize(a[:p], 50_001)])
    elif text == "identical":
        check([a, a, a[:1000]])
    elif text == "random":
        check([a])
    elif text == "many":
        check([rng.integers(0, 4, size=int(rng.integers(0, 900)), dtype=np.uint8) for _ in range(251)])
    else:
        for n in range(1, 40):
            check([rng.integers(0, 2, size=n, dtype=np.uint8), rng.integers(0, 4, size=n // 3, dtype=np.uint8)])


_CHILD = """
import sys
sys.path.insert(0, sys.argv[1])
import torch
from paper_1404_3448_amd import lor, synth
w = synth.long_text(seed=31, num_seqs=2, seq_len=1 << 21, num_queries=1)
getattr(lor, sys.argv[2])(torch.from_numpy(w.concat).cuda(), w.offsets)
torch.cuda.synchronize()
"""


@pytest.mark.parametrize("call", ["lor_build_sa", "lor_build_sa_dc3"])
def test_the_trace_does_not_change_what_builds_the_array(call):
    """The notes of a traced call end with those of the code that builds its
    result without the trace."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    say("trace child", call)
    r = subprocess.run([sys.executable, "-c", _CHILD, root, call], env=dict(os.environ, LOR_TRACE="1"),
                       capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    notes = [x for x in r.stderr.splitlines() if x.startswith("[lor]")]
    assert notes and ("prefix sort" in notes[-1]) == (call == "lor_build_sa"), r.stderr[-2000:]
    assert sum("parent-order" in x for x in notes) >= 2, r.stderr[-2000:]

"""Suffix arrays by prefix sorting against the oracle, at the sizes and texts
where its parts meet: key widths (1,024 / 131,072 symbols), workgroup tiles of
2,048 ranks, groups of 63 to 66 equal keys, suffixes near separators, tandem
repeats (large groups, breaking upwards, downwards and at a separator), long
exact repeats (handed to DC3), one text per sequence count, and the batched
and reference texts built on the same sort."""
import sys

import numpy as np
import pytest

import oracle
from paper_1404_3448_amd import lor, synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def say(*a):
    print(*a, flush=True, file=sys.stderr)


def flat(seqs):
    seqs = [np.asarray(s, dtype=np.uint8) for s in seqs]
    offs = np.concatenate([[0], np.cumsum([s.size for s in seqs])]).astype(np.int64)
    cat = np.concatenate(seqs) if offs[-1] else np.zeros(1, np.uint8)
    return cat, torch.from_numpy(np.ascontiguousarray(cat)).cuda(), offs


def check(seqs):
    cat, d, offs = flat(seqs)
    sa, joined = lor.lor_build_sa(d, offs)
    want = oracle.join(cat[:offs[-1]], offs)
    got = sa.cpu().numpy()
    assert np.array_equal(joined.cpu().numpy(), want)
    expect = oracle.suffix_array(want)
    bad = np.flatnonzero(got != expect)
    assert bad.size == 0, (bad.size, bad[:5], got[bad[:5]], expect[bad[:5]])


def tandem(rng, n, units, copies):
    s = synth.gc40_bases(rng, n)
    for u in units:
        u = np.asarray(u, dtype=np.uint8)
        at = int(rng.integers(0, max(1, n - u.size * copies)))
        part = np.tile(u, copies)[:n - at]
        s[at:at + part.size] = part
    return s


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 15, 16, 17, 63, 64, 65, 1021, 1023, 1024, 2045, 2046, 2047, 2048, 2049,
                               4097, 131070, 131073])
def test_sizes(n):
    say("prefix size", n)
    rng = np.random.default_rng(n)
    check([rng.integers(0, 4, size=n - n // 3, dtype=np.uint8), rng.integers(0, 4, size=n // 3, dtype=np.uint8)])


@pytest.mark.parametrize("copies", [2, 31, 62, 63, 64, 65, 66, 130])
def test_group_sizes(copies):
    """One 40-base word planted `copies` times between random bases: groups of
    exactly that many equal keys on both sides of the workgroup's limit, some
    across tile edges."""
    say("prefix groups", copies)
    rng = np.random.default_rng(copies)
    word = rng.integers(0, 4, size=40, dtype=np.uint8)
    parts = []
    for _ in range(copies):
        parts += [rng.integers(0, 4, size=int(rng.integers(20, 90)), dtype=np.uint8), word]
    check([np.concatenate(parts), rng.integers(0, 4, size=500, dtype=np.uint8)])


@pytest.mark.parametrize("seed", range(4))
def test_tandem_repeats(seed):
    """Repeats of period 1 to 20, within and at the ends of sequences, so that
    they break upwards, downwards and at separators."""
    say("prefix tandem", seed)
    rng = np.random.default_rng(seed)
    units = [rng.integers(0, 4, size=p) for p in (1, 2, 2, 3, 5, 6, 7, 11, 12, 13, 17, 20)]
    a = tandem(rng, 60000, units, 150)
    b = tandem(rng, 50001, units[::2], 90)
    ends = [np.tile(np.array(u, np.uint8), 300) for u in ([3], [0], [3, 2], [3, 3, 0])]
    check([a, *ends, b, np.full(200, 3, np.uint8), np.zeros(0, np.uint8), np.full(7, 3, np.uint8)])


@pytest.mark.parametrize("text", ["zeros", "threes", "pairs", "identical", "unit40", "related", "close", "copies"])
def test_repetitive_texts(text):
    """Whole texts of one repeat (DC3 builds these); an identical, a 1%- and a
    0.1%-mutated copy, and 2 to 60 exact copies of 300 to 5,000 bases (runs of
    suffixes that rounds of doubling settle, many across tile edges)."""
    say("prefix repetitive", text)
    rng = np.random.default_rng(5)
    a = synth.gc40_bases(rng, 70000)
    if text == "zeros":
        check([np.zeros(9000, np.uint8), np.zeros(3000, np.uint8)])
    elif text == "threes":
        check([np.full(3000, 3, np.uint8), np.full(2999, 3, np.uint8), np.full(10, 3, np.uint8)])
    elif text == "pairs":
        check([np.tile(np.array([0, 3], np.uint8), 4000), np.tile(np.array([3, 0], np.uint8), 3000)])
    elif text == "identical":
        check([a, a])
    elif text == "close":
        check([a, synth.mutate(rng, a, 0.001), synth.mutate(rng, a[10000:50000], 0.001)])
    elif text == "copies":
        parts = []
        for count, length in ((2, 5000), (3, 2500), (20, 700), (60, 300), (64, 256), (63, 257)):
            word = synth.gc40_bases(rng, length)
            for _ in range(count):
                parts += [word, synth.gc40_bases(rng, int(rng.integers(1, 60)))]
        check([np.concatenate(parts), a[:20000]])
    elif text == "unit40":
        check([np.tile(a[:40], 500), np.tile(a[:40], 77)])
    else:
        check([a, synth.mutate(rng, a, 0.01)])


@pytest.mark.parametrize("k", [1, 2, 3, 100, 251])
def test_sequence_counts(k):
    """Many sequences around the key length, so near suffixes are as many as
    sorted ones, many of them equal up to their separators."""
    say("prefix sequences", k)
    rng = np.random.default_rng(k)
    seqs = [rng.integers(0, 2, size=int(rng.integers(0, 40)), dtype=np.uint8) + 2 for _ in range(k)]
    seqs[0] = rng.integers(0, 4, size=5000, dtype=np.uint8)
    check(seqs)
    check([s[:12] for s in seqs])
    # every sequence ends in one long run: more equal ends than a workgroup resolves
    check([np.concatenate([s[:9], np.full(30, 3, np.uint8)]) for s in seqs])


def test_doubling_above_the_plain_store_limit():
    """More than 2^24 suffixes with exact copies of 3,000 bases: the ranks of
    the doubling rounds come from a bucketed scatter."""
    say("prefix doubling, 17M")
    rng = np.random.default_rng(17)
    a, b = synth.gc40_bases(rng, 9_000_000), synth.gc40_bases(rng, 8_000_001)
    for k in range(40):
        b[k * 100_000:k * 100_000 + 3000] = a[k * 77_777:k * 77_777 + 3000]
    check([a, b])


def test_word_windows_at_every_alignment():
    """joined_out 4 to 60 bytes past a 64-byte boundary."""
    rng = np.random.default_rng(9)
    a = tandem(rng, 30000, [[0, 1], [2, 2, 3]], 100)
    cat, d, offs = flat([a, a[5000:9000]])
    n = int(offs[-1]) + 2
    want = oracle.suffix_array(oracle.join(cat, offs))
    for off in (4, 8, 20, 60):
        buf = torch.zeros(n + 64, dtype=torch.uint8, device="cuda")
        sa, _ = lor.lor_build_sa(d, offs, joined_out=buf[off:off + n])
        assert np.array_equal(sa.cpu().numpy(), want)


def oracle_pair(a, b):
    offs = np.array([0, a.size, a.size + b.size], np.int64)
    joined = oracle.join(np.concatenate([a, b]) if a.size + b.size else np.zeros(0, np.uint8), offs)
    sa = oracle.suffix_array(joined)
    return joined, sa, oracle.lcp(joined, sa), offs


@pytest.mark.parametrize("pairs", [1, 2, 40, 300])
def test_batched_state(pairs):
    """Every pair's own LCP and ISA, which determine its suffix array."""
    say("prefix batched", pairs)
    rng = np.random.default_rng(pairs)
    seqs = []
    for p in range(pairs):
        na, nb = (int(x) for x in rng.integers(0, 3000 if p % 3 else 30, size=2))
        a, b = synth.noncoding_like(rng, na), synth.noncoding_like(rng, nb)
        if p % 5 == 0:
            b[:min(na, nb)] = a[:min(na, nb)]
        if p % 7 == 0:
            a[-50:] = 3
            b[-70:] = 3
        seqs += [a, b]
    cat, d, offs = flat(seqs)
    rec, lcp, isa = lor.lor_longest_overlap_batched_state(d, offs)
    rec, lcp, isa, s = lor.records_to_tuples(rec), lcp.cpu().numpy(), isa.cpu().numpy(), lor.pair_starts(offs)
    for p in range(pairs):
        joined, sa, want, o = oracle_pair(seqs[2 * p], seqs[2 * p + 1])
        assert np.array_equal(lcp[s[p]:s[p + 1]], want), p
        assert np.array_equal(isa[s[p]:s[p + 1]] - s[p], oracle.isa(sa)), p
        assert rec[p] == oracle.overlap(sa, want, o), p


def test_bad_bases_leave_every_access_inside():
    """Bases of every byte value: the call fails with LOR_EALPHABET."""
    rng = np.random.default_rng(3)
    seqs = [rng.integers(0, 256, size=n, dtype=np.uint8) for n in (9000, 5000, 100, 0, 7, 3000)]
    cat, d, offs = flat(seqs)
    for call in (lor.lor_build_sa, lor.lor_longest_overlap_batched, lor.lor_longest_overlap_ref):
        with pytest.raises(lor.LorError) as e:
            call(d, offs)
        assert e.value.status == lor.LOR_EALPHABET


@pytest.mark.parametrize("n", [(1 << 21) - 1, 1 << 21, (1 << 21) + 1])
@pytest.mark.parametrize("copies", ["none", "one", "few", "many"])
def test_open_runs_by_slot_and_by_list(n, copies):
    """Up to 2^21 suffixes, runs of suffixes that are still equal are settled
    slot by slot, above from a list of them: no copies, one of 1,500 bases
    (longer than one comparison, shorter than the second), copies of 9,000
    bases (doubling), and so many that the list is as long as the text."""
    say("prefix open runs", n, copies)
    rng = np.random.default_rng(n)
    la = n // 2
    a, b = synth.gc40_bases(rng, la), synth.gc40_bases(rng, n - 2 - la)   # two separators
    if copies == "one":
        b[5000:6500] = a[777:2277]
    elif copies == "few":
        for k in range(4):
            b[k * 20_000:k * 20_000 + 9000] = a[1234:10_234]
    elif copies == "many":
        b[:] = synth.mutate(rng, a, 0.0004)[:b.size] if la >= b.size else np.resize(a, b.size)
    check([a, b])


@pytest.mark.parametrize("n", [900, 40_000, 1_000_000])
@pytest.mark.parametrize("k", [1, 3])
def test_repeats_at_every_phase(n, k):
    """Tandem repeats of units 1 to 16 (periods up to and beyond half a key)
    that start at every offset of the 32- and 128-position words their extents
    are kept in, end at another repeat, at a separator and at the end, cross
    tiles of 2,048 positions, and run on past the 16,383 symbols that a sort
    key describes; n selects the key width."""
    say("prefix repeats", n, k)
    rng = np.random.default_rng(n + k)
    seqs = []
    for j in range(k):
        parts, size, long = [], 0, n >= 40_000 and j == 0
        while size < n // k:
            unit = rng.integers(0, 4, size=int(rng.integers(1, 17)), dtype=np.uint8)
            copies = 17_000 // unit.size if long else int(rng.integers(3, 40))
            part = np.resize(unit, unit.size * copies + int(rng.integers(0, unit.size + 1)))
            if rng.random() < 0.5:
                parts.append(rng.integers(0, 4, size=int(rng.integers(1, 200)), dtype=np.uint8))
            parts.append(part)
            size += part.size + (parts[-2].size if len(parts) > 1 else 0)
            long = False
        seqs.append(np.concatenate(parts))
    seqs[-1][-60:] = np.resize(np.array([1, 2], np.uint8), 60)
    seqs.append(np.resize(np.array([1, 2], np.uint8), 61))
    check(seqs)


@pytest.mark.parametrize("n,seqs", [((1 << 21) - 1, 2), (1 << 21, 2), ((1 << 21) + 1, 251), ((1 << 21) + 15, 251),
                                    ((1 << 26) + 17, 251)])
def test_lcp_of_packed_text(n, seqs):
    """LCP on both sides of the sizes from which the text is packed for it and
    from which a flag covers 64 window starts; ends at, before and behind a
    multiple of 16; windows that meet separators and the end; copies longer
    than a window."""
    say("lcp packed", n, seqs)
    rng = np.random.default_rng(n)
    cuts = np.sort(rng.choice(np.arange(100, n - seqs - 1), seqs - 1, replace=False))
    cuts[1:4] = cuts[0] + np.array([1, 3, 40])[:cuts[1:4].size]            # sequences of 1, 2 and 37 bases
    cuts = np.sort(cuts)
    cat = rng.integers(0, 4, size=n - seqs, dtype=np.uint8)
    cat[-3000:] = cat[5000:8000]
    offs = np.concatenate([[0], cuts, [cat.size]]).astype(np.int64)
    sa_d, joined_d = lor.lor_build_sa(torch.from_numpy(cat).cuda(), offs)
    lcp_d, isa_d = lor.lor_build_lcp(joined_d, sa_d, want_isa=True)
    lcp2_d, _ = lor.lor_build_lcp(joined_d, sa_d, want_isa=False)
    assert torch.equal(lcp_d, lcp2_d)
    sa, lcp, isa, joined = (x.cpu().numpy() for x in (sa_d, lcp_d, isa_d, joined_d))
    assert joined.size == n and np.array_equal(sa[isa[::977]], np.arange(0, n, 977))
    bad = np.flatnonzero(lcp != oracle.lcp(joined, sa))
    assert bad.size == 0, (bad.size, bad[:5], lcp[bad[:5]])


@pytest.mark.parametrize("aligned", [True, False])
def test_lcp_of_other_bytes(aligned):
    """A text that is not bases: every window is flagged; and one that does not
    start on a word."""
    n = (1 << 21) + 5
    rng = np.random.default_rng(8)
    text = rng.integers(0, 7, size=n, dtype=np.uint8)
    text[-1] = 200
    order = oracle.suffix_array(text)
    buf = torch.zeros(n + 1, dtype=torch.uint8, device="cuda")
    t = buf[:n] if aligned else buf[1:]
    t.copy_(torch.from_numpy(text))
    lcp, _ = lor.lor_build_lcp(t, torch.from_numpy(order.astype(np.int32)).cuda(), want_isa=False)
    assert np.array_equal(lcp.cpu().numpy(), oracle.lcp(text, order))


def test_batched_lcp_of_packed_text():
    """A batch large enough to be packed for its LCP: neighbours of different
    pairs share nothing; pairs of 1 to 400,000 bases."""
    rng = np.random.default_rng(21)
    sizes = [(400_000, 390_001), (1, 1), (5, 300_000), (700_000, 3), (64, 64), (250_000, 249_999), (0, 40), (30, 0)]
    seqs = []
    for a, b in sizes:
        x, y = synth.gc40_bases(rng, a), synth.gc40_bases(rng, b)
        m = min(a, b, 2000) // 2
        y[:m] = x[:m]
        seqs += [x, y]
    cat, d, offs = flat(seqs)
    rec, lcp, isa = lor.lor_longest_overlap_batched_state(d, offs)
    rec, lcp, s = lor.records_to_tuples(rec), lcp.cpu().numpy(), lor.pair_starts(offs)
    for p in range(len(sizes)):
        joined, sa, want, o = oracle_pair(seqs[2 * p], seqs[2 * p + 1])
        assert np.array_equal(lcp[s[p]:s[p + 1]], want), p
        assert rec[p] == oracle.overlap(sa, want, o), p

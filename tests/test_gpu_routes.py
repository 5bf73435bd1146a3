"""Which kernels build a call's suffix array, by the event timing of every
launch, next to the oracle's results: DC3 gives the same array wherever the
prefix sort declines, so results alone do not tell the two apart."""
import sys

import numpy as np
import pytest

import oracle
import test_gpu_prefix as prefix
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


# --------------------------------------------- words with more than 64 copies

POOL = {"k_pool_start", "k_pool_count", "k_pool_collect", "k_pool_ranks", "k_pool_keys"}


def planted(rng, n, words):
    """n random bases with `copies` copies of each (word, copies), none overlapping."""
    parts = [w for w, copies in words for _ in range(copies)]
    rest = n - sum(p.size for p in parts)
    assert rest >= 3 * len(parts)
    order = rng.permutation(len(parts))
    cuts = np.sort(rng.choice(np.arange(1, rest), len(parts), replace=False))
    base = np.split(synth.gc40_bases(rng, rest), cuts)
    out = [base[0]]
    for i, b in zip(order, base[1:]):
        out += [parts[i], b]
    return np.concatenate(out)


def check_sa(seqs):
    cat, d, offs = flat(seqs)
    (sa, joined), k = launches(lambda: lor.lor_build_sa(d, offs))
    expect = oracle.suffix_array(oracle.join(cat[:offs[-1]], offs))
    got = sa.cpu().numpy()
    bad = np.flatnonzero(got != expect)
    assert bad.size == 0, (bad.size, bad[:5], got[bad[:5]], expect[bad[:5]])
    return k


@pytest.mark.parametrize("n", [20_000, 400_000, (1 << 21) - 1, (1 << 21) + 1, (1 << 24) + 3])
def test_words_with_many_copies(n):
    """65 copies of 100 bases are ordered without DC3, slot by slot and from a list,
    with plain and with bucketed ranks; so are longer and more copies next to runs
    that a workgroup holds, tandem repeats, and copies that end at separators."""
    say("route, copies", n)
    rng = np.random.default_rng(n)
    word = rng.integers(0, 4, size=100, dtype=np.uint8)
    k = check_sa([planted(rng, n - n // 4, [(word, 65)]), synth.gc40_bases(rng, n // 4)])
    assert not used_dc3(k) and POOL <= set(k), k
    if n < 100_000:
        return
    words = [(synth.gc40_bases(rng, w), c) for w, c in ((60, 66), (111, 65), (300, 90), (77, 300), (700, 5), (400, 40),
                                                        (1 + n // 100, 3))]
    words += [(np.resize(rng.integers(0, 4, size=p, dtype=np.uint8), 90), 70) for p in (2, 5, 9, 13, 21)]
    seqs = [planted(rng, n // 2, words), planted(rng, n // 4, words[:1]), *[word[:c] for c in (100, 99, 65, 30, 1, 0)]]
    seqs += [np.concatenate([synth.gc40_bases(rng, 20), word]) for _ in range(80)]
    k = check_sa(seqs)
    assert not used_dc3(k) and POOL <= set(k), k


def test_many_equal_sequences():
    """100 equal sequences of 3,000 bases, a third of the text: every suffix of
    theirs is one of 100 that differ at their separators alone."""
    say("route, equal sequences")
    rng = np.random.default_rng(77)
    a = synth.gc40_bases(rng, 3000)
    k = check_sa([*([a] * 100), synth.gc40_bases(rng, 600_000)])
    assert not used_dc3(k) and POOL <= set(k), k


def test_copies_in_pairs_of_a_batch():
    say("route, copies in pairs")
    rng = np.random.default_rng(78)
    seqs = []
    for p in range(6):
        words = [(rng.integers(0, 4, size=120, dtype=np.uint8), 70 + 30 * p)]
        seqs += [planted(rng, 40_000, words), planted(rng, 30_000, words[:p % 2])]
    cat, d, offs = flat(seqs)
    (rec, lcp, isa), k = launches(lambda: lor.lor_longest_overlap_batched_state(d, offs))
    assert not used_dc3(k) and POOL <= set(k), k
    rec, lcp, isa, s = lor.records_to_tuples(rec), lcp.cpu().numpy(), isa.cpu().numpy(), lor.pair_starts(offs)
    for p in range(6):
        o = np.array([0, seqs[2 * p].size, seqs[2 * p].size + seqs[2 * p + 1].size], np.int64)
        joined = oracle.join(np.concatenate(seqs[2 * p:2 * p + 2]), o)
        sa = oracle.suffix_array(joined)
        want = oracle.lcp(joined, sa)
        assert np.array_equal(lcp[s[p]:s[p + 1]], want), p
        assert np.array_equal(isa[s[p]:s[p + 1]] - s[p], oracle.isa(sa)), p
        assert rec[p] == oracle.overlap(sa, want, o), p


@pytest.mark.parametrize("same", [64, 65, 400])
def test_equal_queries(same):
    """Equal queries share their separator too, so their suffixes agree past it."""
    say("route, equal queries", same)
    rng = np.random.default_rng(same)
    ref = synth.noncoding_like(rng, 50_000)
    q = np.concatenate([synth.gc40_bases(rng, 150), ref[1000:1200], synth.gc40_bases(rng, 51)])
    queries = [q if i % 3 == 0 and i < 3 * same else synth.gc40_bases(rng, int(rng.integers(1, 600)))
               for i in range(3 * same + 900)]
    cat, d, offs = flat([ref, *queries])
    rec, k = launches(lambda: lor.lor_longest_overlap_ref(d, offs))
    assert not used_dc3(k) and (same == 64 or POOL <= set(k)), k
    rec = lor.records_to_tuples(rec)
    pick = [0, 3 * (same - 1), *rng.choice(len(queries), 12, replace=False).tolist()]
    for i in pick:
        o = np.array([0, ref.size, ref.size + queries[i].size], np.int64)
        joined = oracle.join(np.concatenate([ref, queries[i]]), o)
        sa = oracle.suffix_array(joined)
        L = oracle.overlap(sa, oracle.lcp(joined, sa), o)[0]
        length, sp, op, sq, oq = rec[i]
        assert (length, sp, sq) == (L, i + 1, 0), (i, rec[i], L)
        assert np.array_equal(queries[i][op:op + L], ref[oq:oq + L]), (i, rec[i])
    assert len({rec[3 * i] [2] for i in range(same)}) == 1


# ------------------------------------------------------------ where DC3 is left

def test_long_periods_are_given_up_in_time():
    """Nearly half of the text is one word of 171 bases over and over: its groups
    are sorted for as long as that costs a part of a DC3 run, which builds the array."""
    say("route, satellite")
    rng = np.random.default_rng(171)
    n = 12_000_000
    a = synth.gc40_bases(rng, n)
    a[:n * 9 // 20] = np.resize(rng.integers(0, 4, size=171, dtype=np.uint8), n * 9 // 20)
    cat, d, offs = flat([a, synth.gc40_bases(rng, 1000)])
    (sa, _), k = launches(lambda: lor.lor_build_sa(d, offs))
    assert used_dc3(k) and k["k_group_keys"] + k.get("k_pool_keys", 0) <= 2, k
    want, _ = lor.lor_build_sa_dc3(d, offs)
    assert torch.equal(sa, want)


def test_long_comparisons_are_given_up():
    """A run of 300,000 equal bases in a reference, whose repeats are found by
    comparing: the budget for that is spent and DC3 builds the array."""
    say("route, budget")
    rng = np.random.default_rng(172)
    queries = [synth.gc40_bases(rng, 600) for _ in range(1000)]
    cat, d, offs = flat([np.zeros(300_000, np.uint8), *queries])
    rec, k = launches(lambda: lor.lor_longest_overlap_ref(d, offs))
    assert used_dc3(k) and k["k_group_keys"] == 1, k
    for i, (length, sp, op, sq, oq) in enumerate(lor.records_to_tuples(rec)):
        z = np.concatenate([[0], (queries[i] == 0).astype(np.int8), [0]])
        starts, ends = np.flatnonzero(np.diff(z) == 1), np.flatnonzero(np.diff(z) == -1)
        runs = ends - starts
        assert (length, sp, sq) == (runs.max(), i + 1, 0) and op == starts[np.argmax(runs)], (i, length)


def test_text_of_one_repeat_is_left_at_once():
    say("route, one repeat")
    cat, d, offs = flat([np.zeros(9000, np.uint8), np.zeros(3000, np.uint8)])
    _, k = launches(lambda: lor.lor_build_sa(d, offs))
    assert used_dc3(k) and "k_group_keys" not in k, k


def test_doubling_is_given_up_in_time():
    """Copies of 35 bases, which doubling tells apart at once, next to copies of 3,000 that
    it does not: it starts, and DC3 builds the array."""
    say("route, doubling given up")
    rng = np.random.default_rng(173)
    words = [(synth.gc40_bases(rng, 35), 1500) for _ in range(40)] + [(synth.gc40_bases(rng, 3000), 1300)]
    cat, d, offs = flat([planted(rng, 12_000_000, words), synth.gc40_bases(rng, 1000)])
    (sa, _), k = launches(lambda: lor.lor_build_sa(d, offs))
    assert used_dc3(k) and 1 <= k["k_pool_keys"] <= 2, k
    want, _ = lor.lor_build_sa_dc3(d, offs)
    assert torch.equal(sa, want)


# ------------------------------------- the prefix sort's own tests take its paths

def check_route(call, with_, without=()):
    _, k = launches(call)
    assert set(with_) <= set(k) and not set(without) & set(k), k
    if "k_records" not in with_:
        assert not used_dc3(k), k


@pytest.mark.parametrize("text,with_", [("zeros", ["k_records"]), ("threes", ["k_records"]), ("pairs", ["k_records"]),
                                        ("unit40", ["k_records"]), ("identical", ["k_double", "k_ranks"]),
                                        ("close", ["k_double", "k_ranks"]), ("copies", ["k_double", "k_group_keys"]),
                                        ("related", ["k_settle"])])
def test_route_of_repetitive_texts(text, with_):
    check_route(lambda: prefix.test_repetitive_texts(text), with_)


@pytest.mark.parametrize("copies", [2, 31, 62, 63, 64, 65, 66, 130])
def test_route_of_group_sizes(copies):
    check_route(lambda: prefix.test_group_sizes(copies), ["k_settle"] if copies <= 64 else ["k_group_keys", *POOL])


def test_route_of_doubling_above_the_plain_store_limit():
    check_route(prefix.test_doubling_above_the_plain_store_limit, ["k_open_list", "k_double", "k_scatter_window"],
                ["k_ranks"])


@pytest.mark.parametrize("n", [(1 << 21) - 1, 1 << 21, (1 << 21) + 1])
@pytest.mark.parametrize("copies", ["none", "one", "few", "many"])
def test_route_of_open_runs(n, copies):
    listed, doubled = n > 1 << 21, copies in ("few", "many")
    check_route(lambda: prefix.test_open_runs_by_slot_and_by_list(n, copies),
                ["k_settle"] + ["k_open_list"] * listed + ["k_double", "k_run_ranks"] * doubled,
                ["k_open_list"] * (not listed) + ["k_double"] * (not doubled))


@pytest.mark.parametrize("k", [1, 3])
def test_route_of_repeats_at_every_phase(k):
    check_route(lambda: prefix.test_repeats_at_every_phase(1_000_000, k), ["k_group_keys", "k_double"])


@pytest.mark.parametrize("pairs", [1, 2, 40, 300])
def test_route_of_batched_state(pairs):
    check_route(lambda: prefix.test_batched_state(pairs), ["k_resolve", "k_settle"])


@pytest.mark.parametrize("n,seqs", [((1 << 21) - 1, 2), (1 << 21, 2), ((1 << 21) + 1, 251)])
def test_route_of_packed_lcp(n, seqs):
    packed = n >= 1 << 21
    check_route(lambda: prefix.test_lcp_of_packed_text(n, seqs), ["k_lcp_packed" if packed else "k_lcp_window"],
                ["k_lcp_window" if packed else "k_lcp_packed"])

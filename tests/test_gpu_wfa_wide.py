"""The workgroup kernel for wide wavefronts (k_wfa_wide) against the wavefront
oracle, bit for bit, where it can go wrong: wavefronts and end diagonals around
the edges of its stages (253, 509, 765, 1021 diagonals each side in the first
window, on to 3069 in steps of 512 in the second) and past the last one, both
parities, exact runs that cross wavefronts, scores only, thresholds beside the
optimum, scratch that holds few pairs' codes, and more pairs than the walks'
queue.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
import synth  # noqa: E402
import paper_2208_01243_amd as aim  # noqa: E402
from gpu_util import compare, describe, run  # noqa: E402

AFF = (0, 4, 6, 2)


@pytest.fixture(scope="module")
def ctx():
    c = aim.Context(0)
    yield c
    c.close()


def _noisy(rng, T, rate):
    b = synth.from_lists([T], [T])
    return synth.mutate(rng, b.txt, b.txt_off, [rate])[0]


def stage_pairs(seed, edges, lo=-4, hi=4):
    """One gap of a length around each edge, to either side, in the middle or at
    an end, between exact or noisy halves; and unrelated pairs whose wavefronts
    pass the edge."""
    rng = np.random.default_rng(seed)
    base = lambda n: rng.integers(0, 4, n).astype(np.uint8)  # noqa: E731
    pats, txts = [], []
    for e in edges:
        for d in range(lo, hi + 1):
            T = base(int(rng.integers(60, 300)))
            at = (0, len(T) // 2, len(T))[int(rng.integers(3))]
            P = np.concatenate([T[:at], base(e + d), T[at:]])
            if d % 3 == 0:
                P = _noisy(rng, P, 0.03)
            pats += [P, T]
            txts += [T, P]
        n = 2 * e
        T = base(n)
        pats += [_noisy(rng, T, 0.12), base(n // 2 + 1)]
        txts += [T, base(n // 2)]
    return synth.from_lists(pats, txts)


def check(ctx, b, pen, max_score=-1, want=None, want_cigar=True):
    want = want or oracle.wfa_batch(b, pen, max_score)
    got = run(ctx, b, "wfa", pen, max_score, want_cigar=want_cigar)
    if not want_cigar:
        assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
        return want
    bad = compare(got, want)
    assert not bad, "%d mismatches, first: %s" % (len(bad), describe(b, bad[0], got, want))
    return want


@pytest.mark.parametrize("pen", [AFF, (0, 1, 0, 1), (0, 3, 4, 1), (0, 30, 2, 1), (0, 1, 40, 1)])
def test_first_window(ctx, pen):
    b = stage_pairs(1, (253, 509, 765, 1021))
    want = check(ctx, b, pen)
    check(ctx, b, pen, want=want, want_cigar=False)


@pytest.mark.parametrize("pen", [AFF, (0, 1, 0, 1), (0, 2, 5, 1)])
def test_second_window(ctx, pen):
    b = stage_pairs(2, (1533, 2045, 2557, 3069), -2, 2)
    want = check(ctx, b, pen)
    check(ctx, b, pen, want=want, want_cigar=False)


def test_thresholds(ctx):
    b = stage_pairs(3, (253, 509), -1, 1)
    full = oracle.wfa_batch(b, AFF)[0]
    for smax in sorted({0, 1, 506, 512, int(full[0]) - 2, int(full[0]) - 1, int(full[0]), int(full[0]) + 1}):
        check(ctx, b, AFF, smax)


def test_long_exact_runs(ctx):
    # exact stretches of thousands of bases on far diagonals: one gap of several
    # hundred bases first
    rng = np.random.default_rng(4)
    pats, txts = [], []
    for k in range(24):
        T = rng.integers(0, 4, 2000 + 37 * k).astype(np.uint8)
        P = np.concatenate([rng.integers(0, 4, 300 + 20 * k).astype(np.uint8), T])
        P[700 + 900 * (k % 2)] ^= 1
        pats.append(P if k % 3 else T)
        txts.append(T if k % 3 else P)
    check(ctx, synth.from_lists(pats, txts), AFF)


@pytest.mark.parametrize("limit", [12 << 20, 40 << 20, 1 << 30])
def test_little_scratch(limit):
    # room for the codes of few pairs, or of none that reaches the last stage
    b = stage_pairs(5, (253, 1021, 2045), -1, 1)
    with aim.Context(0, scratch_limit=limit) as c:
        check(c, b, AFF)


def test_more_pairs_than_await_their_walks(ctx):
    uniq = stage_pairs(6, (100, 253, 300, 509, 1021), -3, 3)
    want = oracle.wfa_batch(uniq, AFF)
    k = np.random.default_rng(7).integers(0, uniq.n, 9000)
    got = run(ctx, uniq.subset(k), "wfa", AFF)
    assert np.array_equal(got[0], want[0][k]) and np.array_equal(got[1], want[1][k])
    assert np.array_equal(np.diff(got[3]), np.diff(want[3])[k])
    for i in range(len(k)):
        assert np.array_equal(got[2][got[3][i]:got[3][i + 1]], want[2][want[3][k[i]]:want[3][k[i] + 1]]), i


@pytest.mark.parametrize("alg", ["wfa", "swg"])
@pytest.mark.parametrize("lmax", [761, 762, 1021, 1100, 3069])
def test_small_batches_start_wide(ctx, alg, lmax):
    # around the length from which a small batch has no group pass, and where a
    # second window follows the first; invalid pairs and thresholds on that route
    rng = np.random.default_rng(lmax)
    T = [rng.integers(0, 4, int(n)).astype(np.uint8) for n in [lmax, lmax, 0, 1] + rng.integers(0, lmax, 40).tolist()]
    P = [rng.integers(0, 4, max(0, len(t) - 3)).astype(np.uint8) if k % 7 == 0 else _noisy(rng, t, 0.05)[:lmax]
         for k, t in enumerate(T)]
    b = synth.from_lists(P, T)
    for smax in (-1, 40):
        want = oracle.wfa_batch(b, AFF, smax)
        got = run(ctx, b, alg, AFF, smax)
        bad = compare(got, want)
        assert not bad, "%d mismatches, first: %s" % (len(bad), describe(b, bad[0], got, want))
    short = run(ctx, b, alg, AFF, max_len=lmax - 1)
    over = np.maximum(b.pat_len, b.txt_len) > lmax - 1
    assert (short[1][over] == aim.PAIR_INVALID).all() and (short[1][~over] == aim.PAIR_ALIGNED).all()


@pytest.mark.parametrize("alg,pen", [("wfa", AFF), ("swg", AFF), ("wfa", (0, 3, 4, 1))])
@pytest.mark.parametrize("lmax", [1021, 1533, 3069])
def test_gap_alone_ends_at_a_stage_edge(ctx, alg, pen, lmax):
    # one side empty (or a base or two) and the other as long as a stage's
    # furthest diagonal: the whole alignment ends, and its walk starts, there
    rng = np.random.default_rng(lmax)
    base = lambda n: rng.integers(0, 4, n).astype(np.uint8)  # noqa: E731
    pats, txts = [], []
    for e in (253, 509, 765, 1021, 1533, 2045, 2557, 3069):
        for n in range(e - 3, e + 4):
            for m in (0, 1, 2):
                if n <= lmax:
                    pats += [base(m), base(n)]
                    txts += [base(n), base(m)]
    b = synth.from_lists(pats, txts)
    for smax in (-1, 6 + 2 * (lmax - 1) if pen == AFF else 4 + lmax - 1):
        want = oracle.wfa_batch(b, pen, smax)
        got = run(ctx, b, alg, pen, smax)
        failed = ctx.last_call_stats()["wfa_walk_failed"]
        bad = compare(got, want)
        assert not bad, "%d mismatches, first: %s" % (len(bad), describe(b, bad[0], got, want))
        assert failed == 0


def length_difference_pairs(seed, diffs, max_len):
    """Pairs that differ by one gap of each length, with a few errors beside it
    or none, and unrelated ones of the same lengths; one pair of max_len bases."""
    rng = np.random.default_rng(seed)
    base = lambda n: rng.integers(0, 4, n).astype(np.uint8)  # noqa: E731
    pats, txts = [base(max_len)], [base(max_len)]
    for d in diffs:
        n = int(rng.integers(0, min(90, max_len - d) + 1))
        T = base(n)
        at = (0, n // 2, n)[int(rng.integers(3))]
        P = np.concatenate([T[:at], base(d), T[at:]])
        for a, b in ((P, T), (T, P), (_noisy(rng, P, 0.02)[:max_len], T), (base(n + d), T)):
            pats.append(a)
            txts.append(b)
    return synth.from_lists(pats, txts)


@pytest.mark.parametrize("alg", ["wfa", "swg"])
@pytest.mark.parametrize("max_len,smax", [(762, 514), (800, 520), (2000, 1000), (2000, 2048), (2000, 2050),
                                          (4095, 3000), (4095, 6144), (4095, 6146)])
def test_thresholds_without_filter(alg, max_len, smax):
    # no pre-alignment filter: the kernel itself rejects pairs whose length
    # difference passes the threshold, also where the end lies outside the last
    # window (1021 or 3069 diagonals) that the threshold leaves in the plan
    reach = smax // 2 - 3
    diffs = sorted({d for e in (253, 509, reach, 1021, 3069, max_len - 2) for d in range(e - 2, e + 3) if 0 < d <= max_len})
    b = length_difference_pairs(max_len + smax, diffs, max_len)
    want = oracle.wfa_batch(b, AFF, smax)
    print("no filter: %s, %d pairs up to %d bp, threshold %d" % (alg, b.n, max_len, smax), flush=True)
    with aim.Context(0, prefilter=False) as c:
        got = run(c, b, alg, AFF, smax)
        bad = compare(got, want)
        assert not bad, "%d mismatches, first: %s" % (len(bad), describe(b, bad[0], got, want))
        got = run(c, b, alg, AFF, smax, want_cigar=False)
        assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])


@pytest.mark.parametrize("pen,wide", [((0, 10, 16, 1), True), ((0, 18, 0, 1), False), ((0, 20, 8, 1), False)])
def test_large_rings(pen, wide):
    # batches that fill the chip take the narrower window where two workgroups'
    # rings fit a CU (x or o + 1 up to 17), else the class kernel; small ones the
    # window, and so do those under a limit that has no room for the later passes
    n, small = 4200, 200
    rng = np.random.default_rng(n + pen[1])
    lens = synth.log_uniform_int(rng, 300, 620, n)
    b = synth._gen_chunk(rng, n, lens, rng.uniform(0.04, 0.1, n), None)
    print("large rings: %s, %d pairs" % (pen, n), flush=True)
    with aim.Context(0) as c:
        got = run(c, b, "wfa", pen)
        window = c.last_call_stats()["wfa_class_window"][0]
        assert (window == 2048) == wide, window
        with aim.Context(0, scratch_limit=64 << 20, hard_limit=True) as hc:
            assert not compare(run(hc, b, "wfa", pen), got)
            assert hc.last_call_stats()["wfa_class_window"][0] == 2048
        part = b.subset(np.arange(small))
        few = run(c, part, "wfa", pen)
        assert c.last_call_stats()["wfa_class_window"][0] == 2048
    assert not compare(few, oracle.wfa_batch(part, pen, -1))
    end = few[3][small]
    assert not compare((got[0][:small], got[1][:small], got[2][:end], got[3][:small + 1]), few)
    some = b.subset(np.arange(small, n, 40))
    want = oracle.wfa_batch(some, pen, -1)
    for t, i in enumerate(range(small, n, 40)):
        assert (got[0][i], got[1][i]) == (want[0][t], want[1][t]), i
        assert np.array_equal(got[2][got[3][i]:got[3][i + 1]], want[2][want[3][t]:want[3][t + 1]]), i

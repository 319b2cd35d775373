"""The group pass of WFA and WFA-adaptive (k_wfa_group: several narrow pairs
per wavefront) against the oracles, bit for bit, where it can go wrong:
lengths around its 16- and 32-base words, end diagonals and gaps around the
edge of its window (61 diagonals each side) and of both parities, drifting
diagonals that move the adaptive window round its lanes, scores only,
thresholds at and beside the optimum, more runs than a slot, invalid pairs,
and rings of codes too small for a pair.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
import synth  # noqa: E402
import paper_2208_01243_amd as aim  # noqa: E402
from gpu_util import compare, describe, run, to_device  # noqa: E402

AFF = (0, 4, 6, 2)


@pytest.fixture(scope="module")
def ctx():
    c = aim.Context(0)
    yield c
    c.close()


def _noisy(rng, T, rate):
    b = synth.from_lists([T], [T])
    return synth.mutate(rng, b.txt, b.txt_off, [rate])[0]


def edge_pairs(seed):
    """Every length from 0 to 70 at a few error rates, one gap of 55-66 bases
    at either side, end, or middle, and unrelated pairs about as long as the
    window is wide."""
    rng = np.random.default_rng(seed)
    base = lambda n: rng.integers(0, 4, n).astype(np.uint8)  # noqa: E731
    pats, txts = [], []

    def add(P, T):
        pats.append(P)
        txts.append(T)
    for n in list(range(71)) + [95, 96, 97, 125, 126, 127, 128, 129, 160]:
        T = base(n)
        for rate in (0.0, 0.03, 0.2):
            add(_noisy(rng, T, rate), T)
    for gap in range(55, 67):
        for at in (0, 40, 90):
            T = base(90)
            P = np.concatenate([T[:at], base(gap), T[at:]])
            add(P, T)
            add(T, P)
            add(_noisy(rng, P, 0.02), T)
    for m in (1, 2, 59, 60, 61, 62, 63, 64, 65, 100):
        for n in (0, 1, 61, 62, 64, 120):
            add(base(m), base(n))
    return synth.from_lists(pats, txts)


def drift_pairs(seed, lo, hi):
    """Pairs whose path wanders over the diagonals: insertions in one stretch,
    deletions in the next, and a long gap now and then."""
    rng = np.random.default_rng(seed)
    pats, txts = [], []
    for _ in range(60):
        T = rng.integers(0, 4, int(rng.integers(lo, hi + 1))).astype(np.uint8)
        out = []
        for k, c in enumerate(T):
            up = (k // max(1, lo // 4)) % 2 == 0
            u = rng.random()
            if u < 0.03:
                if up:
                    out.append(int(rng.integers(0, 4)))
                    out.append(int(c))
            elif u < 0.032:
                out.extend(rng.integers(0, 4, int(rng.integers(5, 25))).tolist())
            else:
                out.append(int(c))
        pats.append(np.array(out, np.uint8))
        txts.append(T)
    return synth.from_lists(pats, txts)


def check(ctx, b, alg, pen, max_score=-1, adaptive=(10, 50), **kw):
    if alg == "wfa_adaptive":
        ctx.wfa_adaptive_params(*adaptive)
        want = oracle.wfa_batch(b, pen, max_score, adaptive=adaptive)
    else:
        want = oracle.align_batch(b, alg, pen, max_score)
    got = run(ctx, b, alg, pen, max_score, **kw)
    if not kw.get("want_cigar", True):
        assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
        return
    bad = compare(got, want)
    assert not bad, "%d mismatches, first: %s" % (len(bad), describe(b, bad[0], got, want))


@pytest.mark.parametrize("pen", [AFF, (0, 1, 0, 1), (0, 3, 4, 1), (0, 1, 3, 1), (0, 30, 2, 1)])
def test_edges(ctx, pen):
    b = edge_pairs(1)
    check(ctx, b, "wfa", pen)
    check(ctx, b, "wfa", pen, want_cigar=False)
    for adaptive in ((10, 50), (2, 3)):
        check(ctx, b, "wfa_adaptive", pen, adaptive=adaptive)
    check(ctx, b, "wfa_adaptive", pen, want_cigar=False)


@pytest.mark.parametrize("alg", ["wfa", "wfa_adaptive"])
def test_thresholds(ctx, alg):
    b = edge_pairs(2)
    for smax in (0, 1, 2, 4, 8, 37, 120, 134, 136, 140):
        check(ctx, b, alg, AFF, smax)


@pytest.mark.parametrize("lo,hi", [(100, 192), (193, 600), (2000, 4000)])
@pytest.mark.parametrize("adaptive", [(10, 50), (10, 20), (30, 100)])
def test_drifting_window(ctx, lo, hi, adaptive):
    check(ctx, drift_pairs(lo + adaptive[1], lo, hi), "wfa_adaptive", AFF, adaptive=adaptive)


def test_more_runs_than_a_slot(ctx):
    rng = np.random.default_rng(5)
    txts = [rng.integers(0, 4, 3000).astype(np.uint8) for _ in range(70)]
    b = synth.from_lists([_noisy(rng, T, 0.08) for T in txts], txts)
    check(ctx, b, "wfa_adaptive", AFF)
    # many runs on few diagonals: mismatches only, within the window
    pats = [T.copy() for T in txts]
    for P in pats:
        P[::50] = (P[::50] + 1) % 4
    b = synth.from_lists(pats, txts)
    got = run(ctx, b, "wfa", (0, 1, 60, 1))
    want = oracle.wfa_batch(b, (0, 1, 60, 1))
    assert not compare(got, want)
    assert (np.diff(got[3]) > 100).all()


@pytest.mark.parametrize("alg", ["wfa", "wfa_adaptive"])
def test_small_code_ring(alg):
    # 24 MiB of scratch for the plans: rings of 512 steps, which 3 kbp pairs at
    # 10 % outgrow
    b = drift_pairs(9, 2500, 3000)
    with aim.Context(0, scratch_limit=24 << 20) as c:
        check(c, b, alg, AFF)


@pytest.mark.parametrize("alg", ["wfa", "wfa_adaptive"])
def test_invalid_and_overflowing_outputs(ctx, alg):
    b = edge_pairs(3)
    dev, enc = to_device(b, "ascii")
    seq = dev[0].clone()
    off = dev[1].cpu().numpy()
    bad = [i for i in range(0, b.n, 7) if b.pat_len[i] > 0]
    for i in bad:
        seq[off[i]] = ord("N")
    dev = (seq,) + tuple(dev[1:])
    ctx.wfa_adaptive_params(10, 50)
    got = run(ctx, b, alg, AFF, dev=(dev, enc))
    want = list(oracle.wfa_batch(b, AFF, -1, adaptive=(10, 50) if alg == "wfa_adaptive" else None))
    assert (got[1][bad] == aim.PAIR_INVALID).all() and (got[0][bad] == -1).all()
    ok = np.setdiff1d(np.arange(b.n), bad)
    assert np.array_equal(got[0][ok], want[0][ok])
    for i in ok:
        assert np.array_equal(got[2][got[3][i]:got[3][i + 1]], want[2][want[3][i]:want[3][i + 1]]), i
    # a cigar buffer that ends inside the batch: whole pairs up to there
    cap = int(want[3][b.n // 2]) + 1
    s, st, cg, off = run(ctx, b, alg, AFF, cigar_cap=cap)
    cut = int(np.searchsorted(want[3], cap, side="right")) - 1
    assert off[-1] == want[3][cut] and np.array_equal(cg[:off[-1]], want[2][:off[-1]])
    late = np.arange(cut, b.n)
    late = late[np.diff(want[3])[late] > 0]
    assert (st[late] == aim.PAIR_CIGAR_OVERFLOW).all()


def test_many_equal_pairs(ctx):
    # every pair ends at score 0: more of them than one walk takes
    rng = np.random.default_rng(8)
    seqs = [rng.integers(0, 4, int(n)).astype(np.uint8) for n in rng.integers(0, 200, 9000)]
    b = synth.from_lists(seqs, seqs)
    for alg in ("wfa", "wfa_adaptive"):
        s, st, cg, off = run(ctx, b, alg, AFF)
        assert not s.any() and not st.any()
        assert np.array_equal(np.diff(off), (b.pat_len > 0).astype(np.int64))
        assert np.array_equal(cg[:off[-1]] >> 4, b.pat_len[b.pat_len > 0].astype(np.uint32))


@pytest.mark.parametrize("alg,pen", [("nw", (0, 1, 0, 1)), ("nw", (0, 2, 0, 1)), ("swg", AFF), ("swg", (0, 1, 1, 1))])
def test_small_band_batches(ctx, alg, pen):
    # NW and SWG batches that take the wavefront passes at once, alone in them
    # (short reads) or with every later pass behind them (longer ones)
    b = edge_pairs(4)
    for smax in (-1, 0, 3, 13, 30, 61):
        check(ctx, b, alg, pen, smax)
    check(ctx, b, alg, pen, want_cigar=False)
    check(ctx, drift_pairs(11, 500, 900), alg, pen)


@pytest.mark.parametrize("alg,pen", [("nw", (0, 1, 0, 1)), ("swg", AFF)])
def test_band_escalates_to_wavefronts(ctx, alg, pen):
    # 66,000 short pairs: the packed band and its second-stream walk, with the
    # pairs it cannot decide (a third of these) in the wavefront passes beside it
    rng = np.random.default_rng(12)
    T = [rng.integers(0, 4, 60).astype(np.uint8) for _ in range(600)]
    uniq = synth.from_lists([_noisy(rng, t, float(rng.choice([0.02, 0.3]))) if k % 3 else
                             rng.integers(0, 4, 60).astype(np.uint8) for k, t in enumerate(T)], T)
    b = uniq.subset(np.arange(66_000) % uniq.n)
    got = run(ctx, b, alg, pen)
    want = oracle.align_batch(uniq, alg, pen)
    assert ctx.last_call_stats()["band_escalated"] > 1000
    k = np.arange(b.n) % uniq.n
    assert np.array_equal(got[0], want[0][k]) and np.array_equal(got[1], want[1][k])
    for i in range(0, b.n, 37):
        assert np.array_equal(got[2][got[3][i]:got[3][i + 1]], want[2][want[3][k[i]]:want[3][k[i] + 1]]), i
    runs = np.diff(want[3])[k]
    assert np.array_equal(np.diff(got[3]), runs)


@pytest.mark.parametrize("alg,pen,unit", [("wfa", AFF, 2), ("wfa_adaptive", AFF, 2), ("swg", AFF, 2), ("nw", (0, 1, 0, 1), 1)])
def test_thresholds_without_filter(alg, pen, unit):
    # no pre-alignment filter: pairs whose length difference passes the threshold
    # reach the passes, at thresholds that end the plan at each of the windows
    # (13, 29, 61, 125 and 253 diagonals each side)
    with aim.Context(0, prefilter=False) as c:
        for reach in (13, 29, 61, 125, 253):
            rng = np.random.default_rng(reach)
            T = [rng.integers(0, 4, int(n)).astype(np.uint8) for n in rng.integers(0, 300, 40)]
            P = []
            for k, t in enumerate(T):
                gap = rng.integers(0, 4, max(0, reach - 3 + k % 7)).astype(np.uint8)
                at = (0, len(t) // 2, len(t))[k % 3]
                P.append(np.concatenate([t[:at], gap, t[at:]]) if k % 8 else rng.integers(0, 4, 3 * reach).astype(np.uint8))
            b = synth.from_lists(P + T, T + P)
            for smax in {unit * (reach + d + pen[2] // unit) for d in (-1, 0, 1)}:
                check(c, b, alg, pen, smax)


@pytest.mark.parametrize("alg,pen,most", [("nw", (0, 1, 0, 1), 1), ("swg", AFF, 2), ("wfa", AFF, 2)])
@pytest.mark.parametrize("n", [300, 1024])
def test_small_batches_take_little_scratch(alg, pen, most, n):
    # a new context's scratch after one small batch: a ring of codes for one pair
    # in each wavefront of the widest pass (four words a lane, a step in 256
    # bytes; a pair of edit distance takes at most its length in scores, a
    # gap-affine one twice that), an eighth more for growth, and 32 MiB for the rest
    rng = np.random.default_rng(n)
    T = [rng.integers(0, 4, 150).astype(np.uint8) for _ in range(n)]
    b = synth.from_lists([_noisy(rng, t, 0.03)[:150] for t in T], T)
    steps = 1 << int(np.ceil(np.log2(most * (150 + 8) + 8)))
    with aim.Context(0) as c:
        run(c, b, alg, pen)
        current, peak = c.scratch_usage()
    assert current == peak <= n * steps * 256 * 9 // 8 + (32 << 20)


@pytest.mark.parametrize("alg,pen,L", [("nw", (0, 1, 0, 1), 150), ("swg", AFF, 100), ("swg", AFF, 150)])
def test_large_band_batch_under_a_hard_limit(alg, pen, L):
    # 70,000 pairs in 64 MiB of scratch: room for the band tiers, but not for the
    # wavefront passes with every later class behind them
    rng = np.random.default_rng(L)
    T = [rng.integers(0, 4, L).astype(np.uint8) for _ in range(500)]
    uniq = synth.from_lists([_noisy(rng, t, float(rng.choice([0.01, 0.15])))[:L] for t in T], T)
    k = np.arange(70_000) % uniq.n
    want = oracle.align_batch(uniq, alg, pen)
    with aim.Context(0, scratch_limit=64 << 20, hard_limit=True) as c:
        got = run(c, uniq.subset(k), alg, pen)
        assert c.last_call_stats()["band_escalated"] > 0
    assert np.array_equal(got[0], want[0][k]) and np.array_equal(got[1], want[1][k])
    assert np.array_equal(np.diff(got[3]), np.diff(want[3])[k])
    for i in range(0, len(k), 41):
        assert np.array_equal(got[2][got[3][i]:got[3][i + 1]], want[2][want[3][k[i]]:want[3][k[i] + 1]]), i


@pytest.mark.parametrize("alg,pen", [("wfa", AFF), ("swg", AFF), ("nw", (0, 1, 0, 1))])
def test_unrelated_pairs_fit_the_pool(alg, pen):
    # 10,000 unrelated pairs of 250 bp: most have 130 to 190 runs where the pool
    # holds 125 a pair beside the slots of 128; none may need the in-place re-run
    rng = np.random.default_rng(21)
    base = lambda n: rng.integers(0, 4, n).astype(np.uint8)  # noqa: E731
    uniq = synth.from_lists([base(int(rng.integers(200, 251))) for _ in range(500)], [base(250) for _ in range(500)])
    k = np.arange(10_000) % uniq.n
    want = oracle.align_batch(uniq, alg, pen)
    with aim.Context(0) as c:
        got = run(c, uniq.subset(k), alg, pen)
        stats = c.last_call_stats()
    assert (np.diff(want[3]) > 128).any() and stats["cigar_reruns"] == 0
    assert np.array_equal(got[0], want[0][k]) and np.array_equal(got[1], want[1][k])
    assert np.array_equal(np.diff(got[3]), np.diff(want[3])[k])
    for i in range(len(k)):
        assert np.array_equal(got[2][got[3][i]:got[3][i + 1]], want[2][want[3][k[i]]:want[3][k[i] + 1]]), i


@pytest.mark.parametrize("lo,hi", [(0, 0), (100, 192), (193, 600), (2000, 3000)])
@pytest.mark.parametrize("adaptive", [(10, 50), (2, 3), (30, 20)])
def test_adaptive_batches_that_start_narrow(ctx, lo, hi, adaptive):
    # more pairs than the chip has wavefronts for: those start in 16 or 32 lanes
    uniq = drift_pairs(lo + adaptive[1], lo, hi) if lo else edge_pairs(6)
    k = np.arange(4200) % uniq.n
    ctx.wfa_adaptive_params(*adaptive)
    want = oracle.wfa_batch(uniq, AFF, -1, adaptive=adaptive)
    got = run(ctx, uniq.subset(k), "wfa_adaptive", AFF)
    assert np.array_equal(got[0], want[0][k]) and np.array_equal(got[1], want[1][k])
    assert np.array_equal(np.diff(got[3]), np.diff(want[3])[k])
    for i in range(len(k)):
        assert np.array_equal(got[2][got[3][i]:got[3][i + 1]], want[2][want[3][k[i]]:want[3][k[i] + 1]]), i

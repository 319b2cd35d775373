"""Packing (8 bases a lane, sequences at any byte offset), length buckets and
the CIGAR compaction's scan against plain numpy and the oracle, at the edges of
their tiles: every length around words and pieces, every byte value, more tiles
than a block adds up itself, and a cap that cuts inside a tile.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
import synth  # noqa: E402
import paper_2208_01243_amd as aim  # noqa: E402
from gpu_util import compare, run  # noqa: E402


@pytest.mark.parametrize("enc", ["ascii", "code"])
@pytest.mark.parametrize("max_len", [40, 100, 300, 700])
def test_pack_bytes(enc, max_len):
    rng = np.random.default_rng(max_len)
    ok = np.frombuffer(b"ACGT", np.uint8) if enc == "ascii" else np.arange(4, dtype=np.uint8)
    lens = np.array(list(range(min(74, max_len))) + [max_len - 1, max_len] * 300, np.int32)
    off = np.concatenate([[0], np.cumsum(lens + 3)]) + 1  # gaps, so that starts take every alignment
    seq = ok[rng.integers(0, 4, int(off[-1]) + 8)]
    for v in range(256):  # each byte value somewhere in a long sequence
        i = 80 + 2 * v
        seq[off[i] + rng.integers(0, lens[i])] = v
    code = np.full(256, 255, np.uint8)
    code[ok] = np.arange(4)
    want_bad = np.zeros(len(lens), np.int8)
    words = []
    for i, n in enumerate(lens):
        c = code[seq[off[i]:off[i] + n]]
        want_bad[i] = (c > 3).any()
        c = np.where(c > 3, 0, c).astype(np.uint64)
        c = np.concatenate([c, np.zeros(-n % 32, np.uint64)]).reshape(-1, 32)
        words.append((c << (2 * np.arange(32, dtype=np.uint64))).sum(axis=1, dtype=np.uint64))
    want = np.concatenate(words)
    dev = [torch.from_numpy(a).cuda() for a in (seq, off[:-1].copy(), lens)]
    out = torch.full((len(want) + 4,), -1, dtype=torch.int64, device="cuda")
    out_off = torch.empty(len(lens) + 1, dtype=torch.int64, device="cuda")
    bad = torch.empty(len(lens), dtype=torch.int8, device="cuda")
    e = aim.ENC_ASCII if enc == "ascii" else aim.ENC_CODE
    with aim.Context(0) as ctx:
        ctx.pack_2bit(e, *dev, out, out_off, bad)
        torch.cuda.synchronize()
        assert np.array_equal(bad.cpu().numpy(), want_bad)
        assert np.array_equal(out.cpu().numpy().view(np.uint64)[:len(want)], want)
        # the same bytes through a batch: both sides, one slot per sequence
        good = np.flatnonzero(want_bad == 0)
        score = torch.empty(len(lens), dtype=torch.int32, device="cuda")
        status = torch.empty(len(lens), dtype=torch.int8, device="cuda")
        ctx.align_batch(dev[0], dev[1], dev[2], dev[0], dev[1], dev[2], enc=e, max_len=max_len, alg="nw",
                        pen=(0, 1, 0, 1), max_score=-1, score=score, status=status, cigar=None, cigar_off=None,
                        want_cigar=False)
        torch.cuda.synchronize()
        st = status.cpu().numpy()
        assert (st[good] == aim.PAIR_ALIGNED).all() and (score.cpu().numpy()[good] == 0).all()
        assert (st[want_bad == 1] == aim.PAIR_INVALID).all()


@pytest.mark.parametrize("alg,n", [("nw", 2_200_000), ("wfa", 130_000), ("wfa", 1025)])
def test_compaction_tiles_and_cut(alg, n):
    rng = np.random.default_rng(n)
    pen = (0, 1, 0, 1) if alg == "nw" else (0, 4, 6, 2)
    T = [rng.integers(0, 4, int(rng.integers(0, 12))).astype(np.uint8) for _ in range(300)]
    P = [rng.integers(0, 4, int(rng.integers(0, 12))).astype(np.uint8) for _ in range(300)]
    uniq = synth.from_lists(P, T)
    k = rng.integers(0, uniq.n, n)
    b = uniq.subset(k)
    ws, wst, wc, wo = oracle.align_batch(uniq, alg, pen)
    runs = np.diff(wo)[k]
    total = int(runs.sum())
    at = np.concatenate([[0], np.cumsum(runs)])
    src = np.repeat(wo[:-1][k] - at[:-1], runs) + np.arange(total)
    with aim.Context(0) as ctx:
        for cap in (total, total // 2 + 1):
            s, st, cg, off = run(ctx, b, alg, pen, cigar_cap=cap)
            fit = int(at[np.searchsorted(at, cap, side="right") - 1])
            assert np.array_equal(s, ws[k])
            assert np.array_equal(off, np.minimum(at, fit))
            assert np.array_equal(cg[:fit], wc[src[:fit]])
            assert np.array_equal(st == aim.PAIR_CIGAR_OVERFLOW, (at[1:] > fit) & (runs > 0))


def test_length_buckets_of_mixed_wavefronts():
    rng = np.random.default_rng(3)
    T = [rng.integers(0, 4, int(n)).astype(np.uint8) for n in np.concatenate([np.full(640, 90), rng.integers(0, 400, 900)])]
    b = synth.from_lists([t[: len(t) - len(t) // 20] for t in T], T)
    with aim.Context(0) as ctx:
        assert not compare(run(ctx, b, "wfa", (0, 4, 6, 2)), oracle.wfa_batch(b, (0, 4, 6, 2)))

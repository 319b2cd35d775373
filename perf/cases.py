"""What this library is used for, as cases that a timing program can run.

Each case is one `Context.align_batch` call on a batch that is already in
device memory, as a read mapper or a comparison pipeline makes it: pairs of a
read and a reference window, gathered by the caller, scores and CIGARs
wanted.  The sizes are those of the repository's own benchmark workloads
(`bench.py`, `synth`): 100, 150 and 250 bp reads, 1 and 10 kbp reads, a
mixed batch of 100-10,000 bp, and the small batches of 100-1,000 bp that the
serving loop forms.

Inputs are made on the GPU from the seed: uniform random texts, and patterns
that are the text with a substitution, an inserted or a deleted base at each
base with the case's error rate.
"""
import math

import torch

import paper_2208_01243_amd as aim

EDIT = (0, 1, 0, 1)     # match, mismatch, gap open, gap extend
AFFINE = (0, 4, 6, 2)


def _case(name, alg, pairs, lmin, lmax, rmin, rmax, max_rate=0.0, unrelated=0.0, enc="2bit", cigar=True):
    c = dict(alg=alg, pairs=pairs, lmin=lmin, lmax=lmax, rmin=rmin, rmax=rmax, max_rate=max_rate,
             unrelated=unrelated, enc=enc, cigar=cigar)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # a small batch of short reads as text, edit distance under a
        # threshold of 5 %: what a filter step of a mapper asks for, bound by
        # the call's latency
        _case("nw_100bp_10k", "nw", 10_000, 100, 100, 0.02, 0.02, max_rate=0.05, enc="ascii"),
        # the bulk case of short-read mapping: a million 150 bp reads
        _case("swg_150bp_1m", "swg", 1_000_000, 150, 150, 0.04, 0.04),
        # 250 bp reads with a fifth of unrelated candidates and a threshold
        _case("wfa_250bp_1m", "wfa", 1_000_000, 250, 250, 0.05, 0.05, max_rate=0.1, unrelated=0.2),
        # reads of every length from short to long in one batch, the largest
        # case (the benchmark's default workload at two fifths of its pairs)
        _case("wfa_mixed_200k", "wfa", 200_000, 100, 10_000, 0.005, 0.1),
        # the heuristic wavefront algorithm at its three usual read lengths
        _case("adaptive_150bp_1m", "wfa_adaptive", 1_000_000, 150, 150, 0.02, 0.02),
        _case("adaptive_1kbp_100k", "wfa_adaptive", 100_000, 1000, 1000, 0.05, 0.05),
        _case("adaptive_10kbp_10k", "wfa_adaptive", 10_000, 10_000, 10_000, 0.05, 0.05),
        # GenASM with k a tenth of the read length
        _case("genasm_150bp_1m", "genasm", 1_000_000, 150, 150, 0.04, 0.04, max_rate=0.1),
        _case("genasm_1kbp_100k", "genasm", 100_000, 1000, 1000, 0.05, 0.05, max_rate=0.1),
        # the device batches that the serving loop forms from its requests:
        # few pairs of 100-1,000 bp as base codes, one per algorithm; the
        # last is a single small request, the smallest call here
        _case("request_nw_2k", "nw", 2048, 100, 1000, 0.01, 0.08, enc="code"),
        _case("request_swg_4k", "swg", 4096, 100, 1000, 0.01, 0.08, enc="code"),
        _case("request_wfa_64", "wfa", 64, 100, 1000, 0.01, 0.08, enc="code"),
    ]


def _cells(c):
    """Wavefront cells of one pair on average: an error costs about 10/3
    steps (mismatch 2, two thirds of the errors a gap of one, 4, after
    division by the penalties' common divisor; one for edit distance), and s
    scores hold about s^2 cells, or, where the heuristic trims them, about 18
    a score."""
    per_error = 1.0 if c["alg"] in ("nw", "genasm") else 10 / 3
    r1 = (c["rmin"] + c["rmax"]) / 2 * per_error
    r2 = (c["rmin"] ** 2 + c["rmin"] * c["rmax"] + c["rmax"] ** 2) / 3 * per_error ** 2
    cells = _mean_power(c["lmin"], c["lmax"], 2) * r2
    if c["alg"] == "wfa_adaptive":
        cells = min(cells, 18 * _mean_power(c["lmin"], c["lmax"], 1) * r1)
    return cells + 1


def _mean_power(a, b, p):
    """Mean of L^p for L log-uniform in [a, b]."""
    if a == b:
        return float(a) ** p
    return (float(b) ** p - float(a) ** p) / (p * math.log(b / a))


def draw(rng):
    def log(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    alg = rng.choice(["nw", "swg", "wfa", "wfa", "wfa_adaptive", "wfa_adaptive", "genasm"])
    lmax = log(80, {"nw": 1500, "swg": 1500, "wfa": 10_000, "wfa_adaptive": 10_000, "genasm": 3000}[alg])
    lmin = lmax if rng.random() < 0.5 else max(50, int(lmax * rng.uniform(0.05, 1.0)))
    lmin = min(lmin, lmax)
    rmax = round(rng.uniform(0.01, 0.1 if alg in ("wfa", "genasm") else 0.08), 4)
    rmin = rmax if rng.random() < 0.5 else round(rmax * rng.uniform(0.1, 1.0), 4)
    limited = alg == "genasm" or rng.random() < 0.4
    c = _case(None, alg, 1, lmin, lmax, rmin, rmax, max_rate=round(rng.uniform(1.2, 2.5) * rmax, 4) if limited else 0.0,
              unrelated=0.2 if limited and alg != "genasm" and rng.random() < 0.5 else 0.0,
              enc=rng.choice(["2bit", "2bit", "code", "ascii"]), cigar=rng.random() < 0.8)
    # at most a fifth of the largest listed case's cells and a million pairs
    most = min(1_000_000, int(1.5e10 / _cells(c)), int(1.5e8 / _mean_power(lmin, lmax, 1)))
    c["pairs"] = log(32, max(64, most)) | 1
    return c


def _repeat(per_pair, lens, total):
    return torch.repeat_interleave(per_pair, lens, output_size=total)


def _pairs(case, seed, dev):
    """(pattern codes, pattern lengths, text codes, text lengths) on `dev`."""
    g = torch.Generator(device=dev).manual_seed(int(seed))
    n = case["pairs"]
    if case["lmin"] == case["lmax"]:
        tl = torch.full((n,), case["lmin"], dtype=torch.int64, device=dev)
    else:
        u = torch.rand(n, generator=g, device=dev, dtype=torch.float64)
        a, b = math.log(case["lmin"]), math.log(case["lmax"] + 1)
        tl = torch.exp(a + u * (b - a)).long().clamp(case["lmin"], case["lmax"])
    rate = case["rmin"] + torch.rand(n, generator=g, device=dev) * (case["rmax"] - case["rmin"])
    alien = torch.rand(n, generator=g, device=dev) < case["unrelated"]
    rate = torch.where(alien, torch.zeros_like(rate), rate)
    total = int(tl.sum())
    txt = torch.randint(0, 4, (total,), generator=g, device=dev, dtype=torch.uint8)
    err = torch.rand(total, generator=g, device=dev) < _repeat(rate, tl, total)
    kind = torch.randint(0, 3, (total,), generator=g, device=dev, dtype=torch.uint8)
    other = torch.randint(0, 4, (total,), generator=g, device=dev, dtype=torch.uint8)
    sub, ins, dele = err & (kind == 0), err & (kind == 1), err & (kind == 2)
    del err, kind
    # a substitution takes one of the three other bases; an insertion puts a
    # random base before the text's own
    step = torch.randint(1, 4, (total,), generator=g, device=dev, dtype=torch.uint8)
    first = torch.where(sub, (txt + step) & 3, txt)
    first = torch.where(_repeat(alien, tl, total), other, first)
    del step, sub
    count = 1 + ins.to(torch.int32) - dele.to(torch.int32)
    end = torch.cumsum(count, 0)
    pat = torch.empty(int(end[-1]), dtype=torch.uint8, device=dev)
    has = torch.nonzero(~dele).squeeze(1)
    pat[end[has] - 1] = first[has]
    two = torch.nonzero(ins).squeeze(1)
    pat[end[two] - 2] = other[two]
    te = torch.cumsum(tl, 0)
    pe = end[te - 1]
    pl = torch.diff(pe, prepend=torch.zeros(1, dtype=pe.dtype, device=dev))
    return pat, pl, txt, tl


def _encode(codes, lens, enc):
    """(sequence array, offsets) of one side in encoding `enc`."""
    starts = torch.cumsum(lens, 0) - lens
    if enc == "code":
        return codes, starts, aim.ENC_CODE
    if enc == "ascii":
        letters = torch.tensor(list(b"ACGT"), dtype=torch.uint8, device=codes.device)
        return letters[codes.int()], starts, aim.ENC_ASCII
    words = (lens + 31) // 32
    woff = torch.cumsum(words, 0) - words
    total = codes.numel()
    slots = torch.zeros(int(words.sum()) * 32, dtype=torch.uint8, device=codes.device)
    at = torch.arange(total, device=codes.device)
    at += _repeat(woff * 32 - starts, lens, total)
    slots[at] = codes
    del at
    q = slots.view(-1, 4)
    packed = q[:, 0] | (q[:, 1] << 2) | (q[:, 2] << 4) | (q[:, 3] << 6)
    return packed.view(torch.int64), woff, aim.ENC_2BIT


def _threshold(case):
    """(penalties, max_score): the case's error threshold in penalty units
    (edits for edit distance and GenASM, the dearest edit otherwise)."""
    pen = EDIT if case["alg"] in ("nw", "genasm") else AFFINE
    if not case["max_rate"]:
        return pen, -1
    edits = max(1, int(case["max_rate"] * case["lmax"]))
    return pen, edits * max(pen[1], pen[2] + pen[3])


class _State:
    pass


def prepare(case, seed):
    """What a mapper holds: a context, the batch and its result arrays."""
    dev = torch.device("cuda")
    pat, pl, txt, tl = _pairs(case, seed, dev)
    st = _State()
    p, po, enc = _encode(pat, pl, case["enc"])
    t, to, _ = _encode(txt, tl, case["enc"])
    st.batch = (p, po, pl.int(), t, to, tl.int())
    pen, max_score = _threshold(case)
    n = case["pairs"]
    z = dict(device=dev, dtype=torch.int32)
    # room for the runs: two per error and one, with slack that a small batch
    # of unequal pairs needs too
    if n < 4096:
        runs = 2 * case["lmax"] * case["rmax"] + 8
    else:
        runs = 1.5 * _mean_power(case["lmin"], case["lmax"], 1) * (case["rmin"] + case["rmax"]) + 8
    cap = int(n * runs) if case["cigar"] else 0
    st.score = torch.zeros(n, **z)
    st.status = torch.zeros(n, device=dev, dtype=torch.int8)
    st.cigar = torch.zeros(cap, **z) if case["cigar"] else None
    st.cigar_off = torch.zeros(n + 1, device=dev, dtype=torch.int64)
    st.args = dict(enc=enc, max_len=int(torch.maximum(pl, tl).max()), alg=case["alg"], pen=pen, max_score=max_score,
                   score=st.score, status=st.status, cigar=st.cigar, cigar_off=st.cigar_off,
                   want_cigar=case["cigar"])
    st.ctx = aim.Context(0)
    return st


def run(st):
    st.ctx.align_batch(*st.batch, **st.args)
    out = {"score": st.score, "status": st.status, "cigar_off": st.cigar_off}
    if st.cigar is not None:
        out["cigar"] = st.cigar
    return out


def work(case):
    """Bytes: the bases at the encoding's width, offsets and lengths read;
    scores, statuses, offsets and the CIGAR runs (two per error and one)
    written.  Operations: 18 integer operations per wavefront cell (8 for
    the recurrences, 10 for its extension word), the fewest cells an exact
    gap-affine alignment is known to need; for GenASM, 14 per status-vector
    update."""
    n = case["pairs"]
    mean = _mean_power(case["lmin"], case["lmax"], 1)
    rate = (case["rmin"] + case["rmax"]) / 2
    per_base = 0.25 if case["enc"] == "2bit" else 1.0
    related = 1.0 - case["unrelated"]
    byts = n * (2 * mean * per_base + 24 + 5 + 8)
    if case["cigar"]:
        byts += n * related * 4 * (2 * mean * rate + 1)
    if case["alg"] == "genasm":
        flops = 14 * n * mean / 40 * 64 * (64 * rate + 1)
    else:
        flops = 18 * n * related * _cells(case)
    return {"bytes": float(byts), "flops": float(flops)}


def _padded(codes, lens, width, fill):
    n, total = lens.numel(), codes.numel()
    out = torch.full((n, width), fill, dtype=torch.uint8, device=codes.device)
    row = _repeat(torch.arange(n, device=codes.device), lens, total)
    col = torch.arange(total, device=codes.device) - _repeat(torch.cumsum(lens, 0) - lens, lens, total)
    out[row, col] = codes
    return out


def exact(case, seed):
    """Optimal scores and the statuses that follow from them, by the textbook
    affine recurrence over anti-diagonals, all pairs at once in 64-bit
    integers; CIGARs and their offsets have no value here, nor do the
    heuristic algorithms' scores."""
    if case["alg"] in ("wfa_adaptive", "genasm"):
        return None
    if case["pairs"] * (case["lmax"] * 1.1 + 10) ** 2 > 3.2e10 or case["lmax"] > 2000:
        return None
    dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    pat, pl, txt, tl = _pairs(case, seed, dev)
    pen, max_score = _threshold(case)
    _, x, o, e = pen
    score = torch.empty(case["pairs"], dtype=torch.int64, device=dev)
    ps, ts = torch.cumsum(pl, 0) - pl, torch.cumsum(tl, 0) - tl
    block = max(1, int(1e8 / (case["lmax"] * 1.1 + 10)))
    for a in range(0, case["pairs"], block):
        b = min(case["pairs"], a + block)
        p1 = int(ps[b - 1] + pl[b - 1])
        t1 = int(ts[b - 1] + tl[b - 1])
        score[a:b] = _gotoh(pat[int(ps[a]):p1], pl[a:b], txt[int(ts[a]):t1], tl[a:b], x, o, e)
    rejected = (score > max_score) if max_score >= 0 else torch.zeros_like(score, dtype=torch.bool)
    out = {"score": torch.where(rejected, -1, score).int(), "status": rejected.to(torch.int8), "cigar_off": None}
    if case["cigar"]:
        out["cigar"] = None
    return out


def _gotoh(pat, pl, txt, tl, x, o, e):
    """H(m, n) of every pair; column i of each array is the cell (i, d - i)."""
    n, lp, lt = pl.numel(), int(pl.max()), int(tl.max())
    dev = pat.device
    big = 1 << 40
    P = torch.cat([torch.full((n, 1), 4, dtype=torch.uint8, device=dev), _padded(pat, pl, lp, 4)], 1)
    # T flipped between two margins: cell (i, d - i) compares P[i] with
    # column lt - d + i + lp + 1 of it
    margin = torch.full((n, lp + 1), 5, dtype=torch.uint8, device=dev)
    T = torch.cat([margin, _padded(txt, tl, lt, 5).flip(1), margin, margin], 1)
    h1 = torch.full((n, lp + 1), big, dtype=torch.int64, device=dev)
    h1[:, 0] = 0
    h2 = torch.full_like(h1, big)
    E, F = torch.full_like(h1, big), torch.full_like(h1, big)
    want, out = pl + tl, torch.zeros(n, dtype=torch.int64, device=dev)
    wide = torch.full((n, 1), big, dtype=torch.int64, device=dev)
    rows = torch.arange(n, device=dev)

    def down(v):  # the value of the cell above
        return torch.cat([wide, v[:, :-1]], 1)

    for d in range(1, lp + lt + 1):
        E = torch.minimum(h1 + o, E) + e
        F = down(torch.minimum(h1 + o, F)) + e
        at = lt - d + lp + 1
        miss = (P != T[:, at:at + lp + 1]).to(torch.int64) * x
        h = torch.minimum(torch.minimum(E, F), down(h2) + miss)
        h2, h1 = h1, h
        done = want == d
        if bool(done.any()):
            out[done] = h[rows[done], pl[done]]
    return out

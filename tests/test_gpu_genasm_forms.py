"""GenASM's kept differences (k_genasm) against the GenASM oracle: a wavefront
keeps slices of 21 bits while none of its windows has a distance above 10, of 32
bits up to 15, whole vectors above, and walks on after another pass where a
window needs more positions than are kept.  Batches whose pairs all sit at one
of these edges, by substitutions or by gaps that drift as far as the distance
allows, with windows shorter than, as long as and longer than what is kept.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
import synth  # noqa: E402
import paper_2208_01243_amd as aim  # noqa: E402
from gpu_util import compare, describe, run  # noqa: E402

EDIT = (0, 1, 0, 1)


def edited(rng, n, d):
    """A pair of about n bases, d edits in each stretch of 64."""
    T = rng.integers(0, 4, n).astype(np.uint8)
    P = T.copy()
    kind = int(rng.integers(4))
    if kind == 0 or n < 64:
        for s in range(0, n, 64):
            at = s + rng.choice(min(64, n - s), size=min(d, n - s), replace=False)
            P[at] = (P[at] + 1) % 4
    elif kind == 1:  # one gap of d bases: d diagonals away for the rest
        at = int(rng.integers(0, n))
        P = np.concatenate([T[:at], rng.integers(0, 4, d).astype(np.uint8), T[at:]])
    elif kind == 2:
        at = int(rng.integers(0, max(1, n - d)))
        P = np.concatenate([T[:at], T[at + d:]])
    else:  # there and back
        at = int(rng.integers(0, max(1, n // 2)))
        h = d // 2
        P = np.concatenate([T[:at], rng.integers(0, 4, h).astype(np.uint8), T[at:at + 25], T[at + 25 + h:]])
    return P, T


@pytest.mark.parametrize("d", [0, 1, 9, 10, 11, 14, 15, 16, 25, 50])
def test_distance_edges(d):
    rng = np.random.default_rng(100 + d)
    with aim.Context(0) as ctx:
        for n in (12, 39, 40, 41, 63, 64, 65, 79, 80, 104, 105, 150, 400):
            pairs = [edited(rng, n, d) for _ in range(130)]
            b = synth.from_lists([p for p, _ in pairs], [t for _, t in pairs])
            got, want = run(ctx, b, "genasm", EDIT), oracle.genasm_batch(b)
            bad = compare(got, want)
            assert not bad, "n %d: %d mismatches, first: %s" % (n, len(bad), describe(b, bad[0], got, want))
            s, st = run(ctx, b, "genasm", EDIT, want_cigar=False)[:2]
            assert np.array_equal(s, want[0]) and np.array_equal(st, want[1])

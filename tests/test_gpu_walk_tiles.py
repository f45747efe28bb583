"""Paths are walked in tiles of their record (32 rows by 32 steps, 64 by 64
for boxes above 512 rows).  Boxes whose rows and columns end at, before and
after a tile's edge, and paths that leave a tile upwards, to the left, in long
gaps and in many short runs, equal the oracle's."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2208_12350_amd import workloads as W

pytestmark = pytest.mark.gpu


def _check(pairs, scheme):
    from paper_2208_12350_amd.binding import Aligner, DeviceBatch
    b = W.from_pairs(pairs, [0] * len(pairs), [scheme])
    al = Aligner(0)
    try:
        out, off, cig, ln = (t.cpu().numpy() for t in al.align_cigar(DeviceBatch.from_host(b)))
    finally:
        al.close()
    _, oruns, ooff, onr = O.cigar_batch(b, index=np.arange(b.n_pairs))
    for i in range(b.n_pairs):
        got = cig.view(np.uint32)[off[i]:off[i] + ln[i]]
        assert np.array_equal(got, oruns[ooff[i]:ooff[i] + onr[i]]), (i, b.q_len()[i], b.r_len()[i])


@pytest.mark.parametrize("alphabet", [4, 20])
@pytest.mark.parametrize("gap", [0, 1, 40, 150])
def test_tiles(alphabet, gap):
    rng = np.random.default_rng(10 * alphabet + gap)
    M = np.full((alphabet, alphabet), -3, dtype=np.int8)
    np.fill_diagonal(M, 5)
    pairs = []
    for n in (1, 15, 16, 17, 31, 32, 33, 48, 63, 64, 65, 96, 97, 192, 193, 256, 320, 511, 512, 513, 768, 1000, 1500):
        for cut in (0, 1, 2):
            s = rng.integers(0, alphabet, size=n).astype(np.uint8)
            t = s.copy()
            flip = rng.random(n) < 0.05
            t[flip] = rng.integers(0, alphabet, size=int(flip.sum()))
            ins = rng.integers(0, alphabet, size=gap).astype(np.uint8)
            at = n // 2
            if cut == 0:
                t = np.concatenate([t[:at], ins, t[at:]])          # gap in the query
            elif cut == 1:
                s = np.concatenate([s[:at], ins, s[at:]])          # gap in the reference
            else:                                                  # many short gaps
                t = np.delete(t, np.arange(5, n, 23))
            pairs.append((s[:2048], t))
    _check(pairs, W.Scheme(np.ascontiguousarray(M), 4, 0 if gap > 1 else 1, "tiles"))

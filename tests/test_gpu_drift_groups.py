"""Column-word schemes of several gap extension costs in one call: beside another
scheme that needs the pair table each cost has its own drift, so every small
alphabet keeps its column words and the pair table stays.  Work items that hold
pairs of several costs give every pair the result it has alone, scores and paths."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2208_12350_amd import workloads as W

pytestmark = pytest.mark.gpu

FIELDS = ("score", "q_start", "q_end", "r_start", "r_end")


def _batch(rng, schemes, n, hi):
    pairs, sids = [], []
    for _ in range(n):
        s = int(rng.integers(0, len(schemes)))
        A = schemes[s].alphabet
        q = rng.integers(0, A, size=int(rng.integers(1, hi))).astype(np.uint8)
        r = rng.integers(0, A, size=int(rng.integers(1, 2 * hi))).astype(np.uint8)
        k = min(q.size, r.size)
        at = int(rng.integers(0, r.size - k + 1))
        r[at:at + k] = q[:k]
        flip = rng.random(r.size) < 0.15
        r[flip] = rng.integers(0, A, size=int(flip.sum()))
        pairs.append((q, r))
        sids.append(s)
    return W.from_pairs(pairs, sids, schemes)


DNA = [W.dna_scheme(), W.dna_scheme(gap_open=8, gap_extend=2), W.dna_scheme(match=2, gap_open=9),
       W.dna_scheme(gap_open=5, gap_extend=5), W.dna_scheme(gap_open=24, gap_extend=23)]


@pytest.mark.parametrize("schemes", [[DNA[0], DNA[1], W.protein_scheme(5)], [DNA[1], W.protein_scheme(5), DNA[0], DNA[3]],
                                     [DNA[0], DNA[1], DNA[3]], [DNA[3], DNA[0], DNA[1], DNA[4]],
                                     [DNA[0], DNA[1], DNA[2], W.protein_scheme(5)]])
@pytest.mark.parametrize("hi,options", [(60, {}), (400, {}), (400, {"families": 0}), (400, {"mode": 0}),
                                        (400, {"chunk": 64}), (2048, {})])
def test_every_small_alphabet_keeps_its_column_words(schemes, hi, options):
    from paper_2208_12350_amd.binding import Aligner, DeviceBatch
    rng = np.random.default_rng(hi + len(schemes))
    b = _batch(rng, schemes, 500 if hi > 100 else 3000, hi)
    want = O.align_batch(b)
    al = Aligner(0, **options)
    try:
        d = DeviceBatch.from_host(b)
        got = al.align(d).cpu().numpy()
        bins = al.bin_stats()
        for i in np.flatnonzero((got != np.stack([want[f] for f in FIELDS], axis=1)).any(axis=1)):
            raise AssertionError((i, b.scheme_id[i], got[i], want[i]))
        small = np.array([s.alphabet <= 4 for s in schemes])[b.scheme_id]
        taken = {c: sum(s["pairs"] for s in bins if s["pass"] == 0 and s["column"] == c and s["precision"] == 16)
                 for c in (0, 1, 2)}
        assert taken == {0: 0, 1: int(small.sum()), 2: int((~small).sum())}
        out, off, cig, ln = (t.cpu().numpy() for t in al.align_cigar(d))
        assert np.array_equal(out, got)
    finally:
        al.close()
    idx = np.arange(0, b.n_pairs, 3)
    _, oruns, ooff, onr = O.cigar_batch(b, index=idx)
    for k, i in enumerate(idx):
        assert np.array_equal(cig.view(np.uint32)[off[i]:off[i] + ln[i]], oruns[ooff[k]:ooff[k] + onr[k]]), i

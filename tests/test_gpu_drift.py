"""GPU parity of the drifted sweeps (column words, pair table, query profile)
where they can go wrong: every renormalisation period of the drift and the
gap costs at its limits, references across several periods, and tied best
scores without room for the row code, which send pairs to the redo list."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2208_12350_amd import workloads as W

pytestmark = pytest.mark.gpu

FIELDS = ("score", "q_start", "q_end", "r_start", "r_end")


def _oracle_rows(batch):
    o = O.align_batch(batch)
    return np.stack([o[f] for f in FIELDS], axis=1).astype(np.int64)


def _run(batch, **options):
    from paper_2208_12350_amd.binding import Aligner, DeviceBatch
    al = Aligner(0, **options)
    try:
        out = al.align(DeviceBatch.from_host(batch)).cpu().numpy().astype(np.int64)
        stats, bins = al.stats(), al.bin_stats()
    finally:
        al.close()
    return out, stats, bins


def _related(rng, A, n, m):
    q = rng.integers(0, A, size=n).astype(np.uint8)
    r = rng.integers(0, A, size=m).astype(np.uint8)
    mut = q.copy()
    flip = rng.random(n) < 0.15
    mut[flip] = rng.integers(0, A, size=int(flip.sum()))
    if m > n:
        at = int(rng.integers(0, m - n + 1))
        r[at:at + n] = mut
        if n > 8 and rng.random() < 0.5:   # a gap in the middle
            r = np.delete(r, np.arange(at + n // 2, at + n // 2 + 3))
    return q, r


# (gap open, gap extend): periods 128, 64, 32, 16, 8, and beyond the drifted
# sweeps (tables); linear gaps; no extension cost; gap opens whose scores do
# not fit a byte (tables)
@pytest.mark.parametrize("o,e", [(6, 1), (6, 6), (10, 10), (15, 14), (20, 19), (24, 23), (30, 25), (40, 40), (5, 0),
                                 (862, 1), (863, 1), (1024, 0)])
@pytest.mark.parametrize("alphabet", [4, 20])
def test_gap_costs_and_periods(o, e, alphabet):
    rng = np.random.default_rng(1000 * o + e + alphabet)
    M = np.full((alphabet, alphabet), -3, dtype=np.int8)
    np.fill_diagonal(M, 4)
    sc = W.Scheme(np.ascontiguousarray(M), o, e, "g")
    pairs = [_related(rng, alphabet, int(rng.integers(1, 300)), int(rng.integers(1, 700))) for _ in range(300)]
    pairs += [_related(rng, alphabet, n, m) for n in (1, 16, 17, 255, 256, 257, 512, 700)
              for m in (1, 63, 127, 128, 129, 255, 257, 640)]
    b = W.from_pairs(pairs, [0] * len(pairs), [sc])
    got, _, _ = _run(b)
    assert np.array_equal(got, _oracle_rows(b))


@pytest.mark.parametrize("alphabet", [4, 20])
@pytest.mark.parametrize("families", [1, 0])
def test_ties_without_row_code(alphabet, families):
    """Low-complexity sequences tie the best score over many cells; a residue
    that never occurs scores so high that the score bound leaves no room for
    the row code, so the end column can come out too small and the pair must
    be redone.  Results and statistics equal the table-lookup sweeps'."""
    rng = np.random.default_rng(77 + alphabet)
    M = np.full((alphabet, alphabet), -1, dtype=np.int8)
    np.fill_diagonal(M, 1)
    M[alphabet - 1, alphabet - 1] = 120
    sc = W.Scheme(np.ascontiguousarray(M), 2, 1, "ties")
    pairs = []
    for k in range(1500):
        n = int(rng.integers(1, 250)) if k % 5 else int(rng.integers(250, 700))
        m = int(rng.integers(1, 2 * n + 60))
        letters = 2 if k % 2 else 3
        pairs.append((rng.integers(0, letters, size=n).astype(np.uint8),
                      rng.integers(0, letters, size=m).astype(np.uint8)))
    b = W.from_pairs(pairs, [0] * len(pairs), [sc])
    want = _oracle_rows(b)
    got, stats, bins = _run(b, families=families)
    assert np.array_equal(got, want)
    assert any(e["column"] == (1 if alphabet == 4 else 2) and e["pairs"] > 0 for e in bins)
    assert sum(e["cells"] for e in bins if e["pass"] == 1) == stats[1]
    ref, ref_stats, _ = _run(b, families=families, colpath=0, pairtable=0)
    assert np.array_equal(ref, want)
    assert stats == ref_stats


def test_column_schemes_of_two_extension_costs():
    """One drift per launch: a second small-alphabet scheme with another gap
    extension cost takes the pair table beside the first one's column words."""
    rng = np.random.default_rng(5)
    schemes = [W.dna_scheme(), W.dna_scheme(gap_open=8, gap_extend=3), W.dna_scheme(match=2, gap_open=9)]
    pairs = [_related(rng, 4, int(rng.integers(1, 400)), int(rng.integers(1, 600))) for _ in range(900)]
    sids = [int(s) for s in rng.integers(0, 3, size=len(pairs))]
    b = W.from_pairs(pairs, sids, schemes)
    got, _, bins = _run(b)
    assert np.array_equal(got, _oracle_rows(b))
    for column, schemes_of in ((1, (0, 2)), (2, (1,))):
        assert sum(e["pairs"] for e in bins if e["pass"] == 0 and e["lanes"] <= 64 and e["column"] == column) <= \
            sum(s in schemes_of for s in sids)
        assert any(e["column"] == column and e["pairs"] > 0 for e in bins)


def test_search_ties_without_row_code():
    """The same ties through the query profile of a database search."""
    import torch
    from paper_2208_12350_amd.binding import Aligner
    rng = np.random.default_rng(9)
    M = np.full((20, 20), -1, dtype=np.int8)
    np.fill_diagonal(M, 1)
    M[19, 19] = 120
    sc = W.Scheme(np.ascontiguousarray(M), 2, 1, "ties")
    query = rng.integers(0, 2, size=300).astype(np.uint8)
    query[150] = 19   # the bound counts it, no reference holds it
    lens = rng.integers(1, 500, size=800)
    off = np.zeros(lens.size + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    refs = rng.integers(0, 2, size=int(off[-1])).astype(np.uint8)
    for bound in (True, False):   # without and with the row code
        q = query.copy()
        if not bound:
            q[150] = 0
        al = Aligner(0)
        try:
            got = al.search(torch.from_numpy(q).cuda(), torch.from_numpy(refs).cuda(), torch.from_numpy(off).cuda(),
                            sc).cpu().numpy().astype(np.int64)
            assert al.get_option("qprofile_used") == 1
        finally:
            al.close()
        s = W.SearchSet(q, refs, off, sc)
        assert np.array_equal(got, _oracle_rows(s.as_batch()))

"""Above 512 rows the built-in routing also depends on the score source: in calls
of 4097 to 8192 pairs, queries of 769 to 1024 residues take cooperative groups
with column words and 64-lane groups otherwise, beside one another in one call.
Every pair has its own result, and installed tables hold for both sources."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2208_12350_amd import workloads as W

pytestmark = pytest.mark.gpu

FIELDS = ("score", "q_start", "q_end", "r_start", "r_end")


def _batch(n, rows, schemes, seed):
    rng = np.random.default_rng(seed)
    ql = np.resize(rows, n)
    rl = rng.integers(10, 30, n)
    qo, ro = (np.concatenate([[0], np.cumsum(x)]).astype(np.int64) for x in (ql, rl))
    return W.Batch(rng.integers(0, 4, qo[-1]).astype(np.uint8), qo, rng.integers(0, 4, ro[-1]).astype(np.uint8), ro,
                   (np.arange(n) // len(rows) % len(schemes)).astype(np.uint8), schemes, "sources", seed)


def _lanes(al, column, lo, hi):
    return {s["lanes"] for s in al.bin_stats() if s["pass"] == 0 and s["precision"] == 16 and s["pairs"] and
            (s["column"] == 1) == column and lo < s["lanes"] * s["rows"] <= hi}


@pytest.mark.parametrize("n,rows,column,other", [(4096, (600, 768), {256}, {256}), (4100, (600, 768), {64}, {64}),
                                                 (8192, (769, 900, 1024), {256}, {64}), (4096, (769, 1024), {256}, {256}),
                                                 (8192, (1025, 2048), {256}, {256}), (8193, (769, 1024), {64}, {64})])
def test_shape_of_each_source(n, rows, column, other):
    from paper_2208_12350_amd.binding import Aligner, DeviceBatch
    dna, prot = W.dna_scheme(), W.protein_scheme(5)
    hi = 2048 if rows[-1] > 1024 else 1024
    al = Aligner(0)
    try:
        for schemes in ([dna], [prot], [dna, prot], [prot, W.protein_scheme(6), dna]):
            b = _batch(n, rows, schemes, n + len(schemes))
            got = al.align(DeviceBatch.from_host(b)).cpu().numpy()
            idx = np.arange(0, n, 7)
            o = O.align_batch(b, index=idx)
            assert np.array_equal(got[idx], np.stack([o[f] for f in FIELDS], axis=1))
            if schemes[0] is dna or schemes[-1] is dna:
                assert _lanes(al, True, 512, hi) == column, schemes
            if schemes[0] is not dna or len(schemes) > 1:
                assert _lanes(al, False, 512, hi) == other, schemes
        al.set_routing(16, [(512, 32, 16), (2048, 64, 32)])
        b = _batch(n, rows, [dna, prot], 3)
        assert np.array_equal(al.align(DeviceBatch.from_host(b)).cpu().numpy()[::7],
                              np.stack([O.align_batch(b, index=np.arange(0, n, 7))[f] for f in FIELDS], axis=1))
        assert _lanes(al, True, 512, 2048) == _lanes(al, False, 512, 2048) == {64}
    finally:
        al.close()


@pytest.mark.parametrize("n,lanes", [(4096, {256}), (6144, {256}), (6145, {64})])
def test_search_of_a_long_query(n, lanes):
    """Searches keep to cooperative groups for longer than batches."""
    import torch
    from paper_2208_12350_amd.binding import Aligner
    rng = np.random.default_rng(n)
    sc = W.protein_scheme(5)
    query = rng.integers(0, 20, 1000).astype(np.uint8)
    off = np.concatenate([[0], np.cumsum(rng.integers(1, 30, n))]).astype(np.int64)
    refs = rng.integers(0, 20, off[-1]).astype(np.uint8)
    al = Aligner(0)
    try:
        got = al.search(torch.from_numpy(query).cuda(), torch.from_numpy(refs).cuda(), torch.from_numpy(off).cuda(),
                        sc).cpu().numpy()
        assert _lanes(al, False, 512, 1024) == lanes
    finally:
        al.close()
    idx = np.arange(0, n, 11)
    o = O.align_batch(W.SearchSet(query, refs, off, sc).as_batch(), index=idx)
    assert np.array_equal(got[idx], np.stack([o[f] for f in FIELDS], axis=1))

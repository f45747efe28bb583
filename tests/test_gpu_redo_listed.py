"""Pairs whose end column a drifted forward sweep leaves open go to the redo
list.  Every pair here is built to be one: two words of the query, a few rows
apart in one lane, match the reference once each, the lower one in an earlier
column, and nothing else matches.  A residue that fills the rest of the query,
and that no reference holds, scores so high that the sweep cannot carry the row
beside the score; where it scores nothing the same pairs are settled at once."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2208_12350_amd import workloads as W

pytestmark = pytest.mark.gpu

FIELDS = ("score", "q_start", "q_end", "r_start", "r_end")


def _scheme(alphabet, high):
    M = np.full((alphabet, alphabet), -1, dtype=np.int8)
    np.fill_diagonal(M, 1)
    M[alphabet - 1, alphabet - 1] = high
    return W.Scheme(np.ascontiguousarray(M), 2, 1, "listed")


def _query(rng, alphabet, n, R, word):
    """Words 0..0 and 1..1 that end in the first row of a lane and `word` rows below."""
    q = np.full(n, alphabet - 1, np.uint8)
    end = int(rng.integers(1, (n - word - 1) // R + 1)) * R
    if end < word:
        end += R
    q[end - word + 1:end + 1] = 0
    q[end + 1:end + 1 + word] = 1
    return q


def _ref(rng, alphabet, m, word):
    """1..1 somewhere in the first half, 0..0 in the second."""
    r = np.full(m, alphabet - 2, np.uint8)
    a, b = int(rng.integers(0, m // 2 - word)), int(rng.integers(m // 2, m - word))
    r[a:a + word] = 1
    r[b:b + word] = 0
    return r


def _rows(batch):
    o = O.align_batch(batch)
    return np.stack([o[f] for f in FIELDS], axis=1)


# one shape of every kind of sweep: rows per lane up to 8, 16 and 32, and groups of a workgroup
SHAPES = [(16, 9), (16, 16), (32, 8), (32, 16), (64, 6), (64, 16), (64, 20), (64, 32), (256, 3), (256, 4), (256, 5),
          (256, 8)]


@pytest.mark.parametrize("alphabet", [4, 20])
@pytest.mark.parametrize("lanes,rows", SHAPES)
def test_every_pair_is_listed(alphabet, lanes, rows):
    from paper_2208_12350_amd.binding import Aligner, DeviceBatch
    rng = np.random.default_rng(1000 * lanes + rows + alphabet)
    hi = lanes * rows // 16 * 16
    pairs = []
    for _ in range(37):
        n = int(rng.integers(max(133, hi // 2), hi + 1))
        pairs.append((_query(rng, alphabet, n, rows, 2 if rows < 5 else 4), _ref(rng, alphabet, 254, 2 if rows < 5 else 4)))
    al = Aligner(0, tuning="route16=%dx%d@%d" % (lanes, rows, hi) + ("" if hi == 2048 else "/256x8@2048"))
    try:
        for high, listed in ((120, len(pairs)), (0, 0)):
            b = W.from_pairs(pairs, [0] * len(pairs), [_scheme(alphabet, high)])
            got = al.align(DeviceBatch.from_host(b)).cpu().numpy()
            assert np.array_equal(got, _rows(b))
            assert al.get_option("redo_pairs") == listed
            stats = al.stats()
            plain = Aligner(0, tuning="route16=%dx%d@%d" % (lanes, rows, hi) + ("" if hi == 2048 else "/256x8@2048"),
                            colpath=0, pairtable=0)
            try:
                assert np.array_equal(plain.align(DeviceBatch.from_host(b)).cpu().numpy(), got)
                assert plain.get_option("redo_pairs") == 0 and plain.stats() == stats
            finally:
                plain.close()
    finally:
        al.close()


@pytest.mark.parametrize("lanes,rows", [(16, 9), (16, 16), (32, 16), (64, 6), (64, 16), (64, 32)])
def test_every_reference_of_a_search_is_listed(lanes, rows):
    import torch
    from paper_2208_12350_amd.binding import Aligner
    rng = np.random.default_rng(lanes + rows)
    hi = lanes * rows // 16 * 16
    refs = [_ref(rng, 20, int(rng.integers(60, 255)), 4) for _ in range(53)]
    off = np.concatenate([[0], np.cumsum([r.size for r in refs])]).astype(np.int64)
    q = _query(rng, 20, hi, rows, 4)
    al = Aligner(0, tuning="route16=%dx%d@%d" % (lanes, rows, hi) + ("" if hi == 2048 else "/256x8@2048"))
    try:
        for high, listed in ((120, len(refs)), (0, 0)):
            sc = _scheme(20, high)
            got = al.search(torch.from_numpy(q).cuda(), torch.from_numpy(np.concatenate(refs)).cuda(),
                            torch.from_numpy(off).cuda(), sc).cpu().numpy()
            assert al.get_option("qprofile_used") == 1
            assert np.array_equal(got, _rows(W.from_pairs([(q, r) for r in refs], [0] * len(refs), [sc])))
            assert al.get_option("redo_pairs") == listed
    finally:
        al.close()

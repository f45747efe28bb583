"""Redone pairs are searched by the sweeps of their own score source: calls whose
listed pairs mix column words of several gap extension costs and the pair table,
of few and many rows, in neighbouring places of the list.  Each pair is built to be
listed (see test_gpu_redo_listed.py)."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2208_12350_amd import workloads as W

pytestmark = pytest.mark.gpu

FIELDS = ("score", "q_start", "q_end", "r_start", "r_end")


def _scheme(alphabet, gap_open, gap_extend):
    M = np.full((alphabet, alphabet), -1, dtype=np.int8)
    np.fill_diagonal(M, 1)
    M[alphabet - 1, alphabet - 1] = 120
    return W.Scheme(np.ascontiguousarray(M), gap_open, gap_extend, "listed")


@pytest.mark.parametrize("m", [64, 254])
@pytest.mark.parametrize("schemes", [[(4, 2, 1), (20, 2, 1)], [(4, 2, 1), (4, 9, 2), (20, 7, 3)],
                                     [(4, 2, 1), (4, 9, 2), (4, 5, 5), (20, 11, 1)], [(4, 2, 1), (4, 9, 2), (4, 5, 5)]])
def test_lists_of_several_sources(schemes, m):
    from paper_2208_12350_amd.binding import Aligner, DeviceBatch
    rng = np.random.default_rng(m + len(schemes))
    schemes = [_scheme(*s) for s in schemes]
    pairs, sids = [], []
    for k in range(401):
        s = int(rng.integers(0, len(schemes)))
        A = schemes[s].alphabet
        n = int(rng.choice([250, 256, 257, 500, 512, 513, 900, 1024, 1025, 2048]))
        word = 4
        # the first row of a lane in every shape the table below routes to
        end = 128 * int(rng.integers(1, (n - word - 1) // 128 + 1))
        q = np.full(n, A - 1, np.uint8)
        q[end - word + 1:end + 1] = 0
        q[end + 1:end + 1 + word] = 1
        r = np.full(m, A - 2, np.uint8)
        a, b = int(rng.integers(0, m // 2 - word)), int(rng.integers(m // 2, m - word))
        r[a:a + word] = 1
        r[b:b + word] = 0
        pairs.append((q, r))
        sids.append(s)
    b = W.from_pairs(pairs, sids, schemes)
    o = O.align_batch(b)
    want = np.stack([o[f] for f in FIELDS], axis=1)
    al = Aligner(0, tuning="route16=16x16@256/32x16@512/64x16@1024/64x32@2048")
    try:
        for _ in range(2):
            got = al.align(DeviceBatch.from_host(b)).cpu().numpy()
            assert np.array_equal(got, want)
            assert al.get_option("redo_pairs") == len(pairs)
    finally:
        al.close()


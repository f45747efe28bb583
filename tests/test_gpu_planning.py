"""Planning of a pass: pairs are ranked within their length bucket per
workgroup, one pair a thread up to 65536 pairs and two above.  Batches on both
sides of that line, with every pair in one bucket and with pairs spread over
many, empty pairs among them, give every pair the result it has alone."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2208_12350_amd import workloads as W

pytestmark = pytest.mark.gpu

FIELDS = ("score", "q_start", "q_end", "r_start", "r_end")


def _tiled(base, n):
    """n pairs that repeat the pairs of `base`."""
    k = len(base)
    ql = np.array([base[i % k][0].size for i in range(n)])
    rl = np.array([base[i % k][1].size for i in range(n)])
    qo = np.concatenate([[0], np.cumsum(ql)]).astype(np.int64)
    ro = np.concatenate([[0], np.cumsum(rl)]).astype(np.int64)
    q = np.concatenate([p[0] for p in base])
    r = np.concatenate([p[1] for p in base])
    return W.Batch(np.resize(q, qo[-1]).astype(np.uint8), qo, np.resize(r, ro[-1]).astype(np.uint8), ro,
                   np.zeros(n, np.uint8), [W.dna_scheme()], "tiled", 0)


@pytest.mark.parametrize("n", [1, 255, 257, 65536, 65537, 70001])
@pytest.mark.parametrize("spread", [False, True])
def test_every_pair_keeps_its_result(n, spread):
    from paper_2208_12350_amd.binding import Aligner, DeviceBatch
    rng = np.random.default_rng(n + spread)
    if spread:
        base = [(rng.integers(0, 4, size=int(rng.integers(0, 90))).astype(np.uint8),
                 rng.integers(0, 4, size=int(rng.integers(0, 400))).astype(np.uint8)) for _ in range(211)]
    else:
        base = [(rng.integers(0, 4, size=30).astype(np.uint8), rng.integers(0, 4, size=40).astype(np.uint8))
                for _ in range(211)]
    o = O.align_batch(W.from_pairs(base, [0] * len(base), [W.dna_scheme()]))
    want = np.resize(np.stack([o[f] for f in FIELDS], axis=1), (n, 5))
    al = Aligner(0)
    try:
        d = DeviceBatch.from_host(_tiled(base, n))
        for _ in range(2):                          # captured, then replayed
            assert np.array_equal(al.align(d).cpu().numpy(), want)
        out, off, cig, ln = (t.cpu().numpy() for t in al.align_cigar(d))
        assert np.array_equal(out, want)
        k = min(n, len(base))
        runs = [cig[off[i]:off[i] + ln[i]].tolist() for i in range(k)]
        for i in range(k, n, max(1, n // 5000)):
            assert cig[off[i]:off[i] + ln[i]].tolist() == runs[i % len(base)], i
    finally:
        al.close()

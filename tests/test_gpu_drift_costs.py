"""Gap costs that the drifted sweeps take in shapes of up to 16 rows per lane only:
column words and the pair table are used where the routing has no taller shape, in
calls of every size, and paths come from byte tables.  Costs on both sides of each
limit, long queries and an installed table of tall shapes among them."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2208_12350_amd import workloads as W

pytestmark = pytest.mark.gpu

FIELDS = ("score", "q_start", "q_end", "r_start", "r_end")
# (open, extend, drifted under the built-in routing, under any): o + 26 e <= 1024, 5 e - o <= 127, o + 42 e <= 1024
COSTS = [(23, 23, True, True), (24, 24, True, False), (30, 30, True, False), (31, 31, True, False), (32, 32, False, False),
         (100, 35, True, False), (100, 36, False, False), (60, 37, True, False), (62, 37, True, False), (63, 37, False, False)]


def _pairs(rng, A, lens):
    out = []
    for n, m in lens:
        q = rng.integers(0, A, size=n).astype(np.uint8)
        r = rng.integers(0, A, size=m).astype(np.uint8)
        k = min(n, m)
        at = int(rng.integers(0, m - k + 1))
        r[at:at + k] = q[:k]
        flip = rng.random(m) < 0.1
        r[flip] = rng.integers(0, A, size=int(flip.sum()))
        out.append((q, np.delete(r, np.arange(m // 3, m // 3 + 2)) if m > 40 else r))
    return out


@pytest.mark.parametrize("o,e,builtin,tall", COSTS)
@pytest.mark.parametrize("alphabet", [4, 20])
def test_costs_at_the_limits(alphabet, o, e, builtin, tall):
    from paper_2208_12350_amd.binding import Aligner, DeviceBatch
    rng = np.random.default_rng(100 * o + e + alphabet)
    M = np.full((alphabet, alphabet), -20, dtype=np.int8)
    np.fill_diagonal(M, 14)
    sc = W.Scheme(np.ascontiguousarray(M), o, e, "costs")
    lens = [(n, m) for n in (1, 16, 17, 255, 256, 512, 513, 800, 1024, 1025, 2048) for m in (3, 129, 600)]
    lens += [(int(rng.integers(1, 300)), int(rng.integers(1, 700))) for _ in range(300)]
    lens += [(2048, 2300)] * 3                                   # scores near the packed range's end
    b = W.from_pairs(_pairs(rng, alphabet, lens), [0] * len(lens), [sc])
    want = O.align_batch(b)
    want = np.stack([want[f] for f in FIELDS], axis=1)
    column = 1 if alphabet == 4 else 2
    for tuning, drifted in ((None, builtin), ("route16=16x16@256/32x16@512/64x32@2048", tall)):
        al = Aligner(0, tuning=tuning)
        try:
            d = DeviceBatch.from_host(b)
            assert np.array_equal(al.align(d).cpu().numpy(), want)
            taken = {s["column"] for s in al.bin_stats() if s["pairs"] and s["precision"] == 16}
            assert taken == {column if drifted else 0}
            out, off, cig, ln = (t.cpu().numpy() for t in al.align_cigar(d))
        finally:
            al.close()
        assert np.array_equal(out, want)
        idx = np.arange(0, b.n_pairs, 5)
        _, oruns, ooff, onr = O.cigar_batch(b, index=idx)
        for k, i in enumerate(idx):
            assert np.array_equal(cig.view(np.uint32)[off[i]:off[i] + ln[i]], oruns[ooff[k]:ooff[k] + onr[k]]), i


@pytest.mark.parametrize("alphabet", [4, 20])
def test_largest_calls_use_no_tall_shape(alphabet):
    from paper_2208_12350_amd.binding import Aligner, DeviceBatch
    rng = np.random.default_rng(alphabet)
    M = np.full((alphabet, alphabet), -20, dtype=np.int8)
    np.fill_diagonal(M, 14)
    sc = W.Scheme(np.ascontiguousarray(M), 30, 30, "costs")
    n = 262200
    ql = rng.integers(1, 6, n)
    ql[:2100] = rng.integers(1025, 2049, 2100)                   # more than are few
    rl = rng.integers(1, 8, n)
    rl[:2100] = 30
    qo, ro = (np.concatenate([[0], np.cumsum(x)]).astype(np.int64) for x in (ql, rl))
    b = W.Batch(rng.integers(0, alphabet, qo[-1]).astype(np.uint8), qo, rng.integers(0, alphabet, ro[-1]).astype(np.uint8), ro,
                np.zeros(n, np.uint8), [sc], "costs", 0)
    al = Aligner(0)
    try:
        got = al.align(DeviceBatch.from_host(b)).cpu().numpy()
        bins = [s for s in al.bin_stats() if s["pairs"] and s["precision"] == 16]
    finally:
        al.close()
    assert max(s["rows"] for s in bins) <= 16 and {s["column"] for s in bins} == {1 if alphabet == 4 else 2}
    idx = np.concatenate([np.arange(0, 2100, 3), np.arange(2100, n, 37)])
    o = O.align_batch(b, index=idx)
    assert np.array_equal(got[idx], np.stack([o[f] for f in FIELDS], axis=1))

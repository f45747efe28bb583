"""GPU parity of the drifted sweeps in cooperative groups, where a workgroup's
four wavefronts hand their edges on in blocks of columns: every row count,
renormalisation periods down to below a block, references that end within a
wavefront's first blocks, and queries that leave whole wavefronts empty."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2208_12350_amd import workloads as W

pytestmark = pytest.mark.gpu

FIELDS = ("score", "q_start", "q_end", "r_start", "r_end")


@pytest.mark.parametrize("rows", [3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("alphabet,o,e", [(4, 6, 1), (4, 24, 23), (4, 30, 25), (20, 11, 1), (20, 30, 25)])
def test_coop_groups_match_oracle(rows, alphabet, o, e):
    from paper_2208_12350_amd.binding import Aligner, DeviceBatch
    rng = np.random.default_rng(100 * rows + o + e)
    M = np.full((alphabet, alphabet), -3, dtype=np.int8)
    np.fill_diagonal(M, 4)
    sc = W.Scheme(np.ascontiguousarray(M), o, e, "coop")
    pairs = []
    for n, m in [(1, 1), (63, 2), (64 * rows, 31), (64 * rows + 1, 32), (128 * rows, 33), (128 * rows + 1, 95),
                 (192 * rows, 96), (192 * rows + 1, 97), (256 * rows, 128), (256 * rows - 1, 129),
                 (256 * rows, 1000)] + [(int(rng.integers(1, 256 * rows + 1)), int(rng.integers(1, 600)))
                                        for _ in range(20)]:
        q = rng.integers(0, alphabet, size=n).astype(np.uint8)
        r = rng.integers(0, alphabet, size=m).astype(np.uint8)
        at = int(rng.integers(0, max(n - m, 0) + 1))
        k = min(n, m)
        r[:k] = q[at:at + k]                        # a long match across the wavefronts' edges
        flip = rng.random(m) < 0.1
        r[flip] = rng.integers(0, alphabet, size=int(flip.sum()))
        pairs.append((q, r))
    b = W.from_pairs(pairs, [0] * len(pairs), [sc])
    route = "route16=256x%d@%d" % (rows, 256 * rows) + ("" if rows == 8 else "/256x8@2048")
    al = Aligner(0, tuning=route)
    try:
        got = al.align(DeviceBatch.from_host(b)).cpu().numpy().astype(np.int64)
        lanes = {s["lanes"] for s in al.bin_stats() if s["pairs"] and s["precision"] == 16}
    finally:
        al.close()
    want = O.align_batch(b)
    np.testing.assert_array_equal(got, np.stack([want[f] for f in FIELDS], axis=1).astype(np.int64))
    assert lanes == {256}

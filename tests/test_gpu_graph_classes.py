"""A set of buffers has one captured graph for each size class that its calls
fall into.  Two sets used across every class, in turn, replay what was captured
the first time, and each replay gives the pairs' own results."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2208_12350_amd import workloads as W

pytestmark = pytest.mark.gpu

FIELDS = ("score", "q_start", "q_end", "r_start", "r_end")
SIZES = (4096, 4097, 8192, 8193, 262144, 262145)


def _tiled(base, n):
    k = len(base)
    ql, rl = (np.resize([p[c].size for p in base], n) for c in (0, 1))
    qo, ro = (np.concatenate([[0], np.cumsum(x)]).astype(np.int64) for x in (ql, rl))
    q, r = (np.resize(np.concatenate([p[c] for p in base]), off[-1]).astype(np.uint8) for c, off in ((0, qo), (1, ro)))
    return W.Batch(q, qo, r, ro, np.zeros(n, np.uint8), [W.dna_scheme()], "tiled", k)


def test_two_sets_of_buffers_in_every_class():
    import torch
    from paper_2208_12350_amd.binding import Aligner, DeviceBatch
    al = Aligner(0, capacity=max(SIZES))
    sets = []
    for seed in (1, 2):
        rng = np.random.default_rng(seed)
        base = [tuple(rng.integers(0, 4, size=int(x)).astype(np.uint8) for x in rng.integers(1, 40, size=2))
                for _ in range(101)]
        o = O.align_batch(W.from_pairs(base, [0] * len(base), [W.dna_scheme()]))
        want = np.resize(np.stack([o[f] for f in FIELDS], axis=1), (max(SIZES), 5))
        d = DeviceBatch.from_host(_tiled(base, max(SIZES)))
        sets.append((d, torch.empty((max(SIZES), 5), dtype=torch.int32, device="cuda:0"), want))
    try:
        for rep in range(3):
            for n in SIZES:
                for d, out, want in sets:
                    view = DeviceBatch(d.queries, d.q_off[:n + 1], d.refs, d.r_off[:n + 1], d.scheme_id[:n], d.schemes)
                    out.fill_(-7)
                    got = al.align(view, out=out[:n]).cpu().numpy()
                    assert np.array_equal(got, want[:n]), (rep, n)
                    assert int(out[n:].max()) == -7 if n < max(SIZES) else True
            assert al.get_option("captures") == 2 * 4, rep
    finally:
        al.close()

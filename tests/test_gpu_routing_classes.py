"""The built-in int16 routing differs by the size of a call: one handle runs
calls on both sides of every limit in turn, replayed graphs included, and each
gives what a fixed routing table gives.  The shapes it picks cover the queries
it sends them, an installed table is used for calls of every size, and
restoring the built-in table brings the choice by size back."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2208_12350_amd import workloads as W

pytestmark = pytest.mark.gpu

FIELDS = ("score", "q_start", "q_end", "r_start", "r_end")
LONG = [128, 129, 256, 257, 384, 385, 511, 512, 513, 700, 768, 769, 1024, 1025, 1300, 2048]


def _batch(n, scheme, alphabet, seed):
    """n pairs: queries at the edges of the routed ranges, the rest short."""
    rng = np.random.default_rng(seed)
    ql = rng.integers(1, 12, size=n)
    k = min(n, len(LONG))
    ql[:k] = LONG[:k]
    rl = rng.integers(1, 16, size=n)
    rl[:k] = rng.integers(1, 300, size=k)
    qo = np.concatenate([[0], np.cumsum(ql)]).astype(np.int64)
    ro = np.concatenate([[0], np.cumsum(rl)]).astype(np.int64)
    return W.Batch(rng.integers(0, alphabet, size=int(qo[-1])).astype(np.uint8), qo,
                   rng.integers(0, alphabet, size=int(ro[-1])).astype(np.uint8), ro,
                   np.zeros(n, np.uint8), [scheme], "classes", seed)


@pytest.mark.parametrize("alphabet", [4, 20])
def test_calls_on_both_sides_of_each_class(alphabet):
    from paper_2208_12350_amd.binding import Aligner, DeviceBatch
    sc = W.dna_scheme() if alphabet == 4 else W.protein_scheme(5)
    al, fixed = Aligner(0), Aligner(0, tuning="route16=16x8@128/32x16@512/64x32@2048")
    try:
        sizes = [1, 17, 4096, 4097, 8192, 8193, 262144, 262145]
        batches = {n: DeviceBatch.from_host(_batch(n, sc, alphabet, n)) for n in sizes}
        want = {n: fixed.align(d).cpu().numpy() for n, d in batches.items()}
        for n in sizes + sizes[::-1]:               # the second round replays captured graphs
            assert np.array_equal(al.align(batches[n]).cpu().numpy(), want[n]), n
        o = O.align_batch(_batch(4096, sc, alphabet, 4096))
        assert np.array_equal(want[4096], np.stack([o[f] for f in FIELDS], axis=1))
    finally:
        al.close()
        fixed.close()


def test_installed_table_holds_for_every_size():
    from paper_2208_12350_amd.binding import Aligner, DeviceBatch
    sc = W.dna_scheme()
    al = Aligner(0)

    def shapes(n):
        al.align(DeviceBatch.from_host(_batch(n, sc, 4, n)))
        return {(s["lanes"], s["rows"]) for s in al.bin_stats() if s["pass"] == 0 and s["pairs"] and s["precision"] == 16}
    try:
        builtin = al.routing(16)
        by_size = {n: shapes(n) for n in (4096, 8192, 8193, 262145)}
        assert len({frozenset(s) for s in by_size.values()}) == 4
        al.set_routing(16, builtin)                 # installed, so used for every size
        assert al.routing(16) == builtin
        assert len({frozenset(shapes(n)) for n in by_size}) == 1
        al.set_routing(16, [])
        assert al.routing(16) == builtin
        assert {n: shapes(n) for n in by_size} == by_size
    finally:
        al.close()

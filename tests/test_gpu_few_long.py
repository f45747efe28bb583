"""Long queries that the built-in routing sends to 64-lane groups are swept by
cooperative groups when a pass has few of them, whatever the size of the call.
Calls with few and with many, at the limit and one above, give every pair its own
result, in every way of launching the sweeps."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2208_12350_amd import workloads as W

pytestmark = pytest.mark.gpu

FIELDS = ("score", "q_start", "q_end", "r_start", "r_end")
LIMIT = 2048
ROWS = (513, 576, 577, 700, 768, 769, 1000, 1024)       # (queries up to 1024 go to 64 lanes above 8192 pairs)


def _batch(n_long, schemes, alphabet, seed, n_short=8300, rows=ROWS):
    """n_short pairs of a few residues, and n_long long queries against references of 30 or so."""
    rng = np.random.default_rng(seed)
    ql = np.concatenate([rng.integers(1, 6, n_short), np.resize(rows, n_long)])
    rl = np.concatenate([rng.integers(1, 6, n_short), rng.integers(20, 40, n_long)])
    perm = rng.permutation(ql.size)
    ql, rl = ql[perm], rl[perm]
    qo, ro = (np.concatenate([[0], np.cumsum(x)]).astype(np.int64) for x in (ql, rl))
    return W.Batch(rng.integers(0, alphabet, qo[-1]).astype(np.uint8), qo, rng.integers(0, alphabet, ro[-1]).astype(np.uint8),
                   ro, rng.integers(0, len(schemes), ql.size).astype(np.uint8), schemes, "few long", seed)


def _want(b):
    o = O.align_batch(b)
    return np.stack([o[f] for f in FIELDS], axis=1)


@pytest.mark.parametrize("options", [{}, {"families": 0}, {"mode": 0}, {"chunk": 64}, {"graph": 0, "timing": 2}])
@pytest.mark.parametrize("source", ["column", "pair table", "table", "mixed"])
def test_few_and_many(source, options):
    from paper_2208_12350_amd.binding import Aligner, DeviceBatch
    dna, prot = W.dna_scheme(), W.protein_scheme(5)
    schemes = {"column": [dna], "pair table": [prot], "table": [prot, W.protein_scheme(6)], "mixed": [dna, prot]}[source]
    al = Aligner(0, **options)
    try:
        for n_long in (1, 2, 333, LIMIT, LIMIT + 1, 0):
            b = _batch(n_long, schemes, 4 if schemes[0] is dna else 20, n_long)
            d = DeviceBatch.from_host(b)
            want = _want(b)
            for _ in range(2):
                assert np.array_equal(al.align(d).cpu().numpy(), want), n_long
            if source != "mixed" and not options:
                hi = {s["family_hi"] for s in al.bin_stats()
                      if s["pass"] == 0 and s["precision"] == 16 and s["lanes"] == 64 and s["rows"] > 8 and s["pairs"]}
                assert hi == ({8} if 0 < n_long <= LIMIT else {20} if n_long else set()), n_long
    finally:
        al.close()


@pytest.mark.parametrize("alphabet", [4, 20])
def test_among_many_short_pairs(alphabet):
    """Above 262144 pairs every long query goes to 64 lanes; one graph serves few and many."""
    import torch
    from paper_2208_12350_amd.binding import Aligner, DeviceBatch
    sc = W.dna_scheme() if alphabet == 4 else W.protein_scheme(5)
    rows = ROWS + (1025, 1280, 1281, 1536, 1537, 1792, 1793, 2048)
    few = _batch(32, [sc], alphabet, 7, n_short=262200, rows=rows)
    many = _batch(LIMIT + 32, [sc], alphabet, 8, n_short=262200 - LIMIT, rows=rows)
    al = Aligner(0)
    try:
        df, dm = DeviceBatch.from_host(few), DeviceBatch.from_host(many)
        buf = DeviceBatch(torch.zeros(max(df.queries.numel(), dm.queries.numel()), dtype=torch.uint8, device="cuda:0"),
                          df.q_off.clone(), torch.zeros(max(df.refs.numel(), dm.refs.numel()), dtype=torch.uint8, device="cuda:0"),
                          df.r_off.clone(), df.scheme_id.clone(), [sc])
        out = torch.empty((few.n_pairs, 5), dtype=torch.int32, device="cuda:0")
        for src, batch in ((df, few), (dm, many), (df, few)):
            buf.queries[:src.queries.numel()] = src.queries
            buf.refs[:src.refs.numel()] = src.refs
            buf.q_off.copy_(src.q_off)
            buf.r_off.copy_(src.r_off)
            assert np.array_equal(al.align(buf, out=out).cpu().numpy(), _want(batch))
        assert al.get_option("captures") == 1
    finally:
        al.close()

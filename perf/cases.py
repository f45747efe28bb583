"""Performance cases: the work that users of this library have it do.

Each case is one pass through a public entry point (Aligner.align, search,
align_cigar, Server, the grid diffusion step) on seeded inputs made on the
GPU (host arrays for the server).  The sizes are those of the workloads in
workloads.py and of bench.py, the smallest call among them, with generic odd
ones beside them; ``draw`` gives more cases of the same ranges.

Sequences follow workloads.mutate_embed: every reference embeds a mutated
copy of its query at a random place between random flanks.  Alignment
results are whole numbers and have no value in floating point, so ``exact``
answers for the diffusion cases only.
"""
import math

import numpy as np
import torch

from paper_2208_12350_amd import stencil
from paper_2208_12350_amd import workloads as W
from paper_2208_12350_amd.binding import Aligner, DeviceBatch, Server

DEV = "cuda:0"

# integer operations a cell cannot do without: the recurrence's 9 and 3 for
# the running best; the reverse pass sweeps about 0.65 of the forward cells
OPS_PER_CELL = 12 * 1.65


def listed():
    dna = dict(kind="align", data="dna", precision=0)
    return [
        # a single small batch, one call at a time: latency and launches
        dict(dna, name="align_dna_1k", pairs=1000, q_lo=50, q_hi=150, r_lo=100, r_hi=300),
        # short reads against their candidate windows, the throughput batch
        dict(dna, name="align_dna_200k", pairs=200_000, q_lo=100, q_hi=256, r_lo=200, r_hi=600),
        # protein homology batch: a 20-residue matrix
        dict(name="align_protein_100k", kind="align", data="protein", precision=0, pairs=100_000,
             q_lo=100, q_hi=500, r_lo=200, r_hi=1000),
        # DNA and protein pairs of log-normal lengths with a long tail, up to
        # 2048 query residues: the largest batch
        dict(name="align_mixed_1m", kind="align", data="mixed", precision=0, pairs=1_000_000,
             q_lo=32, q_hi=2048, r_lo=0, r_hi=0),
        # the exact 32-bit path on an odd-sized protein batch
        dict(name="align_protein_i32", kind="align", data="protein", precision=32, pairs=10_007,
             q_lo=100, q_hi=500, r_lo=200, r_hi=1000),
        # database search: one query against many references
        dict(name="search_protein_200k", kind="search", data="protein", pairs=200_000, q_lo=400, q_hi=400,
             r_lo=100, r_hi=1000),
        dict(name="search_dna_300k", kind="search", data="dna", pairs=300_000, q_lo=256, q_hi=256,
             r_lo=200, r_hi=600),
        # alignments with their paths, as a SAM writer needs them
        dict(name="cigar_dna_100k", kind="cigar", data="dna", pairs=100_000, q_lo=100, q_hi=256,
             r_lo=200, r_hi=600),
        dict(name="cigar_mixed_50k", kind="cigar", data="mixed", pairs=50_001, q_lo=32, q_hi=2048, r_lo=0, r_hi=0),
        # one request of host arrays through the server, alone
        dict(name="serve_mixed_2500", kind="serve", data="mixed", pairs=2500, requests=1),
        # grid diffusion: the paper's held-out grid for some steps (in cache,
        # bounds-checked), and a streaming grid (zero-padded)
        dict(name="diffuse_checked_2500", kind="diffuse", form="checked", nx=2500, ny=2500, steps=20),
        dict(name="diffuse_padded_16384", kind="diffuse", form="padded", nx=16384, ny=16384, steps=2),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["align", "align", "align", "search", "cigar", "serve", "diffuse"])
    if kind == "diffuse":
        form = rng.choice(["checked", "padded"])
        nx, ny = _log_int(rng, 100, 16000), _log_int(rng, 100, 16000)
        return dict(kind=kind, form=form, nx=nx, ny=ny, steps=rng.choice([1, 2, 5, 10]))
    if kind == "serve":
        return dict(kind=kind, data="mixed", pairs=rng.randint(1, 5000), requests=rng.choice([1, 2, 4]))
    data = rng.choice(["dna", "protein"] if kind == "search" else ["dna", "protein", "mixed"])
    case = dict(kind=kind, data=data)
    if kind == "align":
        case["precision"] = rng.choice([0, 0, 0, 0, 32])
    if data == "mixed":
        case.update(q_lo=32, q_hi=2048, r_lo=0, r_hi=0)
        cells = 431e3
    else:
        q_lo = _log_int(rng, 30, 1200)
        q_hi = q_lo if kind == "search" else min(2048, int(q_lo * rng.uniform(1.0, 3.0)))
        r_lo = int(q_lo * rng.uniform(0.8, 2.0))
        r_hi = int(max(r_lo, q_hi) * rng.uniform(1.0, 3.0))
        case.update(q_lo=q_lo, q_hi=q_hi, r_lo=r_lo, r_hi=r_hi)
        cells = 0.25 * (q_lo + q_hi) * (r_lo + r_hi)
    # a bound on the cells of a call: 32-bit and path calls are smaller
    most = {"align": 5e10, "search": 5e10, "cigar": 1.5e10}[kind]
    if case.get("precision") == 32:
        most = 4e9
    case["pairs"] = _log_int(rng, 20, max(40, min(500_000, most / cells)))
    return case


# ---- inputs ---------------------------------------------------------------------

def _schemes(data, seed):
    dna, prot = W.dna_scheme(), W.protein_scheme(seed)
    return {"dna": [dna], "protein": [prot], "mixed": [dna, prot]}[data]


def _residues(n, prot, cdf, g):
    """n residues: DNA letters where prot is 0, protein letters by their frequencies where it is 1."""
    u = torch.rand(n, device=DEV, generator=g)
    d = (u * 4).to(torch.uint8).clamp_(max=3)
    if cdf is None:
        return d
    p = torch.searchsorted(cdf, u).clamp_(max=19).to(torch.uint8)
    return p if prot is None else torch.where(prot, p, d)


def _offsets(lens):
    off = torch.zeros(lens.numel() + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(lens, 0, out=off[1:])
    return off


def _uniform(n, lo, hi, g):
    return torch.randint(lo, hi + 1, (n,), device=DEV, generator=g, dtype=torch.int64)


def _pairs(case, seed, one_query=False):
    """(queries, q_off, refs, r_off, scheme_id): the mutated embedding of
    workloads.mutate_embed; for a search, one query, of which 1% of the
    references embed a copy."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 7919 + 13)
    n, data = case["pairs"], case["data"]
    if data == "mixed":
        ql = torch.exp(torch.randn(n, device=DEV, generator=g) * 0.8 + math.log(150.0)).round().clamp(32, 1024)
        long_tail = torch.rand(n, device=DEV, generator=g) >= 0.95
        ql = torch.where(long_tail, _uniform(n, 1024, 2048, g), ql.to(torch.int64))
        rl = (ql * (1.5 + 1.5 * torch.rand(n, device=DEV, generator=g))).round().to(torch.int64)
        is_prot = torch.rand(n, device=DEV, generator=g) < 0.2
    else:
        ql = _uniform(n, case["q_lo"], case["q_hi"], g)
        rl = _uniform(n, case["r_lo"], case["r_hi"], g)
        is_prot = torch.full((n,), data == "protein", device=DEV)
    cdf = None
    if data != "dna":
        cdf = torch.from_numpy(np.cumsum(W.protein_frequencies(seed))).to(DEV, torch.float32)
    q_off = _offsets(ql)
    total = int(q_off[-1])
    mixed = data == "mixed"
    q_prot = torch.repeat_interleave(is_prot, ql, output_size=total) if data != "dna" else None
    p_sub, p_indel = (0.30, 0.03) if data == "protein" else (0.10, 0.02)
    if mixed:
        p_sub = torch.where(q_prot, 0.30, 0.10)
        p_indel = torch.where(q_prot, 0.03, 0.02)
    if one_query:
        queries = _residues(case["q_lo"], None, cdf, g).repeat(n)
    else:
        queries = _residues(total, q_prot if mixed else None, cdf, g)
    # mutate: each position becomes an indel or a substitution, or is kept
    u = torch.rand(total, device=DEV, generator=g)
    half = torch.rand(total, device=DEV, generator=g) < 0.5
    is_ins, is_del = (u < p_indel) & half, (u < p_indel) & ~half
    sub = (u >= p_indel) & (torch.rand(total, device=DEV, generator=g) < p_sub)
    kept = torch.where(sub, _residues(total, q_prot if mixed else None, cdf, g), queries)
    first = torch.where(is_ins, _residues(total, q_prot if mixed else None, cdf, g), kept)
    take = torch.stack([~is_del, is_ins], 1).reshape(-1)
    copy = torch.stack([first, kept], 1).reshape(-1)[take]
    emitted = _offsets((~is_del).to(torch.int64) + is_ins.to(torch.int64))
    copy_off = emitted[q_off]
    copy_len = copy_off[1:] - copy_off[:-1]
    homolog = torch.rand(n, device=DEV, generator=g) < 0.01 if one_query else None
    rl = torch.maximum(rl, copy_len if homolog is None else torch.where(homolog, copy_len, 0))
    r_off = _offsets(rl)
    total_r = int(r_off[-1])
    r_prot = torch.repeat_interleave(is_prot, rl, output_size=total_r) if mixed else None
    refs = _residues(total_r, r_prot, cdf, g)
    if homolog is not None:
        keep = torch.repeat_interleave(homolog, copy_len, output_size=copy.numel())
        copy, copy_len = copy[keep], torch.where(homolog, copy_len, 0)
    start = r_off[:-1] + ((rl - copy_len + 1) * torch.rand(n, device=DEV, generator=g)).to(torch.int64)
    start = torch.minimum(start, r_off[1:] - copy_len)
    marks = torch.zeros(total_r + 1, dtype=torch.int32, device=DEV)
    marks.scatter_add_(0, start, torch.ones(n, dtype=torch.int32, device=DEV))
    marks.scatter_add_(0, start + copy_len, torch.full((n,), -1, dtype=torch.int32, device=DEV))
    refs.masked_scatter_(torch.cumsum(marks[:-1], 0) > 0, copy)
    return queries, q_off, refs, r_off, (is_prot.to(torch.uint8) if mixed else torch.zeros_like(is_prot, dtype=torch.uint8))


def _grid(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 7919 + 17)
    return torch.rand((case["ny"], case["nx"]), device=DEV, generator=g)


SPREAD = 0.3   # the diffusion fraction D


def prepare(case, seed):
    kind = case["kind"]
    if kind == "diffuse":
        grid = _grid(case, seed)
        if case["form"] == "padded":
            grid = stencil.pad(grid)
        return dict(case=case, src=grid, bufs=[torch.zeros_like(grid), torch.zeros_like(grid)])
    if kind == "serve":
        server = Server(_schemes("mixed", seed), pool_bytes=2 << 30)
        reqs = [W.make_workload("mixed", n_pairs=max(1, case["pairs"] - 7 * k), seed=seed * 100 + k, scheme_seed=seed)
                for k in range(case["requests"])]
        return dict(case=case, server=server, requests=reqs)
    q, qo, r, ro, sid = _pairs(case, seed, one_query=kind == "search")
    schemes = _schemes(case["data"], seed)
    al = Aligner(0, precision=case.get("precision", 0))
    out = torch.empty((case["pairs"], 5), dtype=torch.int32, device=DEV)
    st = dict(case=case, al=al, out=out)
    if kind == "search":
        st.update(query=q[:case["q_lo"]].clone(), refs=r, r_off=ro, scheme=schemes[0])
        return st
    st["batch"] = DeviceBatch(q, qo, r, ro, sid, schemes)
    if kind == "cigar":
        # room for q_len + r_len runs per pair, which always suffices
        st["off"] = _offsets((qo[1:] - qo[:-1]) + (ro[1:] - ro[:-1]))
        st["cigar"] = torch.empty(int(st["off"][-1]), dtype=torch.int32, device=DEV)
        st["len"] = torch.empty(case["pairs"], dtype=torch.int32, device=DEV)
        # and for the runs of the whole batch back to back (a path changes
        # its operation far less often than once per query residue)
        mean_q = 275 if case["data"] == "mixed" else (case["q_lo"] + case["q_hi"]) // 2
        st["runs"] = torch.zeros(case["pairs"] * (mean_q + 64), dtype=torch.int32, device=DEV)
    return st


def run(st):
    kind = st["case"]["kind"]
    if kind == "align":
        return st["al"].align(st["batch"], out=st["out"])
    if kind == "search":
        return st["al"].search(st["query"], st["refs"], st["r_off"], st["scheme"], out=st["out"])
    if kind == "cigar":
        out, off, cigar, length = st["al"].align_cigar(st["batch"], out=st["out"], cigar_off=st["off"],
                                                       cigar=st["cigar"], cigar_len=st["len"])
        # the runs of all pairs back to back, as a writer takes them, zero past their end
        ends = torch.cumsum(length, 0, dtype=torch.int64)
        total = int(ends[-1])
        at = torch.repeat_interleave(off[:-1] - (ends - length), length, output_size=total)
        st["runs"][:total] = cigar[at + torch.arange(total, device=DEV)]
        st["runs"][total:] = 0
        return out, length, st["runs"]
    if kind == "serve":
        tickets = [st["server"].submit(b) for b in st["requests"]]
        return [st["server"].poll(t)[0] for t in tickets]
    src = st["src"]
    for k in range(st["case"]["steps"]):
        dst = st["bufs"][k % 2]
        if st["case"]["form"] == "padded":
            stencil.diffuse_padded(src, dst, st["case"]["nx"], st["case"]["ny"], SPREAD)
        else:
            stencil.diffuse_checked(src, dst, SPREAD)
        src = dst
    return src


def work(case):
    if case["kind"] == "diffuse":
        points = float(case["nx"]) * case["ny"] * case["steps"]
        return {"bytes": 8 * points, "flops": 10 * points}
    n = float(case["pairs"]) * case.get("requests", 1)
    if case["data"] == "mixed":
        q, r, cells = 275.0, 618.0, 431e3
    else:
        q, r = 0.5 * (case["q_lo"] + case["q_hi"]), 0.5 * (case["r_lo"] + case["r_hi"])
        cells = q * r
    residues = r if case["kind"] == "search" else q + r
    return {"bytes": n * (residues + 17 + 20), "flops": n * cells * OPS_PER_CELL}


def exact(case, seed):
    if case["kind"] != "diffuse":
        return None
    c = _grid(case, seed).double()
    for _ in range(case["steps"]):
        p = torch.nn.functional.pad(c, (1, 1, 1, 1))
        rows = p[:, :-2] + p[:, 1:-1] + p[:, 2:]
        box = rows[:-2] + rows[1:-1] + rows[2:]
        c = (1.0 - SPREAD) * c + (SPREAD / 8.0) * (box - c)
    if case["form"] == "padded":
        nx, ny = case["nx"], case["ny"]
        full = torch.zeros((ny + 2, stencil.padded_pitch(nx)), dtype=torch.float64, device=DEV)
        full[1:ny + 1, 1:nx + 1] = c
        c = full
    return c

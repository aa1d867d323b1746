"""Timed cases of the alignment library, over the range of calls a program makes.

Every case runs one call (or, when serving, one burst of calls) through the
public entry points on planted genes drawn from the seed
(``paper_2210_08052_amd.workloads``): the letters, anchors or profiles, the
output buffers and the handles a program keeps are made by ``prepare``, the
call itself by ``run``.  One ``Context`` with its own stream serves all batch
cases of the process, as it would in a program; serving has a context of its
own, since its parameters are fixed by the first job.  Widths and packing are
the library's defaults (no autotuning).

Results are whole numbers and bytes (records, op strings), except the fp64
chaining scores, whose 64-bit values ``exact`` gives.
"""
import math

import numpy as np
import torch

from paper_2210_08052_amd import mpg
from paper_2210_08052_amd import workloads as W

# Means of the batch recipe (workloads.batch_pairs), for work(): residues and
# nucleotides of a pair, cells of a pair, pieces' cells of a chain, second-pass
# cells of a rescored pair, anchors and candidate pairs of an anchor set.
RESIDUES, BASES, CELLS = 450.0, 4200.0, 2.04e6
CHAIN_CELLS, RESCORE_CELLS = 2.6e5, 8.0e5
ANCHORS, CANDIDATES = 105.0, 7.9e3
OPS_CELL = 23      # max-plus operations of one DP cell
OPS_CELL_FS = 12   # without introns, one mode (the second pass of rescoring)
OPS_LINK = 12      # fp64 operations of one candidate link

# kind -> (smallest, largest) number of pairs, chains, sets or jobs
RANGE = {
    "single": (1, 1),          # one traced pair, sequences resident
    "host": (4, 400),          # host buffers in, results out
    "score": (100, 10000),     # resident batch, score-only
    "traced": (100, 3000),     # resident batch, op strings
    "int16": (100, 4000),      # resident score-only batch, 16-bit lanes allowed
    "long": (2, 8),            # long proteins on long regions, with short ones
    "profile": (30, 1000),     # position-specific queries
    "rescore": (100, 3000),    # pseudogene guard on a traced batch
    "chains": (100, 3000),     # anchor-driven alignment
    "chaining": (100, 3000),   # anchor sets to chains
    "graph": (8, 256),         # a planned batch replayed from its graph
    "serve": (16, 512),        # jobs submitted and polled
}


def listed():
    return [
        # One gene looked up: the smallest call, its time is launch latency
        # and one pair's serial steps.
        {"name": "single_traced", "kind": "single", "n": 1},
        # A few proteins from host memory, results back on the host.
        {"name": "host_60", "kind": "host", "n": 60},
        # A proteome's worth of pairs screened by score: the largest batch.
        {"name": "score_10000", "kind": "score", "n": 10000},
        # The same kind of pairs with their alignments.
        {"name": "traced_3000", "kind": "traced", "n": 3000},
        # Screening with 16-bit lanes allowed by the caller.
        {"name": "int16_4000", "kind": "int16", "n": 4000},
        # Long proteins on regions of 100-300 kb among short pairs, traced.
        {"name": "long_6", "kind": "long", "n": 6},
        # Family profiles instead of proteins, score-only.
        {"name": "profile_1000", "kind": "profile", "n": 1000},
        # The pseudogene guard after a traced batch (end to end, no introns).
        {"name": "rescore_3000", "kind": "rescore", "n": 3000},
        # Alignment between and beyond the anchors of a chain, traced.
        {"name": "chains_3000", "kind": "chains", "n": 3000},
        # Seed anchors to chains (fp64).
        {"name": "chaining_3000", "kind": "chaining", "n": 3000},
        # A small planned batch replayed from a graph, as a request loop does.
        {"name": "graph_48", "kind": "graph", "n": 48},
        # A burst of jobs through the serving queue, half of them traced.
        {"name": "serve_300", "kind": "serve", "n": 300},
    ]


def draw(rng):
    kind = rng.choice(sorted(RANGE))
    lo, hi = RANGE[kind]
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    case = {"kind": kind, "n": max(lo, min(hi, n))}
    if kind == "single":  # any one gene, wanted traced or not, in each mode
        case["residues"] = int(round(math.exp(rng.uniform(math.log(20), math.log(900)))))
        case["mode"] = rng.choice(["LOCAL", "EXTEND", "EXTEND_LEFT"])
        case["traced"] = rng.random() < 0.7
    if kind in ("score", "traced"):
        case["introns"] = rng.random() < 0.8
        case["frameshifts"] = rng.random() < 0.8
        case["mode"] = rng.choice(["LOCAL", "LOCAL", "EXTEND"])
    return case


# ------------------------------------------------------------------ handles
_handles = {}


def _context():
    """The process's batch context and its stream."""
    if "batch" not in _handles:
        stream = torch.cuda.Stream()
        ctx = mpg.Context(0)
        ctx.set_stream(stream.cuda_stream)
        _handles["batch"] = (ctx, stream)
    return _handles["batch"]


def _server():
    if "serve" not in _handles:
        _handles["serve"] = mpg.Context(0)
    return _handles["serve"]


def _to_gpu(data):
    return torch.frombuffer(bytearray(data + b"\0" * 16), dtype=torch.uint8).cuda()


def _params(case):
    flags = 0
    if not case.get("introns", True):
        flags |= mpg.MPG_NO_INTRON
    if not case.get("frameshifts", True):
        flags |= mpg.MPG_NO_FRAMESHIFT
    if case["kind"] == "int16":
        flags |= mpg.MPG_ALLOW_I16
    mode = {"LOCAL": mpg.MPG_LOCAL, "EXTEND": mpg.MPG_EXTEND, "EXTEND_LEFT": mpg.MPG_EXTEND_LEFT,
            "GLOBAL": mpg.MPG_GLOBAL}[case.get("mode", "LOCAL")]
    return mpg.params(flags=flags, mode=mode)


def _outputs(state, n, need):
    """Records of n pairs and an op-string buffer.  The buffer's size depends
    on the number of pairs alone, as in a program that keeps one buffer for
    calls of a size; it grows where the pairs at hand need more."""
    if state["kind"] in ("score", "int16", "profile") or not state.get("traced", True):
        room = n
    elif state["kind"] == "long":
        room = 700000 * n
    else:
        room = 12000 * n + int(100000 * math.sqrt(n))
    state["cap"] = max(room, need)
    state["rec"] = torch.zeros(n * mpg.DEV_RESULT_DTYPE.itemsize, dtype=torch.uint8,
                               device="cuda")
    state["ops"] = torch.zeros(state["cap"], dtype=torch.uint8, device="cuda")


def _resident(state, pairs):
    """Letters of (prot, dna, traced) pairs on the GPU, and the outputs."""
    pb, db, segs = mpg.pack_pairs(pairs)
    state["prot"], state["dna"], state["segs"] = _to_gpu(pb), _to_gpu(db), segs
    _outputs(state, len(pairs), int(mpg.lib().mpg_ops_capacity(segs.ctypes.data, len(segs))))


def _gene(rng, L):
    """One planted gene of L residues in a region about 1.2 times its span."""
    while True:
        p = W._short_pair(rng, L)
        if p is not None:
            return p


def _seed_hits(pair, k=6):
    """Runs of k residues left unchanged whose codons are whole and
    consecutive in the region: (x, y) of each, as seeding finds them."""
    at, same = pair.truth["codon_at"], pair.truth["kept"]
    n = len(at) - k + 1
    if n <= 0:
        return np.zeros((0, 2), np.int64)
    good = (at >= 0) & same
    step = np.zeros(len(at), bool)
    step[:-1] = good[:-1] & good[1:] & (np.diff(at) == 3)
    run = np.concatenate([[0], np.cumsum(step)])
    y = np.nonzero(good[:n] & (run[k - 1:k - 1 + n] - run[:n] == k - 1))[0]
    return np.stack([at[y], y], axis=1)


_AA = np.zeros(256, np.int64)
_AA[[ord(c) for c in W.STD20]] = np.arange(20)
_B62 = W._b62_20().astype(np.float64)


def _profile(prot, rng):
    """A family profile of a protein (the rule of workloads.family_profile)."""
    idx = _AA[np.frombuffer(prot, np.uint8)]
    m = len(idx)
    rows = np.repeat(idx[:, None], 4, axis=1)
    other = (rng.random((m, 3))[:, :, None] >= W._CDF[idx][:, None, :]).sum(axis=2).clip(0, 19)
    rows[:, 1:] = np.where(rng.random((m, 3)) < 0.7, rows[:, 1:], other)
    score = np.full((m, 24), -1, np.int8)
    score[:, :20] = np.rint(_B62[rows].mean(axis=1)).astype(np.int8)
    score[:, 23] = -4
    gap = np.tile(np.array([11, 1, 11, 1], np.int16), (m + 1, 1))
    for s in np.nonzero(rng.random(m + 1) < 0.02)[0]:
        gap[s:s + 6, 0] = 5
        gap[s:s + 6, 2] = 5
    return score, gap


def _anchor_sets(n, seed):
    """Anchor sets of planted genes: half of the true seed hits at a locus of
    a 100-Mb genome in 256-bp bins, and as many spurious ones within 2 Mb."""
    rng = np.random.Generator(np.random.PCG64(seed + 2000))
    sets = []
    for p in W.batch_pairs(n, seed=seed):
        hits = _seed_hits(p)
        hits = hits[rng.random(len(hits)) < 0.5]
        base = int(rng.integers(2_000_000, 98_000_000))
        k = int(rng.poisson(len(hits) + 5))
        noise = np.stack([rng.integers(-2_000_000, 2_000_000, k),
                          rng.integers(0, max(1, len(p.prot) - 5), k)], axis=1)
        a = np.concatenate([hits, noise]).astype(np.int64)
        a[:, 0] = (a[:, 0] + base) // 256
        sets.append(a[np.lexsort((a[:, 1], a[:, 0]))].astype(np.int32))
    return sets


def _room(n):
    """Anchors that the buffers of a call with n sets hold."""
    return 100 * n + int(2500 * math.sqrt(n))


# ------------------------------------------------------------------ prepare
def prepare(case, seed):
    kind, n = case["kind"], case["n"]
    rng = np.random.Generator(np.random.PCG64([seed, 77]))
    state = {"kind": kind, "n": n, "params": _params(case), "traced": case.get("traced", True)}
    if kind == "serve":
        state["jobs"] = [(p.prot, p.dna, k % 2 == 0)
                         for k, p in enumerate(W.batch_pairs(n, seed=seed))]
        state["ctx"] = _server()
        return state
    ctx, stream = _context()
    state["ctx"], state["stream"] = ctx, stream
    if kind == "single":
        p = _gene(rng, case["residues"]) if "residues" in case else W.single_pair(seed)
        _resident(state, [(p.prot, p.dna, state["traced"])])
    elif kind == "host":
        state["pairs"] = [(p.prot, p.dna, True) for p in W.batch_pairs(n, seed=seed)]
    elif kind in ("score", "traced", "int16"):
        _resident(state, [(p.prot, p.dna, kind == "traced") for p in W.batch_pairs(n, seed=seed)])
    elif kind == "long":
        _resident(state, [(p.prot, p.dna, True) for p in W.long_tail(n, 10 * n, seed=seed)])
    elif kind == "profile":
        jobs = [_profile(p.prot, rng) + (p.dna,) for p in W.batch_pairs(n, seed=seed)]
        fb, db, segs, cap = mpg.pack_profiles(jobs)
        state["prof"], state["dna"], state["segs"] = _to_gpu(fb), _to_gpu(db), segs
        _outputs(state, n, cap)
    elif kind == "rescore":
        _resident(state, [(p.prot, p.dna, True) for p in W.batch_pairs(n, seed=seed)])
        state["fin"] = torch.zeros((3, n), dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()
        _align(state)
    elif kind == "chains":
        chains = []
        for p in W.batch_pairs(n, seed=seed):
            hits = _seed_hits(p)
            hits = hits[rng.random(len(hits)) < 0.25] if len(hits) > 1 else hits
            if not len(hits):  # one seed where the gene starts
                hits = np.array([[p.truth["gene_start"], 0]])
            chains.append((p.prot, p.dna, hits, 6, True))
        pb, db, segs = mpg.pack_chains(chains)
        state["prot"], state["dna"], state["segs"] = _to_gpu(pb), _to_gpu(db), segs
        _outputs(state, n, segs.ops_capacity(state["params"]))
    elif kind == "chaining":
        sets = _anchor_sets(n, seed)
        off = np.zeros(n + 1, np.int64)
        off[1:] = np.cumsum([len(a) for a in sets])
        total = max(int(off[-1]), _room(n))
        state["params"] = mpg.chaining_params()
        state["off"] = off
        state["anchors"] = torch.from_numpy(np.concatenate(sets)).cuda()
        state["f"] = torch.zeros(total, dtype=torch.float64, device="cuda")
        state["pred"] = torch.zeros(total, dtype=torch.int32, device="cuda")
        state["idx"] = torch.zeros(total, dtype=torch.int32, device="cuda")
        state["top"] = torch.zeros((n, state["params"].max_chains, 2), dtype=torch.float64,
                                   device="cuda")
        state["ntop"] = torch.zeros(n, dtype=torch.int32, device="cuda")
    elif kind == "graph":
        _resident(state, [(p.prot, p.dna, k % 2 == 0)
                          for k, p in enumerate(W.batch_pairs(n, seed=seed))])
        torch.cuda.synchronize()
        state["plan"] = ctx.plan(state["params"], state["prot"].data_ptr(),
                                 state["dna"].data_ptr(), state["segs"], state["rec"].data_ptr(),
                                 state["ops"].data_ptr(), state["cap"])
        state["plan"].graph(stream.cuda_stream)
    torch.cuda.synchronize()
    return state


# ---------------------------------------------------------------------- run
def _align(s):
    s["ctx"].align_batch_dev(s["params"], s["prot"].data_ptr(), s["dna"].data_ptr(), s["segs"],
                             s["rec"].data_ptr(), s["ops"].data_ptr(), s["cap"])


def _host_results(results):
    """Results of a host call as arrays: the number fields, and the op strings
    in a buffer of one size for a number of results."""
    keys = ("status", "score", "g_beg", "g_end", "p_beg", "p_end")
    text = "\n".join(r["ops"] or "" for r in results).encode()
    text = text.ljust(2000 * len(results) + 20000, b"\0")
    return {"fields": np.array([[r[k] for k in keys] for r in results], np.int32),
            "ops": np.frombuffer(text, np.uint8)}


def run(s):
    kind = s["kind"]
    if kind in ("single", "score", "traced", "int16", "long"):
        _align(s)
    elif kind == "host":
        return _host_results(s["ctx"].align_batch(s["pairs"], s["params"]))
    elif kind == "profile":
        s["ctx"].align_profiles_dev(s["params"], s["prof"].data_ptr(), s["dna"].data_ptr(),
                                    s["segs"], s["rec"].data_ptr(), s["ops"].data_ptr(), s["cap"])
    elif kind == "rescore":
        fin = s["fin"]
        s["ctx"].rescore_spliced_dev(s["params"], s["prot"].data_ptr(), s["dna"].data_ptr(),
                                     s["segs"], s["rec"].data_ptr(), s["ops"].data_ptr(),
                                     fin[0].data_ptr(), fin[1].data_ptr(), fin[2].data_ptr())
        return fin
    elif kind == "chains":
        s["ctx"].align_chains_dev(s["params"], s["prot"].data_ptr(), s["dna"].data_ptr(), s["segs"],
                                  s["rec"].data_ptr(), s["ops"].data_ptr(), s["cap"])
    elif kind == "chaining":
        s["ctx"].chain_anchors_dev(s["params"], s["anchors"].data_ptr(), s["off"],
                                   s["f"].data_ptr(), s["pred"].data_ptr(), s["idx"].data_ptr(),
                                   s["top"].data_ptr(), s["ntop"].data_ptr())
        return {"f": s["f"], "pred": s["pred"], "idx": s["idx"], "ntop": s["ntop"],
                "score": s["top"][:, :, 0], "range": s["top"].view(torch.int32)[:, :, 2:]}
    elif kind == "graph":
        s["plan"].launch(s["stream"].cuda_stream)
    elif kind == "serve":
        ctx, p = s["ctx"], s["params"]
        place = {ctx.submit(p, a, b, t): k for k, (a, b, t) in enumerate(s["jobs"])}
        results = [None] * len(place)
        left = len(place)
        while left:
            for r in ctx.poll(512, 2000):
                results[place[r["job_id"]]] = r
                left -= 1
        return _host_results(results)
    return {"records": s["rec"].view(torch.int32).view(s["n"] if kind != "long" else -1, 10),
            "ops": s["ops"]}


# --------------------------------------------------------------------- work
def work(case):
    kind, n = case["kind"], case["n"]
    letters, ops_out = (RESIDUES + BASES) * n, 0.0
    cells, ops = CELLS * n, OPS_CELL
    if kind == "single":
        m = case.get("residues", 100)
        letters, cells = m * 10.4 if "residues" in case else 3100.0, 0
        cells = m * (letters - m)
    elif kind == "long":
        letters, cells = 2.06e5 * n + 10 * n * 2.3e3, 1.1e9 * n + 10 * n * 4.3e5
    elif kind == "profile":
        letters = (32 * RESIDUES + BASES) * n
    elif kind == "rescore":
        cells, ops = RESCORE_CELLS * n, OPS_CELL_FS
    elif kind == "chains":
        cells = CHAIN_CELLS * n
    elif kind == "chaining":
        return {"bytes": n * (ANCHORS * (8 + 16) + 30 * 16), "flops": n * CANDIDATES * OPS_LINK}
    if kind in ("single", "host", "traced", "long", "chains"):
        ops_out = 0.05 * letters  # op strings
    return {"bytes": letters + ops_out + 40.0 * n, "flops": cells * ops}


# -------------------------------------------------------------------- exact
def exact(case, seed):
    """fp64 chaining scores of every anchor, from the recurrence: f(j) =
    max(k, max over i of f(i) + min(dy, k) - gamma(g)); all sets at once,
    anchor by anchor.  The other cases return whole numbers and bytes."""
    if case["kind"] != "chaining":
        return None
    sets = _anchor_sets(case["n"], seed)
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    top, n = max(len(a) for a in sets), len(sets)
    order = sorted(range(n), key=lambda s: -len(sets[s]))
    size = np.array([len(sets[s]) for s in order])
    xy = np.zeros((n, top, 2))
    for r, s in enumerate(order):
        xy[r, :len(sets[s])] = sets[s]
    xy = torch.from_numpy(xy).to(dev)
    f = torch.full((n, top), 6.0, dtype=torch.float64, device=dev)
    for j in range(1, top):
        live = int((size > j).sum())
        dx = xy[:live, j, 0:1] - xy[:live, :j, 0]
        dy = xy[:live, j, 1:2] - xy[:live, :j, 1]
        lo, hi = 256 * (dx - 1), 256 * (dx + 1)
        g = torch.where(3 * dy < lo, 3 * dy - lo, torch.where(3 * dy > hi, 3 * dy - hi, 0.0))
        a = g.abs()
        third, lg = a / 3.0, 0.75 * torch.log2(a + 1.0)
        gamma = torch.where(g > 0, third + lg, torch.minimum(third, lg))
        v = f[:live, :j] + dy.clamp(max=6.0) - gamma
        v = torch.where((dx >= 0) & (dy > 0) & (a < 200000), v, -math.inf)
        f[:live, j] = torch.maximum(f[:live, j], v.max(dim=1).values)
    where = np.argsort(order)
    f = f.cpu()
    parts = [f[where[s], :len(sets[s])] for s in range(n)]
    rest = max(0, _room(n) - sum(len(a) for a in sets))  # the buffer's unused end
    parts.append(torch.zeros(rest, dtype=torch.float64))
    return {"f": torch.cat(parts), "idx": None,
            "ntop": None, "pred": None, "range": None, "score": None}

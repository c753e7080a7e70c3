"""The work that programs built on this library have it do, as timed cases.

A program loads a graph (validation), builds its proposal tables, and then
estimates pattern counts: one pattern with a fixed number of samples, one
pattern to an error target, or a set of patterns to an error target.  Clique
programs orient the graph by degree first.  Programs that learn a proposal
also produce training rows from the sampler, train the network, and turn its
output into pick tables.  Each of these is one kind of case here, called
through the package's public entry points.

Graphs are R-MAT (edge factor 16, a = .57, b = c = .19) and Chung-Lu
(gamma 2.1) power-law graphs, drawn from the case's seed.
"""

from __future__ import annotations

import math

import numpy as np
import torch

import synth
from paper_2601_01388_amd import (agis_compile_pattern, agis_learn_rows, agis_mlp_param_count, agis_tables_export,
                                  make_params, make_pattern)
from paper_2601_01388_amd.session import Session, mlp_init

HIDDEN, INPUTS = 64, 8


def listed():
    return [
        # the smallest call: one quick estimate on a small graph, a service
        # answering interactive questions (latency and launches count)
        dict(name="small_triangle", kind="estimate", graph="chung_lu", n=2000, m=12000, pattern="triangle",
             mode="switch", samples=4096, eps=0.0),
        # fixed-size estimates on the R-MAT-20 graph: an intersecting pattern
        # that lives in the dense core, a sparse one, and one whose samples
        # are independent single-row draws
        dict(name="rmat20_5clique", kind="estimate", graph="rmat", scale=20, pattern="5-clique", mode="switch",
             samples=4_000_000, eps=0.0),
        dict(name="rmat20_5cycle", kind="estimate", graph="rmat", scale=20, pattern="5-cycle", mode="switch",
             samples=4_000_001, eps=0.0),
        dict(name="rmat20_4star", kind="estimate", graph="rmat", scale=20, pattern="4-star", mode="switch",
             samples=20_000_000, eps=0.0),
        # a larger graph and a larger pattern, every step weighted
        dict(name="rmat22_7cycle", kind="estimate", graph="rmat", scale=22, pattern="chordal-7-cycle", mode="always",
             samples=300_000, eps=0.0),
        # an estimate to +-1% at 95%: the stop decision is part of the call
        dict(name="rmat20_house_eps", kind="estimate", graph="rmat", scale=20, pattern="house", mode="switch",
             samples=50_000_000, eps=0.01),
        # concentrations: every connected 5-vertex pattern to an error target
        # in batched launches, uneven costs side by side
        dict(name="rmat20_conc5", kind="concentrations", scale=20, k=5, budget=5_000_000, eps=0.01),
        # what a program pays before its first estimate on a new graph:
        # validation and the proposal tables
        dict(name="rmat20_preprocess", kind="preprocess", scale=20),
        # cliques as the method runs them: orientation, its tables, estimate
        dict(name="rmat20_clique_dag", kind="clique_dag", scale=20, pattern="4-clique", samples=1_000_000),
        # learned proposal: training rows from the sampler's own samples
        dict(name="rmat18_targets", kind="targets", scale=18, pattern="5-clique", samples=1 << 20),
        # learned proposal: full-batch Adam steps of the network
        dict(name="train_48k", kind="train", rows=48_001, vertices=1 << 18, epochs=48),
        # learned proposal: features and pick tables of a graph
        dict(name="rmat22_tables", kind="tables", scale=22, pattern="house"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["estimate"] * 6 + ["concentrations", "preprocess", "clique_dag", "targets", "train", "tables"])
    scale = rng.randint(10, 20)
    if kind == "estimate":
        # every named pattern of at least a wedge, each proposal, fixed sizes
        # and error targets, on both kinds of graph
        pattern = rng.choice(sorted(n for n in synth.NAMED_PATTERNS if n != "edge"))
        k = synth.named_pattern(pattern).k
        case = dict(kind=kind, pattern=pattern, mode=rng.choice(["switch", "switch", "always", "uniform"]))
        if rng.random() < 0.3:
            n = _log_int(rng, 500, 20_000)
            case.update(graph="chung_lu", n=n, m=n * rng.randint(5, 10))
        else:
            case.update(graph="rmat", scale=scale)
        if rng.random() < 0.3:
            case.update(eps=rng.choice([0.01, 0.02, 0.05]), samples=_log_int(rng, 1e5, 1e6))
        else:
            case.update(eps=0.0, samples=_log_int(rng, 1000, 2e6 if k <= 5 else 5e5))
        return case
    if kind == "concentrations":
        return dict(kind=kind, scale=min(scale, 18), k=rng.choice([3, 4, 5]), budget=_log_int(rng, 1e5, 2e6),
                    eps=rng.choice([0.01, 0.02, 0.05]))
    if kind == "preprocess":
        return dict(kind=kind, scale=scale)
    if kind == "clique_dag":
        return dict(kind=kind, scale=scale, pattern=rng.choice(["triangle", "4-clique", "5-clique"]),
                    samples=_log_int(rng, 10_000, 1_000_000))
    if kind == "targets":
        return dict(kind=kind, scale=min(scale, 18), pattern=rng.choice(["triangle", "5-clique", "house", "5-cycle"]),
                    samples=_log_int(rng, 10_000, 1_000_000))
    if kind == "train":
        return dict(kind=kind, rows=_log_int(rng, 100, 48_000), vertices=1 << rng.randint(12, 18),
                    epochs=rng.randint(4, 48))
    return dict(kind=kind, scale=rng.randint(10, 21), pattern=rng.choice(["house", "5-clique", "4-path"]))


# ---------------------------------------------------------------- inputs

_sessions = {}


def _session():
    """The one library context of the program, on torch's current stream."""
    stream = torch.cuda.current_stream().cuda_stream
    if stream not in _sessions:
        _sessions[stream] = Session(torch.cuda.current_device())
    return _sessions[stream]


class _State:
    """What a program holds between calls; frees its handles at its end."""

    def __init__(self, case, sess):
        self.case = case
        self.sess = sess
        self.graph = None
        self.tables = None

    def __del__(self):
        for handle in (self.tables, self.graph):
            if handle is not None:
                handle.close()


def _csr(case, seed):
    if case.get("graph") == "chung_lu":
        g = synth.chung_lu(n=case["n"], m=case["m"], seed=seed)
        return g.off, g.nbr
    return synth.graphs.rmat_device(case["scale"], 16, seed=seed, device="cuda")


def _training_set(case, seed):
    """Rows as the sampler produces them: vertices in proportion to a
    power-law degree, counts as weights, residual targets around zero."""
    rng = np.random.Generator(np.random.PCG64(seed))
    n, rows = case["vertices"], case["rows"]
    deg = np.floor(2.0 * (1.0 - rng.random(n)) ** -0.8)
    feats = np.stack([np.log2(1 + deg), np.log2(1 + deg * rng.uniform(20, 400, n)),
                      np.log2(1 + deg * (deg - 1) * 0.5 * rng.random(n) ** 2),
                      np.log2(1 + np.minimum(deg, rng.integers(1, 400, n)))], axis=1).astype(np.float32)
    vtx = rng.choice(n, size=rows, p=deg / deg.sum()).astype(np.int32)
    cls = rng.integers(0, 4, rows).astype(np.uint8)
    x = feats[vtx].astype(np.float64)
    target = (0.3 * (x[:, 2] - x[:, 0]) - 0.1 * x[:, 3] + 0.5 * cls + rng.normal(0, 0.7, rows)).astype(np.float32)
    weight = np.floor(2.0 * (1.0 - rng.random(rows)) ** -0.7).astype(np.float32)
    params = mlp_init(seed, target_mean=float(np.average(target, weights=weight)))
    return feats, vtx, cls, target, weight, params


def prepare(case, seed):
    sess = _session()
    st = _State(case, sess)
    kind = case["kind"]
    st.seed = 1000 + seed
    if kind == "train":
        feats, vtx, cls, target, weight, params = _training_set(case, seed)
        dev = sess.device
        st.feats, st.params = torch.from_numpy(feats).to(dev), torch.from_numpy(params).to(dev)
        st.rows = {"vtx": torch.from_numpy(vtx).to(dev), "cls": torch.from_numpy(cls).to(dev),
                   "target": torch.from_numpy(target).to(dev), "weight": torch.from_numpy(weight).to(dev),
                   "rows": case["rows"]}
        return st
    if "pattern" in case:
        st.pattern = synth.named_pattern(case["pattern"])
    off, nbr = _csr(case, seed)
    if kind == "preprocess":
        st.off, st.nbr = off, nbr
        return st
    st.graph = sess.graph(off, nbr)
    if kind != "clique_dag":
        st.tables = sess.tables(st.graph, cv_seed=1)
    if kind == "targets":
        # row buffers of full capacity, kept by the program
        cap = st.pattern.k * st.graph.n
        st.row_buffers = {k: torch.zeros(cap, dtype=d, device=sess.device)
                          for k, d in (("vtx", torch.int32), ("cls", torch.uint8), ("target", torch.float32),
                                       ("weight", torch.float32))}
    if kind == "tables":
        st.params = torch.from_numpy(mlp_init(seed, target_mean=0.25)).to(sess.device)
    return st


# ---------------------------------------------------------------- one pass

def _estimate_out(r):
    return {"estimate": float(r.estimate), "variance": float(r.variance), "n": int(r.n),
            "n_nonzero": int(r.n_nonzero)}


def _tables_out(sess, tables, n):
    dev = sess.device
    out = {k: torch.empty(n, dtype=d, device=dev)
           for k, d in (("deg", torch.int32), ("s2", torch.int64), ("hits", torch.int64), ("trials", torch.int64),
                        ("la", torch.int32), ("lc", torch.int32))}
    agis_tables_export(sess.ctx, tables.handle, **{k: t.data_ptr() for k, t in out.items()})
    return out


def run(st):
    case, sess = st.case, st.sess
    kind = case["kind"]
    if kind == "estimate":
        r = sess.estimate(st.graph, st.tables, st.pattern, case["samples"], st.seed, mode=case["mode"],
                          eps=case["eps"], delta=0.05, check_every=4096 if case["eps"] else 0,
                          min_samples=4096 if case["eps"] else 0)
        return _estimate_out(r)
    if kind == "concentrations":
        c = sess.concentrations(st.graph, st.tables, case["k"], case["budget"], st.seed, mode="switch",
                                eps=case["eps"], delta=0.05, check_every=4096, min_samples=4096)
        runs = [_estimate_out(r) for r in c["results"]]
        return {**{k: np.array([r[k] for r in runs]) for k in runs[0]}, "conc_edge": np.asarray(c["conc_edge"]),
                "conc_induced": np.asarray(c["conc_induced"])}
    if kind == "preprocess":
        graph = sess.graph(st.off, st.nbr)
        tables = sess.tables(graph, cv_seed=1)
        out = _tables_out(sess, tables, graph.n)
        tables.close()
        graph.close()
        return out
    if kind == "clique_dag":
        dag = sess.orient(st.graph)
        tables = sess.tables(dag, cv_seed=1)
        out = _tables_out(sess, tables, dag.n)
        out.update(_estimate_out(sess.estimate(dag, tables, st.pattern, case["samples"], st.seed, mode="switch")))
        tables.close()
        dag.close()
        return out
    if kind == "targets":
        sums, counts = sess.learn_targets(st.graph, st.tables, st.pattern, case["samples"], st.seed, mode="switch")
        base = sess.step_log_weights(st.tables, st.pattern)
        mask = sum(1 << i for i in sess.weighted_steps(st.pattern))
        b = st.row_buffers
        count = agis_learn_rows(sess.ctx, sums.data_ptr(), counts.data_ptr(), st.pattern.k, st.graph.n, mask, 2,
                                b["vtx"].data_ptr(), b["cls"].data_ptr(), b["target"].data_ptr(),
                                b["weight"].data_ptr(), base.data_ptr())
        return {"sums": sums, "counts": counts, "rows": int(count), **b}
    if kind == "train":
        params = st.params.clone()
        losses = sess.mlp_train(params, st.feats, st.rows, epochs=case["epochs"], batch=max(case["rows"], 4096),
                                lr=3e-3, seed=st.seed)
        return {"params": params, "losses": np.asarray(losses)}
    feats = sess.features(st.tables)
    base = sess.step_log_weights(st.tables, st.pattern)
    tabs = sess.learned_tables(st.params, feats, st.pattern, base=base)
    return {"feats": feats, "tables": [tabs[i] for i in sorted(tabs)]}


# ---------------------------------------------------------------- references

def exact(case, seed):
    """The training pass in 64 bits.  The other kinds return whole numbers,
    statistics of the library's own sample stream, or features of sampled
    quantities, which have no value apart from the library's definitions."""
    if case["kind"] != "train":
        return None
    feats, vtx, cls, target, weight, params = _training_set(case, seed)
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    f64 = dict(dtype=torch.float64, device=dev)
    onehot = np.zeros((case["rows"], 4))
    onehot[np.arange(case["rows"]), np.minimum(cls, 3)] = 1.0
    x = torch.tensor(np.concatenate([feats[vtx].astype(np.float64), onehot], axis=1), **f64)
    y, w = torch.tensor(target.astype(np.float64), **f64), torch.tensor(weight.astype(np.float64), **f64)
    w = w / w.sum()
    p = torch.tensor(params.astype(np.float64), **f64)
    m, v = torch.zeros_like(p), torch.zeros_like(p)
    sizes = (HIDDEN * INPUTS, HIDDEN, HIDDEN * HIDDEN, HIDDEN, HIDDEN, 1)
    losses = []
    for step in range(1, case["epochs"] + 1):
        q = p.clone().requires_grad_(True)
        w1, b1, w2, b2, w3, b3 = torch.split(q, sizes)
        h = torch.nn.functional.gelu(x @ w1.view(HIDDEN, INPUTS).T + b1)
        h = torch.nn.functional.gelu(h @ w2.view(HIDDEN, HIDDEN).T + b2)
        loss = (w * (h @ w3 + b3 - y) ** 2).sum()
        (g,) = torch.autograd.grad(loss, q)
        losses.append(float(loss.detach()))
        m = 0.9 * m + 0.1 * g
        v = 0.999 * v + 0.001 * g * g
        p = p - 3e-3 * (m / (1 - 0.9 ** step)) / (torch.sqrt(v / (1 - 0.999 ** step)) + 1e-8)
    return {"params": p, "losses": np.array(losses)}


def work(case):
    """Bytes and operations of one pass that no implementation can avoid."""
    kind = case["kind"]
    n = case["n"] if "n" in case else case.get("vertices", 1 << case.get("scale", 0))
    slots = 2 * case["m"] if "m" in case else 30 * n
    csr = 8 * (n + 1) + 4 * slots
    if kind == "estimate":
        # per sample and step: a row's two offsets and one neighbour, and the
        # ten rounds of the random block (some 100 integer operations)
        k = synth.named_pattern(case["pattern"]).k
        samples = case["samples"] if not case["eps"] else 4096
        return {"bytes": 20 * k * samples, "flops": 100 * k * samples}
    if kind == "concentrations":
        patterns = {3: 2, 4: 6, 5: 21}[case["k"]]
        return {"bytes": 20 * case["k"] * 4096 * patterns, "flops": 100 * case["k"] * 4096 * patterns}
    if kind == "preprocess":
        # the graph in, six table columns out; per slot one trial (two draws)
        return {"bytes": csr + 36 * n, "flops": 200 * slots}
    if kind == "clique_dag":
        k = synth.named_pattern(case["pattern"]).k
        return {"bytes": csr + 8 * (n + 1) + 2 * slots + 36 * n + 20 * k * case["samples"],
                "flops": 100 * slots + 100 * k * case["samples"]}
    if kind == "targets":
        k = synth.named_pattern(case["pattern"]).k
        return {"bytes": 12 * k * n + 20 * k * case["samples"], "flops": 100 * k * case["samples"]}
    if kind == "train":
        macs = HIDDEN * INPUTS + HIDDEN * HIDDEN + HIDDEN
        return {"bytes": 29 * case["rows"] + 8 * agis_mlp_param_count(),
                "flops": 6 * macs * case["rows"] * case["epochs"]}
    # features from the graph (16 bytes each), then per weighted step its log
    # weights and its table
    pattern = synth.named_pattern(case["pattern"])
    plan = agis_compile_pattern(make_pattern(pattern.k, pattern.adj8()), params=make_params(mode="learned"))
    steps = sum(1 for i in range(pattern.k) if plan.decision[i] and plan.f1[i] > 0)
    return {"bytes": csr + 16 * n + 8 * steps * n,
            "flops": steps * 2 * (HIDDEN * INPUTS + HIDDEN * HIDDEN + HIDDEN) * n}

"""Workloads of the design library that its speed is judged by.

Each case is one call (or one short stream of calls) of the public Python binding with inputs of
the kind the tests and the benchmark use: synthetic proteins (Met, uniform residues, stop), the
seeded codon table and the T04-shaped parameter file.  Inputs are host strings by nature: a pass
takes them through the whole call, from protein to mRNA and structure.

A program keeps one context for its designs (and one server for its request stream), so the
module does too.  The library's schedule tuners explore on the first calls of a size class;
`prepare` runs a new class's first calls until its schedule has settled, once per process, as a
long-running program has.
"""
import math

import numpy as np
import torch  # noqa: F401  (before the library, so that both use one HIP runtime)

import paper_2609_32308_amd as sd
import sdinputs as S

# automaton states per residue and cells per state pair of uniform synthetic proteins
STATES_PER_AA = 3.29


def listed():
    return [
        # a peptide tag: the smallest call, where launches and fixed costs count
        dict(name="plain_12", kind="plain", aa=12, lam=4.0),
        # a short protein, the size most parity tests run
        dict(name="plain_50", kind="plain", aa=50, lam=4.0),
        # an ordinary protein, designed on its own
        dict(name="plain_300", kind="plain", aa=300, lam=0.0),
        # a long protein (the shorter of the two long benchmark lengths)
        dict(name="plain_925", kind="plain", aa=925, lam=4.0),
        # a very long protein (the longer of the two)
        dict(name="plain_1976", kind="plain", aa=1976, lam=0.0),
        # a handful of variants designed together: a batch far too small to fill the chip
        dict(name="batch_7", kind="batch", members=7, lo=50, hi=150),
        # a library of proteins in one batched call, the benchmark's length law at a quarter of its count
        dict(name="batch_64", kind="batch", members=64, lo=50, hi=1000),
        # a burst of requests through the continuous-batching server
        dict(name="served_24", kind="served", members=24, lo=50, hi=500),
        # a design that avoids an inventory of 16 restriction-site-like 6-mers
        dict(name="motifs_105", kind="motifs", aa=105, motifs=16, lam=4.0),
        # a short design that avoids a few sites
        dict(name="motifs_31", kind="motifs", aa=31, motifs=5, lam=0.0),
        # the supported lambda envelope of a short protein: many small batched calls in a row
        dict(name="envelope_40", kind="envelope", aa=40, hi=8.0),
        # one gradient and one prediction of the learned sizer on its training log (FP32)
        dict(name="sizer_1800", kind="sizer", samples=1800),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["plain", "plain", "plain", "noalloc", "batch", "batch", "served", "motifs", "envelope", "sizer"])
    lam = rng.choice([0.0, 4.0, round(rng.uniform(0.1, 8.0), 2)])
    if kind == "plain":
        return dict(kind=kind, aa=_log(rng, 6, 1976), lam=lam)
    if kind == "noalloc":  # the same design without device allocation (up to about 500 aa)
        return dict(kind=kind, aa=_log(rng, 6, 450), lam=lam)
    if kind == "batch":
        lo = _log(rng, 10, 100)
        return dict(kind=kind, members=_log(rng, 2, 60), lo=lo, hi=_log(rng, lo + 10, 900))
    if kind == "served":
        lo = _log(rng, 20, 100)
        return dict(kind=kind, members=_log(rng, 3, 40), lo=lo, hi=_log(rng, lo + 10, 500))
    if kind == "motifs":
        return dict(kind=kind, aa=_log(rng, 15, 105), motifs=rng.randint(1, 16), lam=lam)
    if kind == "envelope":
        return dict(kind=kind, aa=_log(rng, 10, 60), hi=round(rng.uniform(2.0, 8.0), 2))
    return dict(kind=kind, samples=_log(rng, 16, 2000))


class _Kept:
    """What a program keeps for its lifetime: handles, one context, one server, settled classes."""

    def __init__(self):
        self.params = sd.Params(S.default_params_path())
        self.table = sd.CodonTable(S.codon_weights(2026))
        self.ctx = sd.Context(0)
        self.settled = set()
        self._server = None

    @property
    def server(self):
        if self._server is None:
            self._server = sd.Server(sd.Context(0), self.table, self.params)
        return self._server


_kept = None


def _keep():
    global _kept
    if _kept is None:
        _kept = _Kept()
    return _kept


def _lengths(case):
    """Log-uniform member lengths, the case's own (the seed draws the residues)."""
    return S.batch_lengths(case["members"], case["lo"], case["hi"], 7)


def _size_class(case, st):
    """The library tunes per floor log2 of the (mean) length in nucleotides and of the member count."""
    lens = [len(p) for p in st["proteins"]]
    n = 3.0 * sum(lens) / len(lens)
    return case["kind"], int(math.log2(n)), min(4, int(math.log2(len(lens))))


def prepare(case, seed):
    k = _keep()
    kind = case["kind"]
    st = {"case": dict(case), "kept": k}
    if kind == "sizer":
        st["X"], st["Y"], weights = _sizer_inputs(case, seed)
        st["sizer"] = sd.Sizer(k.ctx, 64, 8)
        st["sizer"].set_params(weights)
        return st
    if kind in ("batch", "served"):
        st["proteins"] = [S.protein(a, seed * 1000 + i) for i, a in enumerate(_lengths(case))]
        m = len(st["proteins"])
        st["lams"] = [0.0 if i < m // 2 else 4.0 for i in range(m)]
    else:
        st["proteins"] = [S.protein(case["aa"], seed)]
    if kind == "motifs":
        for j in range(100):  # an inventory that leaves the protein a coding sequence
            ms = S.motifs(case["motifs"], seed * 100 + j)
            try:
                sd.motif_lattice_size(st["proteins"][0], ms)
            except sd.SDError:
                continue
            st["motifs"] = ms
            break
    if kind == "served":
        st["server"] = k.server
    if kind in ("plain", "batch", "envelope"):
        cls = _size_class(case, st)
        for _ in range(12):
            if cls in k.settled:
                break
            if all(r.sched_tuned for r in _results(st)):
                k.settled.add(cls)
    return st


def _results(st):
    case, k = st["case"], st["kept"]
    kind = case["kind"]
    if kind == "plain":
        return [k.ctx.design(st["proteins"][0], k.table, k.params, case["lam"])]
    if kind == "noalloc":
        return [k.ctx.design_noalloc(st["proteins"][0], k.table, k.params, case["lam"])]
    if kind == "batch":
        return k.ctx.design_batch(st["proteins"], st["lams"], k.table, k.params)
    if kind == "served":
        tickets = [st["server"].submit(p, l) for p, l in zip(st["proteins"], st["lams"])]
        return [st["server"].wait(t) for t in tickets]
    if kind == "motifs":
        return [k.ctx.design_motifs(st["proteins"][0], st["motifs"], k.table, k.params, case["lam"])]
    designs, st["breaks"] = k.ctx.lambda_envelope(st["proteins"][0], 0.0, case["hi"], k.table, k.params)
    return designs


def run(st):
    if st["case"]["kind"] == "sizer":
        loss, grad = st["sizer"].gradient(st["X"], st["Y"])
        return {"grad": grad, "loss": np.float32(loss), "yhat": st["sizer"].predict(st["X"])}
    rs = _results(st)
    whole = lambda name: np.array([getattr(r, name) for r in rs], np.int64)  # noqa: E731
    real = lambda name: np.array([getattr(r, name) for r in rs], np.float64)  # noqa: E731
    text = lambda name: np.frombuffer("".join(getattr(r, name) for r in rs).encode(), np.uint8)  # noqa: E731
    if "breaks" in st:  # as many designs as the inputs have: in arrays of the call's capacity
        whole, real, text = (lambda name, f=f: _padded(f(name)) for f in (whole, real, text))
    out = {name: whole(name) for name in ("energy", "objective_fixed", "fixed_shift", "n_states", "n_cells",
                                          "n_candidates", "n_visits", "n_feasible")}
    out.update({name: real(name) for name in ("codon_cost", "objective_kcal", "cai")})
    out.update({name: text(name) for name in ("mrna", "structure")})
    if "breaks" in st:
        out["breaks"] = _padded(np.array(st["breaks"], np.float64))
    return out


def _padded(a):
    """Zeros after the envelope's values, up to its largest number of designs (64)."""
    size = 65 if a.dtype != np.uint8 else 64 * 3 * 60
    return np.concatenate([a, np.zeros(size - len(a), a.dtype)])


def work(case):
    """Per design cell the four values that later cells and the traceback read (one typed closed
    value, the branch value, two multiloop fragments), written once; a few tens of additions and
    comparisons per cell (one per total loop length and multiloop term)."""
    kind = case["kind"]
    if kind == "sizer":
        n, params = case["samples"], 22 * 64 + 64 + 64 * 64 + 64 + 64 * 8 + 8
        return {"bytes": 4 * (n * (22 + 8 + 8) + 2 * params), "flops": 2 * n * params * 4}
    if kind in ("batch", "served"):
        lo, hi = math.log(case["lo"]), math.log(case["hi"])
        sq = case["members"] * (math.exp(2 * hi) - math.exp(2 * lo)) / (2 * (hi - lo))  # E[A^2], A log-uniform
    elif kind == "envelope":
        sq = 24 * case["aa"] ** 2  # about two dozen optima along the search
    elif kind == "motifs":
        # the product with the matcher holds more states (16 6-mers: about 2.7 times as many)
        sq = (case["aa"] * (1 + 0.106 * case["motifs"])) ** 2
    else:
        sq = case["aa"] ** 2
    cells = STATES_PER_AA ** 2 * sq / 2
    return {"bytes": 32 * cells, "flops": 80 * cells}


def _sizer_inputs(case, seed):
    """Occupancy-log rows (log length, residue fractions, lambda / 4), their targets (small
    fractions) and the network's parameters (22 -> 64 -> 64 -> 8)."""
    n = case["samples"]
    rng = np.random.default_rng([seed, 17])
    aa = np.rint(np.exp(rng.uniform(math.log(50), math.log(2000), n)))
    X = np.empty((n, 22), np.float32)
    X[:, 0] = np.log(aa) / math.log(2000)
    X[:, 1:21] = rng.multinomial(aa.astype(np.int64), [0.05] * 20) / aa[:, None]
    X[:, 21] = rng.integers(0, 2, n)
    Y = rng.uniform(0.01, 0.25, (n, 8)).astype(np.float32)
    parts = []
    for fan_out, fan_in in ((64, 22), (64, 64), (8, 64)):
        lim = math.sqrt(6.0 / (fan_in + fan_out))
        parts += [rng.uniform(-lim, lim, fan_out * fan_in), rng.uniform(-0.05, 0.05, fan_out)]
    return X, Y, np.concatenate(parts).astype(np.float32)


def exact(case, seed):
    """The sizer's loss, gradient and prediction in 64 bits.  The designs' optima and strings are
    whole numbers and bytes; their real-valued figures follow from the chosen design, and a
    dense lattice DP in numpy takes minutes per protein: None."""
    if case["kind"] != "sizer":
        return None
    X, Y, w = (v.astype(np.float64) for v in _sizer_inputs(case, seed))
    at, mats = 0, []
    for fan_out, fan_in in ((64, 22), (64, 64), (8, 64)):
        W = w[at:at + fan_out * fan_in].reshape(fan_out, fan_in)
        at += fan_out * fan_in
        mats.append((W, w[at:at + fan_out]))
        at += fan_out
    (W1, b1), (W2, b2), (W3, b3) = mats
    h1 = np.maximum(X @ W1.T + b1, 0.0)
    h2 = np.maximum(h1 @ W2.T + b2, 0.0)
    y = 1.0 / (1.0 + np.exp(-(h2 @ W3.T + b3)))
    loss = np.mean((y - Y) ** 2)
    d3 = 2.0 * (y - Y) / Y.size * y * (1.0 - y)
    d2 = (d3 @ W3) * (h2 > 0)
    d1 = (d2 @ W2) * (h1 > 0)
    grad = np.concatenate([(d1.T @ X).ravel(), d1.sum(0), (d2.T @ h1).ravel(), d2.sum(0), (d3.T @ h2).ravel(), d3.sum(0)])
    return {"grad": grad, "loss": np.float64(loss), "yhat": y}

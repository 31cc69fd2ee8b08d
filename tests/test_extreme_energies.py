"""Parameter sets whose entries reach the parser's limits, at weights of the codon cost that fill the
fixed-point range: every finite DP value lies within 2^60, and so does every partial sum of a loop that a
kernel compares (the minima over biased bit patterns need values above -2^60; the motif-constrained
step takes values from 2^60 on for infinite).  On the CPU from the oracle's dense tables; on the device
tables and designs against the oracle, exactly."""
import re

import numpy as np
import pytest

import oracle as O
import sdinputs as S
from tests.test_fixed_point import energy_bound, max_codon_costs, parse_params, shift_rule

LIMIT = 1 << 60
INITS = ("hairpin", "bulge", "interior")
SEEDS = range(8)


def write_extreme(path, seed):
    """Random magnitudes per table, from nothing to the largest entry a file may hold."""
    rng = np.random.default_rng(900 + seed)
    ps = S.synthetic_params(seed=900 + seed)

    def draw(size, most):
        m = min(most, int(rng.choice([0, 60, 3000, 100000])))
        sign = int(rng.integers(3))  # negative, positive, both
        return rng.choice([[-m, -m, 0], [0, m, m], [-m, 0, m]][sign], size)

    arrays = {k: draw(np.shape(a), 32767 if k in ("int21", "int22") else 100000) for k, a in ps.arrays.items()}
    i = np.tril_indices(6, -1)
    arrays["stack"][i] = arrays["stack"].T[i]
    for k in ("ML_closing", "ML_intern", "ML_base", "TerminalAU", "Ninio", "NinioMax"):
        ps.scalars[k] = int(draw(None, 100000))
    ps.arrays.update({k: a for k, a in arrays.items() if k not in INITS})
    text = S.params_text(ps)
    for k, lo in zip(INITS, (3, 1, 2)):  # (the writer has no negative initiation)
        text = re.sub(rf"\[{k}\] 31\n[^\[]*", f"[{k}] 31\n" + " ".join(["INF"] * lo + [str(v) for v in arrays[k][lo:]]) + "\n", text)
    with open(path, "w") as fh:
        fh.write(text)


def partial_terms(par):
    """What a kernel adds to an inner value before a loop is whole, by the value it is added to."""
    A, sc, _ = par
    mm = [A["mismatch_interior"], A["mismatch_interior_23"], A["mismatch_interior_1n"]]
    both, au = [], (0, sc["TerminalAU"])
    for l1 in range(1, 30):
        for l2 in range(1, 31 - l1):
            base = A["interior"][l1 + l2] + min(sc["NinioMax"], abs(l1 - l2) * sc["Ninio"])
            X = 2 if 1 in (l1, l2) else 1 if l1 + l2 == 5 else 0
            both += [base + min(mm[X]), base + max(mm[X])]
    closed = [v for m in mm for v in (min(m), max(m))] + both + list(au) + [A["bulge"][l] + a for l in range(2, 31) for a in au]
    return closed, [sc["ML_closing"] + sc["ML_intern"]]


def filling_lambda(p, w, par):
    """The largest lambda of a shift some steps below the one at 0: the codon costs fill the range."""
    target = max(16, shift_rule(p, w, par, 0.0) - 8)
    lo, hi = 0.0, 1.0
    while (s := shift_rule(p, w, par, hi)) is not None and s >= target:
        lo, hi = hi, hi * 2
    for _ in range(50):
        mid = 0.5 * (lo + hi)
        s = shift_rule(p, w, par, mid)
        lo, hi = (mid, hi) if s is not None and s >= target else (lo, mid)
    return lo


@pytest.mark.parametrize("seed", SEEDS)
def test_partial_sums_inside_the_range(seed, weights, tmp_path):
    path = str(tmp_path / "extreme.par")
    write_extreme(path, seed)
    par, P = parse_params(path), O.Params(path)
    closed, multi = partial_terms(par)
    # a single term is no larger than a whole loop may be
    n = 1000
    assert max(map(abs, closed + multi)) * (n // 2) <= max(-energy_bound(par, n)[0], energy_bound(par, n)[1])
    for A in (8, 26):
        p = S.protein(A, 10 + seed)
        lam_full = filling_lambda(p, weights, par)
        for lam in (0.0, 4.0, lam_full):
            d = O.design(p, weights, P, lam, tables=True)
            s = d.fixed_shift
            assert s == shift_rule(p, weights, par, lam)
            if lam == lam_full:
                e_lo, e_hi = energy_bound(par, 3 * A)
                assert sum(max_codon_costs(p, weights, lam, s)) + max(-e_lo, e_hi) * 2 ** s > LIMIT * 0.999
            for key, terms in (("V", closed), ("D2", multi), ("B", [0]), ("D1", [0]), ("X", [0])):
                t = d.tables[key]
                fin = t[t < (1 << 61)]
                lo, hi = (int(fin.min()), int(fin.max())) if fin.size else (0, 0)
                assert -LIMIT < lo + min(0, *terms) * 2 ** s, (key, lam)
                assert hi + max(0, *terms) * 2 ** s < LIMIT, (key, lam)


@pytest.mark.gpu
@pytest.mark.parametrize("seed", SEEDS)
def test_designs_match_the_oracle(seed, weights, tmp_path):
    import paper_2609_32308_amd as sd
    path = str(tmp_path / "extreme.par")
    write_extreme(path, seed)
    par, P = parse_params(path), O.Params(path)
    gp, gt = sd.Params(path), sd.CodonTable(weights)
    c = sd.Context(0)

    def same(r, d):
        assert (r.energy, r.objective_fixed, r.mrna, r.structure) == (d.energy, d.objective_fixed, d.mrna, d.structure)

    p, q = S.protein(26, 10 + seed), S.protein(16, 10 + seed)
    ms = S.motifs(6, seed)
    for lam in (0.0, 4.0, filling_lambda(p, weights, par)):
        print("extreme energies", seed, lam, flush=True)
        d = O.design(p, weights, P, lam, tables=True)
        r, T = c.design_tables(p, gt, gp, lam)
        same(r, d)
        for key, okey in (("V", "V"), ("B", "B"), ("S1", "D1"), ("S2", "D2"), ("X", "X")):
            assert np.array_equal(T[key], d.tables[okey]), key
        dq = O.design(q, weights, P, lam)
        for r, d in zip(c.design_batch([p, q], [lam, lam], gt, gp), (d, dq)):
            same(r, d)
        d = O.design_motifs(q, weights, P, lam, ms, tables=True)
        r, T = c.design_motifs_tables(q, ms, gt, gp, lam)
        same(r, d)
        for key, okey in (("V", "V"), ("B", "B"), ("S1", "D1"), ("S2", "D2"), ("X", "X")):
            assert np.array_equal(T[key], d.tables[okey]), key
    c.close()

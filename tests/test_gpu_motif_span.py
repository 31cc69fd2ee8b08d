"""The motif-constrained span step at the edges of its tiles: one state per layer and the widest layers
(sixteen states, more than eight left edges and more than 64 right edges and rows per size, several rounds
of tasks), the shortest designs, and lengths around the window of thirty-three layers.  Every cell of the
tables and the design against the dense oracle (exact)."""
import random

import pytest

import sdinputs as S

pytestmark = pytest.mark.gpu

CASES = [("MW", 2, 1, 0), ("MW", 12, 1, 0), ("GAVTP", 3, 2, 0), ("GAVTP", 4, 2, 1), ("RSL", 11, 8, 1), ("RSL", 12, 32, 1),
         ("LS", 12, 32, 1), ("LS", 20, 32, 1), ("LS", 26, 32, 1), ("LRSVATGP", 26, 40, 1)]


@pytest.mark.parametrize("kind,aa,k,seed", CASES)
def test_tables_and_designs(kind, aa, k, seed, params_path, weights, oparams):
    import numpy as np
    import oracle as O
    import paper_2609_32308_amd as sd
    gp, gt = sd.Params(params_path), sd.CodonTable(weights)
    rng = random.Random(aa * 7 + len(kind))
    p = "".join(rng.choice(kind) for _ in range(aa))
    ms = S.motifs(k, seed)
    c = sd.Context(0)
    for lam in (0.0, 4.0):
        print("motif span", kind, aa, k, lam, flush=True)
        r, T = c.design_motifs_tables(p, ms, gt, gp, lam)
        d = O.design_motifs(p, weights, oparams, lam, ms, nthreads=8, tables=True)
        assert (r.energy, r.objective_fixed, r.mrna, r.structure) == (d.energy, d.objective_fixed, d.mrna, d.structure)
        assert (r.n_candidates, r.n_visits, r.n_feasible) == (d.n_candidates, d.visits_sparse, d.n_feasible_direct)
        for key, okey in (("V", "V"), ("B", "B"), ("S1", "D1"), ("S2", "D2"), ("X", "X")):
            assert np.array_equal(T[key], d.tables[okey]), key
    c.close()

"""Device traceback on the codon trie: designs whose closing pairs have one and two sources, one and two
states per layer, hairpins of every size class, bulges and interior loops up to the largest sizes, against
the oracle's sequence and structure (exact: ties are broken in one order)."""
import random

import pytest

import sdinputs as S

pytestmark = pytest.mark.gpu


def protein(kind, aa):
    rng = random.Random(1000 * aa + len(kind))
    return "".join(rng.choice(kind) for _ in range(aa))


@pytest.mark.parametrize("kind", ["MW", "RSL", "LRMW", "GAVTP", "KNDEQH"])
@pytest.mark.parametrize("aa", [3, 4, 5, 13, 14, 34, 61])
def test_designs_of_few_residues(kind, aa, params_path, weights, oparams):
    import oracle as O
    import paper_2609_32308_amd as sd
    gp, gt = sd.Params(params_path), sd.CodonTable(weights)
    p = protein(kind, aa)
    c = sd.Context(0)
    for lam in (0.0, 1.0, 60.0):
        d = O.design(p, weights, oparams, lam)
        r = c.design(p, gt, gp, lam)
        assert (r.energy, r.objective_fixed, r.mrna, r.structure) == (d.energy, d.objective_fixed, d.mrna, d.structure)
    c.close()

"""Spans with about as many layer pairs as a tile keeps workgroups resident (256 of sixteen waves, 512 of
eight, 1,024 of four; sixteen pairs per workgroup when every wave takes its own): one item more than a
round holds, and the external column alone in a second round.  Designs against the dense oracle, with
every tile and as a batch of one (whose teams grow as the spans shorten)."""
import pytest

import sdinputs as S

pytestmark = pytest.mark.gpu


def key(r):
    return (r.energy, r.objective_fixed, r.mrna, r.structure, r.n_candidates, r.n_visits, r.n_feasible)


@pytest.mark.parametrize("aa", [85, 86, 171])
def test_tiles_at_residency_edges(aa, params_path, weights, oparams):
    import oracle as O
    import paper_2609_32308_amd as sd
    gp, gt = sd.Params(params_path), sd.CodonTable(weights)
    p, lam = S.protein(aa, 77), 4.0 if aa % 2 else 0.0
    d = O.design(p, weights, oparams, lam)
    ref = None
    for threads, waves in ((64, 0), (256, 0), (512, 0), (1024, 0), (256, 1)):
        print("span tile", aa, threads, waves, flush=True)
        c = sd.Context(0, span_threads=threads, span_item_waves=waves)
        r = c.design(p, gt, gp, lam)
        c.close()
        assert (r.energy, r.objective_fixed, r.mrna, r.structure) == (d.energy, d.objective_fixed, d.mrna, d.structure)
        ref = ref or key(r)
        assert key(r) == ref
    c = sd.Context(0)
    assert key(c.design_batch([p], [lam], gt, gp)[0]) == ref
    c.close()


def test_four_wave_tile_past_one_round(params_path, weights):
    # 342 residues: 1,026 pairs in the first span, two more than the chip holds four-wave workgroups
    import paper_2609_32308_amd as sd
    gp, gt = sd.Params(params_path), sd.CodonTable(weights)
    p = S.protein(342, 78)
    ks = []
    for threads, waves in ((256, 0), (512, 0), (256, 1)):
        print("span tile", threads, waves, flush=True)
        c = sd.Context(0, span_threads=threads, span_item_waves=waves)
        ks.append(key(c.design(p, gt, gp, 4.0)))
        c.close()
    assert ks[0] == ks[1] == ks[2]

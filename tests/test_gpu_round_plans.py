"""Round 0 as a launch of its own, and the plans of later rounds, at the sizes where their code paths change."""
import pytest

import synth
from oracle import csv_oracle as O

from ._harness import Case

pytestmark = pytest.mark.gpu


# several rows per wave of round 0, the widest rows, seed prefixes of one and of several clusters,
# indexes around 1024 and 4096 clusters, prefixes of more than 256 rows, plans that open up to 512 clusters (a
# list of them) and more, softmax prefixes settled by the bounds' class and by their digits
@pytest.mark.parametrize("V,d,C,B,k,eps,comb,noise,mix,split", [
    (4000, 520, 20, 64, 20, 1e-4, O.COMBINE_ALL, 0.05, "single", 1), (4000, 520, 17, 100, 20, 1e-4, O.COMBINE_ALL, 0.05, "mix", 1),
    (3000, 8192, 40, 33, 10, 1e-3, O.COMBINE_ANY, 0.05, "mix", 1), (6000, 72, 1500, 5, 40, 1e-5, O.COMBINE_ALL, 0.5, "mix", 1),
    (6000, 72, 1500, 5, 40, 1e-5, O.COMBINE_ALL, 0.5, "mix", 1000), (6000, 264, 1023, 9, 30, 1e-3, O.COMBINE_ALL, 2.0, "mix", 1),
    (9000, 136, 4096, 3, 64, 1e-3, O.COMBINE_ALL, 0.05, "mix", 1), (9000, 64, 4104, 2, 20, 1e-3, O.COMBINE_ALL, 0.05, "mix", 1),
    (5000, 264, 300, 6, 20, 1e-6, O.COMBINE_ALL, 0.05, "single", 1), (5000, 16, 1, 5, 1, 1e-3, O.COMBINE_ALL, 0.05, "single", 1)])
def test_round_plans_match_the_oracle(V, d, C, B, k, eps, comb, noise, mix, split):
    r = synth.small_recipe(f"plan{V}_{d}_{C}", V=V, d=d, C=C, B=B, steps=2, k=k, eps=eps, h_mode=mix, iso_frac=0.25, row_noise=noise)
    case = Case(r, seed=7, K_cap=V)
    case.ws.set_tail_split(split)
    t = case.run_steps(case.hidden(), k, eps, V, comb, f"plans V={V} d={d} C={C} B={B}", max_rounds=4)
    assert not t.mismatch, "\n".join(t.mismatch[:5])
    case.close()

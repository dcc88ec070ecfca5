"""Round 0 as a launch of its own, and the plans of later rounds, at the sizes where their code paths change."""
import pytest

import synth
from oracle import csv_oracle as O

from ._harness import Case, log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


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


def test_later_rounds_in_every_launch_form():
    """Steps with a round after round 1 and no fallback, repeated: first the single tail kernel, then rounds 0 and 1 as launches with the tail kernel for
    the rest, then (that kernel has met a round) all rounds as launches.  Every form gives the bits of the fixed one-launch-per-phase form."""
    r = synth.small_recipe("ladder-forms", V=6000, d=136, C=60, B=1, steps=60, k=8, eps=2e-3, h_mode="mix", sizes="zipf", row_noise=2.0)
    case = Case(r, seed=21, K_cap=6000, want_W64=False)
    csv, dh = case.csv, case.csv.bits_to_device(case.hidden())

    def step(ws, s, K_max):
        buf = csv.make_step_buffers(case.gidx, 1, r.k, r.eps, K_max, max_rounds=6, delta_clusters=2, relax=True)
        csv.csv_decode_step(ws, case.gidx, dh[s], buf)
        torch.cuda.synchronize()
        return [x.cpu() for x in (buf.ids, buf.logits, buf.lse, buf.flags, buf.n_rows, buf.n_clusters, buf.rounds)]

    case.ws.set_tail_split(1)
    late = []
    for K_max in (600, 1500, 3000, 4500):
        for s in range(60):
            want = step(case.ws, s, K_max)
            if int(want[6][0]) > 2 and not int(want[3][0]) & csv.FLAG_FALLBACK:
                late.append((s, K_max, want))
    assert late, "no step with a later round and no fallback among the inputs"
    for s, K_max, want in late[:6]:
        ws = csv.CsvWorkspace(case.gidx, 1, 6000)                  # no history: the step is the single kernel first
        for i in range(12):
            got = step(ws, s, K_max)
            assert all(torch.equal(x, y) for x, y in zip(got, want)), (s, K_max, i)
        ws.free()
    case.close()


def _launches(csv, ws, idx, h, buf):
    """Kernels that a step of this workspace is made of at this moment: nodes of its captured graph, which is not run."""
    import ctypes
    hip, graph, n, s = csv.lib, ctypes.c_void_p(), ctypes.c_size_t(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        assert hip.hipStreamBeginCapture(ctypes.c_void_p(s.cuda_stream), 2) == 0          # hipStreamCaptureModeRelaxed
        csv.csv_decode_step(ws, idx, h, buf)
        assert hip.hipStreamEndCapture(ctypes.c_void_p(s.cuda_stream), ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0 and hip.hipGraphDestroy(graph) == 0
    return n.value


def test_a_later_round_and_a_fallback_in_the_tail_kernel_after_round_1():
    """Sequences that are certified in round 0 and in round 1, that need a later round and that fall back, in one step: run by the tail kernel after rounds 0 and
    1 had launches of their own, it gives the bits of the form with a launch per phase.  Then the later rounds are launched for a while."""
    rounds = 6
    r = synth.small_recipe("ladder-batch", V=6000, d=136, C=60, B=1, steps=120, k=8, eps=2e-3, h_mode="mix", sizes="zipf", row_noise=2.0, iso_frac=0.1)
    case = Case(r, seed=21, K_cap=6000, want_W64=False)
    csv, dh = case.csv, case.csv.bits_to_device(case.hidden())[:, 0]

    def step(ws, h, K_max):
        buf = csv.make_step_buffers(case.gidx, h.shape[0], r.k, r.eps, K_max, max_rounds=rounds, delta_clusters=2, relax=True)
        csv.csv_decode_step(ws, case.gidx, h, buf)
        torch.cuda.synchronize()
        return buf, [x.cpu() for x in (buf.ids, buf.logits, buf.lse, buf.flags, buf.n_rows, buf.n_clusters, buf.rounds)]

    alone = csv.CsvWorkspace(case.gidx, 120, 6000)
    alone.set_tail_split(1)
    for K_max in (1500, 3000, 4500, 2200, 3700, 600):
        got = step(alone, dh, K_max)[1]
        fell, n = (got[3] & csv.FLAG_FALLBACK) != 0, got[6]
        kinds = [torch.nonzero(x)[:, 0][:2] for x in (~fell & (n == 1), ~fell & (n == 2), ~fell & (n > 2), fell)]
        log(f"K_max {K_max}: {[int((x).sum()) for x in (~fell & (n == 1), ~fell & (n == 2), ~fell & (n > 2), fell)]} sequences by kind")
        if all(k.numel() == 2 for k in kinds):
            break
    else:
        pytest.fail("no limit at which there are sequences of every kind")
    mixed, calm = dh[torch.cat(kinds)].contiguous(), dh[kinds[1].repeat(4)].contiguous()
    want = step(alone, mixed, K_max)[1]
    ws = csv.CsvWorkspace(case.gidx, 8, 6000)
    buf = step(ws, calm, K_max)[0]
    fused = _launches(csv, ws, case.gidx, calm, buf)
    for _ in range(4):
        step(ws, calm, K_max)
    split = _launches(csv, ws, case.gidx, calm, buf)
    assert split > fused
    got = step(ws, mixed, K_max)[1]                                # no fallback and no later round so far: both in the tail kernel
    assert all(torch.equal(x, y) for x, y in zip(got, want))
    for _ in range(20):                                            # the fallback is forgotten after 15 steps
        step(ws, calm, K_max)
    assert _launches(csv, ws, case.gidx, calm, buf) == split + 2 * (rounds - 2)
    assert all(torch.equal(x, y) for x, y in zip(step(ws, mixed, K_max)[1], want))
    alone.free()
    ws.free()
    case.close()

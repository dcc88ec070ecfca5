"""The work this library is used for, as cases that can be timed: decode steps, dense logits, bounds and index builds.

A case is a dict of plain values; `prepare` makes what a serving program holds before the call (an index of a clustered
output head, a workspace, hidden states, output buffers), `run` is one pass through the public entry points.  Heads and
hidden states follow the recipe of `synth/` (planted clusters; rows = centre + small noise, hidden states near one
centre, near a mixture of up to three, or isotropic), drawn on the GPU from the seed.
"""
import math

import numpy as np
import torch

import paper_2511_21702_amd as csv

CENTER_SCALE, ROW_NOISE, BIAS_STD, H_NORM = 4.0, 0.05, 0.1, 8.0


def _case(name, op, V, d, C, B=1, k=50, eps=1e-3, sizes="equal", h="single", iso=0.0, index="plain", steps=1,
          max_rounds=0, delta=0, top_p=0.0, iters=0):
    c = {"op": op, "V": V, "d": d, "C": C}
    if op == "build":
        c.update(sizes=sizes, iters=iters)
    else:
        c.update(B=B, sizes=sizes, h=h, iso=iso, index=index)
    if op == "step":
        c.update(k=k, eps=eps, steps=steps, max_rounds=max_rounds, delta=delta, top_p=top_p)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one user decoding on a small head: a chain of two short launches, latency only
        _case("step_b1_small", "step", 32000, 1024, 256, k=10),
        # one user decoding on an ordinary head: the benchmark's own workload
        _case("step_b1", "step", 128256, 4096, 1024),
        # a few users, every size odd, the fallback levels and the certified distribution in use, a top-3 bias table
        _case("step_b3_ragged", "step", 64007, 2056, 601, B=3, k=20, h="mix", index="bias3", max_rounds=4, delta=16, top_p=0.9),
        # a small serving batch, clusters of very unequal sizes, hidden states between several clusters, a strict
        # tolerance: thousands of rows are opened and a few sequences in a hundred fall back; four consecutive steps
        _case("step_b8_zipf", "step", 151552, 5120, 2048, B=8, eps=1e-4, sizes="zipf", h="mix", steps=4),
        # a serving batch on a large vocabulary with many small clusters: a second round for every sequence
        _case("step_b32", "step", 256000, 4608, 4096, B=32, k=64),
        # a serving batch on a wide head, a quarter of the sequences fall back to the whole vocabulary
        _case("step_b64_fallback", "step", 128256, 8192, 1024, B=64, eps=1e-4, iso=0.25),
        # the largest batch, fallbacks at the 2 % the adaptive budget aims at
        _case("step_b256", "step", 128256, 4096, 1024, B=256, iso=0.02),
        # dense logits of one sequence (scoring a prompt's last token, checking a step)
        _case("full_b1", "full", 128256, 4096, 1024),
        # dense logits of a batch
        _case("full_b32", "full", 256000, 4608, 4096, B=32),
        # cluster bounds alone, bf16 centroids, a prefill-sized group of hidden states
        _case("bounds_b16_bf16", "bounds", 151552, 5120, 4096, B=16, index="bf16"),
        # index build of a small head: a few Lloyd iterations from the default seeds, metadata exported for saving
        _case("build_small", "build", 32000, 1024, 256, iters=4),
        # index build of an ordinary head
        _case("build", "build", 128256, 4096, 1024, iters=8),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges; sizes odd as often as not (d stays a multiple of 8)."""
    op = rng.choices(["step", "full", "bounds", "build"], [12, 3, 2, 3])[0]
    while True:
        V, d = _log_int(rng, 24000, 256000), 8 * _log_int(rng, 96, 1024)
        if V * d <= 256000 * 4608:
            break
    C = _log_int(rng, 100, 4096)
    C = max(64, min(C, V // 24))
    sizes = rng.choice(["equal", "equal", "zipf"])
    if op == "build":
        V, d, C = min(V, 128256), min(d, 4096), min(C, 1024)
        return _case(None, op, V, d, C, sizes=sizes, iters=rng.randint(0, 8))
    B = _log_int(rng, 1, 256) if op == "step" else _log_int(rng, 1, 64)
    index = rng.choice(["plain", "plain", "plain", "bf16", "bias3", "angular"])
    iso = rng.choice([0.0, 0.0, 0.02, 0.25])
    h = rng.choice(["single", "single", "mix"])
    if op != "step":
        return _case(None, op, V, d, C, B=B, sizes=sizes, h=h, iso=iso, index=index)
    levels = rng.random() < 0.25
    return _case(None, op, V, d, C, B=B, k=rng.choice([1, 5, 10, 20, 40, 50, 64, 100]), eps=rng.choice([1e-2, 1e-3, 1e-3, 1e-4]), sizes=sizes, h=h,
                 iso=iso, index=index, steps=rng.choice([1, 1, 2]), max_rounds=4 if levels else 0, delta=16 if levels else 0,
                 top_p=rng.choice([0.0, 0.0, 0.9]))


# ------------------------------------------------------------------------------------------------ inputs
def _sizes(c, gen):
    """Rows per planted cluster, summing to V: equal, or Zipf(1.1) with at least eight rows, shuffled over cluster ids."""
    V, C = c["V"], c["C"]
    if c["sizes"] == "equal":
        n = np.full(C, V // C, np.int64)
        n[:V % C] += 1
        return n
    w = np.arange(1, C + 1, dtype=np.float64) ** -1.1
    n = np.maximum(8, np.floor(V * w / w.sum())).astype(np.int64)
    over, i = int(n.sum()) - V, 0
    if over < 0:
        n[0] -= over
    while over > 0:
        take = min(over, int(n[i]) - 8)
        n[i] -= take
        over -= take
        i += 1
    return n[torch.randperm(C, generator=gen, device="cuda").cpu().numpy()]


def _head(c, gen):
    """(W bf16 [V,d], b float32 [V], planted labels int32 [V] on the host, unit centres [C,d])"""
    V, d, C = c["V"], c["d"], c["C"]
    centers = torch.randn(C, d, generator=gen, device="cuda") * (CENTER_SCALE / math.sqrt(d))
    n = torch.from_numpy(_sizes(c, gen)).cuda()
    label = torch.repeat_interleave(torch.arange(C, device="cuda"), n)[torch.randperm(V, generator=gen, device="cuda")]
    b = torch.randn(V, generator=gen, device="cuda") * BIAS_STD
    W = torch.empty(V, d, dtype=torch.bfloat16, device="cuda")
    for lo in range(0, V, 16384):
        hi = min(V, lo + 16384)
        x = torch.randn(hi - lo, d, generator=gen, device="cuda").mul_(ROW_NOISE / math.sqrt(d))
        W[lo:hi] = x.add_(centers[label[lo:hi]])
    return W, b, label.to(torch.int32).cpu().numpy(), torch.nn.functional.normalize(centers, dim=1)


def _hidden(c, n, centers, gen):
    """Hidden states bf16 [n,d] of norm 8 before rounding."""
    d, C = c["d"], c["C"]
    g = torch.nn.functional.normalize(torch.randn(n, d, generator=gen, device="cuda"), dim=1)
    if c["h"] == "single":
        a = centers[torch.randint(C, (n,), generator=gen, device="cuda")]
    else:                               # one to three centres with Dirichlet(1/2) weights
        ids = torch.rand(n, C, generator=gen, device="cuda").topk(3, dim=1).indices
        m = torch.randint(1, 4, (n, 1), generator=gen, device="cuda")
        w = torch.randn(n, 3, generator=gen, device="cuda").square() * (torch.arange(3, device="cuda") < m)
        a = torch.nn.functional.normalize((w[:, :, None] * centers[ids]).sum(1), dim=1)
    v = 0.9 * a + 0.1 * g
    iso = torch.rand(n, 1, generator=gen, device="cuda") < c["iso"]
    return (torch.nn.functional.normalize(torch.where(iso, g, v), dim=1) * H_NORM).to(torch.bfloat16)


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    W, b, labels, centers = _head(case, gen)
    if case["op"] == "build":
        return {"case": case, "W": W, "b": b}
    kind = case["index"]
    idx = csv.csv_build_index(W, b, case["C"], init_labels=labels, centroid_bf16=kind == "bf16",
                              bias_table_m=3 if kind == "bias3" else 0, spherical=kind == "angular")
    del W
    B, K = case["B"], case["V"] // 4
    ws = csv.CsvWorkspace(idx, B, K)
    T = case.get("steps", 1)
    h = _hidden(case, T * B, centers, gen).reshape(T, B, case["d"])
    s = {"case": case, "idx": idx, "ws": ws, "h": [h[t] for t in range(T)]}
    if case["op"] == "step":
        s["buf"] = [csv.make_step_buffers(idx, B, case["k"], case["eps"], K, max_rounds=case["max_rounds"], delta_clusters=case["delta"],
                                          want_dist=case["top_p"] > 0, top_p=case["top_p"]) for _ in range(T)]
    elif case["op"] == "full":
        s["out"] = torch.empty(B, case["V"], dtype=torch.float32, device="cuda")
    return s


def run(s):
    op = s["case"]["op"]
    if op == "step":
        out = []
        for h, buf in zip(s["h"], s["buf"]):
            csv.csv_decode_step(s["ws"], s["idx"], h, buf)
            out.append([buf.ids, buf.logits, buf.lse, buf.flags, buf.n_rows, buf.n_clusters, buf.rounds, buf.probs, buf.cum, buf.nucleus])
        return out
    if op == "full":
        return csv.csv_full_logits(s["ws"], s["idx"], s["h"][0], s["out"])
    if op == "bounds":
        return csv.csv_bounds(s["ws"], s["idx"], s["h"][0])
    idx = csv.csv_build_index(s["W"], s["b"], s["case"]["C"], iters=s["case"]["iters"])
    meta = idx.export()                 # what a program saves next to the weights
    idx.free()
    return meta


# ------------------------------------------------------------------------------------------------ work and tolerance
def work(case):
    """Bytes and operations of one pass that no implementation can do without.

    Steps: the centroids once a step, the rows of the clusters the sequences open first (distinct ones), and the whole of
    W once where some sequence is expected to fall back.  What mixtures open beyond that depends on the data and is not
    counted, so this is a lower bound for them."""
    V, d, C = case["V"], case["d"], case["C"]
    if case["op"] == "build":           # per assignment: rows and centroids read, labels written; the last pass lays W' out
        n = case["iters"] + 1
        return {"bytes": n * (2.0 * V * d + 4.0 * C * d + 8.0 * V) + 4.0 * V * d + 4.0 * C * d, "flops": n * 2.0 * V * C * d}
    B = case["B"]
    if case["op"] == "full":
        return {"bytes": 2.0 * V * d + 4.0 * V + 2.0 * B * d + 4.0 * B * V, "flops": 2.0 * V * d * B}
    cent = (2.0 if case["index"] == "bf16" else 4.0) * C * d + 12.0 * C + 2.0 * B * d
    if case["op"] == "bounds":
        return {"bytes": cent + 4.0 * B * C + 4.0 * B, "flops": 2.0 * C * d * B}
    near = B * (1.0 - case["iso"])
    clusters = C * (1.0 - (1.0 - 1.0 / C) ** near)
    need = max(case["k"], V / C)
    rows = V if B * case["iso"] >= 1 else min(float(V), clusters * need)
    flops = 2.0 * d * (C * B + near * need + (B - near) * V)
    return {"bytes": case["steps"] * (cent + rows * (2.0 * d + 8.0) + B * (8.0 * case["k"] + 24.0)), "flops": case["steps"] * flops}


def tolerance(case):
    """Exact bf16 products summed in float32, compared once with sums in float64 (2-norm, largest): dense logits on matrix
    cores 3.7e-7, 3.0e-6, on the vector units 5e-8, 2.1e-7; bounds 9e-8, 3.9e-7; returned logits and log-sum-exp 5e-8,
    2.0e-7, and up to four times that where they come from matrix cores.  Of the returned ids 0.016 % stood in another
    order at most: logits a unit in the last place apart."""
    if case["op"] == "build":           # means and radii in float64; of the rows between two centroids a few may change sides
        return {"rel": 1e-6, "max": 1e-5, "differ": 0.01}
    if case["op"] == "full":
        return {"rel": 1.5e-6, "max": 1.2e-5}
    if case["op"] == "bounds":
        return {"rel": 4e-7, "max": 2e-6}
    return {"rel": 8e-7, "max": 3e-6, "differ": 0.01}   # one exchange among a few hundred ids

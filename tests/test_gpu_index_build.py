"""Index build kernels at the edges of their tiles and chunks, through the C ABI (the larger shapes and whole Lloyd runs are in test_gpu_parity.py)."""
import numpy as np
import pytest

import synth
from oracle import csv_oracle as O

from ._harness import log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _same_metadata(e, want):
    """n, perm and bias maxima exactly; centroids to one unit in the last place and radii to two (float64 sums, rounded once)."""
    assert np.array_equal(e["n"], want.n) and np.array_equal(e["perm"], want.perm) and np.array_equal(e["bmax"], want.bmax)
    for key, ulps in (("mu", 1), ("R", 2)):
        diff = np.abs(e[key].view(np.int32).astype(np.int64) - getattr(want, key).view(np.int32).astype(np.int64))
        assert diff.max() <= ulps, (key, int(diff.max()))


# 256 x 256 tiles; 128 x 256 tiles in one and in two column blocks; 128 x 128 tiles.  d ends inside a k-block of 32, V and
# C inside a tile; the last cluster repeats the first one's seed (in another column block where there are two) and stays
# empty, because equal distances go to the smaller id.
@pytest.mark.parametrize("V,d,C", [(65000, 72, 250), (3001, 264, 37), (5003, 40, 300), (70001, 32, 101), (257, 8, 3)])
def test_assignment_tiles_recover_planted_clusters(V, d, C):
    import paper_2511_21702_amd as csv
    r = synth.small_recipe("tiles", V=V, d=d, C=C, B=1, steps=1, row_noise=0.01)
    head = synth.make_head(r, seed=5, threads=8)
    first = np.array([int(np.flatnonzero(head["labels"] == c)[0]) for c in range(C)] + [int(np.flatnonzero(head["labels"] == 0)[0])], dtype=np.int32)
    log(f"assignment V={V} d={d} C={C + 1}")
    g = csv.csv_build_index(csv.bits_to_device(head["W_bits"]), torch.from_numpy(head["b"]).cuda(), C + 1, init_rows=first, iters=0)
    want = O.build_index(head["W_bits"], head["b"], head["labels"], C + 1)
    assert want.n[C] == 0
    _same_metadata(g.export(), want)
    g.free()


# Cluster sizes around a chunk of 128 rows (and around several), empty clusters at both ends, V around a wave's 512 tokens, columns around
# a block's 512, C around the 64 clusters of a scan block and the largest C.
@pytest.mark.parametrize("sizes,d", [([0, 1, 127, 128, 129, 0, 255, 256, 257, 3000, 0], 520), ([512], 8), ([511], 512), ([200, 313], 1032),
                                     ([3] * 63, 16), ([5] * 64 + [0], 16), ([4] * 65, 24), ([1] * 8000 + [0] * 191 + [700], 8)])
@pytest.mark.parametrize("spherical", [False, True])
def test_layout_and_centroids_from_labels(sizes, d, spherical):
    import paper_2511_21702_amd as csv
    C, V = len(sizes), sum(sizes)
    rng = np.random.default_rng(V + d)
    labels = rng.permutation(np.repeat(np.arange(C, dtype=np.int32), sizes))
    W = synth.f32_to_bf16_bits(rng.normal(0, 1, (V, d)).astype(np.float32))
    b = rng.normal(0, 0.1, V).astype(np.float32)
    log(f"layout V={V} d={d} C={C} spherical={spherical}")
    g = csv.csv_build_index(csv.bits_to_device(W), torch.from_numpy(b).cuda(), C, init_labels=labels, iters=0, spherical=spherical)
    e = g.export()
    if not spherical:
        _same_metadata(e, O.build_index(W, b, labels, C))
    else:
        want = O.build_index_angular(W, b, labels, C)
        assert np.array_equal(e["n"], want.n) and np.array_equal(e["perm"], want.perm) and np.array_equal(e["bmax"], want.bmax)
        assert np.abs(e["mu"] - want.mu).max() <= 2.0 ** -23                     # unit directions, float64 sums rounded once
    # the gathered copy: dense logits of a one-hot hidden state are one column of W plus the bias, in token order
    ws = csv.CsvWorkspace(g, 1, max(1, V // 4))
    h = np.zeros((1, d), np.uint16)
    h[0, d - 3] = 0x3F80                                                         # 1.0
    out = csv.csv_full_logits(ws, g, csv.bits_to_device(h)).cpu().numpy()[0]
    assert np.array_equal(out, synth.bf16_bits_to_f32(W)[:, d - 3] + b)
    ws.free()
    g.free()


def test_a_row_that_is_not_finite_leaves_no_finite_radius():
    """The infinite row's distance to its (infinite) centroid is not a number, the other rows' are infinite: the radius is the former."""
    import paper_2511_21702_amd as csv
    V, d, C = 600, 64, 3
    rng = np.random.default_rng(7)
    labels = np.arange(V, dtype=np.int32) % C
    W = synth.f32_to_bf16_bits(rng.normal(0, 1, (V, d)).astype(np.float32))
    W[301, 5] = 0x7F80                                                           # +inf, in cluster 1
    log("radius of a cluster with an infinite row")
    g = csv.csv_build_index(csv.bits_to_device(W), None, C, init_labels=labels, iters=0)
    R = g.export()["R"]
    assert np.isnan(R[1]) and np.isfinite(R[[0, 2]]).all()
    g.free()


# The most partial sums for the rows: clusters one row past a chunk, among clusters without partial sums; then one cluster with all the rows.
@pytest.mark.parametrize("sizes", [[129] * 70, [128, 129] * 40 + [1, 0, 130], [16385], [0, 1] * 30 + [9000]])
@pytest.mark.parametrize("iters", [0, 1])
def test_partial_centroid_sums_fit_their_slots(sizes, iters):
    import paper_2511_21702_amd as csv
    C, V, d = len(sizes), sum(sizes), 40
    # CHUNK_ROWS and PART_SLOTS of the library
    assert sum(-(-n // 128) for n in sizes if n > 128) <= V // 128 + V // 129 + 1
    labels = np.random.default_rng(V).permutation(np.repeat(np.arange(C, dtype=np.int32), sizes))
    centers = np.random.default_rng(d).normal(0, 1, (C, d)).astype(np.float32)
    W = synth.f32_to_bf16_bits(centers[labels] + np.random.default_rng(C).normal(0, 0.01, (V, d)).astype(np.float32))
    b = np.zeros(V, np.float32)
    log(f"partial sums V={V} C={C} iters={iters}")
    g = csv.csv_build_index(csv.bits_to_device(W), torch.from_numpy(b).cuda(), C, init_labels=labels, iters=iters)
    if min(sizes) or not iters:                  # (an empty cluster has no planted centre to be found again)
        _same_metadata(g.export(), O.build_index(W, b, labels, C))
    g.free()


def _labels(e):
    labels = np.empty(e["perm"].size, np.int64)
    labels[e["perm"]] = np.repeat(np.arange(e["n"].size), e["n"])
    return labels


def _nearest(W, mu, labels, tol):
    """Every row's label is a nearest centroid of mu in float64, up to tol * ||row|| * largest ||mu_c|| of score."""
    W, mu, n = W.double(), torch.from_numpy(mu).cuda().double(), torch.from_numpy(labels).cuda()
    d2 = (mu * mu).sum(1) - 2.0 * W @ mu.T
    over = d2.gather(1, n[:, None])[:, 0] - d2.min(1).values
    assert (over <= tol * W.norm(dim=1) * mu.norm(dim=1).max()).all(), over.max().item()


# Heads large enough for the rounded centroids to come first (384 clusters, V d C of 20e9), in most of which they are given up at the first look, so that the
# exact product makes the labels: 256 x 256 and 128 x 256 tiles, d a multiple of 64 and not, V and C inside a tile.  "shared": a planted centre's rows are
# dealt to one to three clusters, whose centroids then differ in the noise, and some clusters hold two centres; "crowd": one centre's rows are dealt to 90
# clusters besides; "alike": all rows equal (every score ties, the smallest id wins).  Two scores that float32 sums of exact products can tell apart are
# told apart right: within the error of a sum with d / 8 roundings to 2^-24 (the exact product has 3 d / 8; a third of the tolerance at the most has been seen).
@pytest.mark.parametrize("V,d,C,spherical", [(70001, 264, 1200, False), (70001, 264, 1200, True), (16000, 3200, 400, False), (45003, 1096, 500, False)])
@pytest.mark.parametrize("kind", ["shared", "crowd", "alike"])
def test_rounded_centroids_find_the_nearest(V, d, C, kind, spherical):
    import paper_2511_21702_amd as csv
    assert C >= 384 and V * d * C >= 20e9                      # assign_near_pays of the library
    gen = torch.Generator(device="cuda").manual_seed(V + d)
    rng = np.random.default_rng(V)
    centers = torch.randn(C, d, device="cuda", generator=gen) * (4.0 / d ** 0.5)
    labels = rng.integers(0, C, V).astype(np.int32)
    labels[:C] = np.arange(C)
    centre = labels // 3 * 3 if kind != "alike" else labels * 0
    centre = np.where((labels % 7 == 0) & (rng.random(V) < 0.5), (labels + C // 2) % C, centre)
    if kind == "crowd":
        centre = np.where(labels < 90, 5, centre)
    W = centers[torch.from_numpy(centre).cuda().long()]
    if kind != "alike":
        W = W + torch.randn(V, d, device="cuda", generator=gen) * (0.05 / d ** 0.5)
    else:
        W = W[:1].expand(V, d)
    W = W.to(torch.bfloat16).contiguous()
    log(f"rounded centroids V={V} d={d} C={C} {kind} spherical={spherical}")
    tol = 2.0 * (d / 8 + 16) * 2.0 ** -24
    g0 = csv.csv_build_index(W, None, C, init_labels=labels, iters=0, spherical=spherical)
    mu = g0.export()["mu"]
    g0.free()
    for iters in (1, 2):
        g = csv.csv_build_index(W, None, C, init_labels=labels, iters=iters, spherical=spherical)
        e = g.export()
        g.free()
        got = _labels(e)
        if kind == "alike":
            assert (got == 0).all()
            break
        if spherical:                                            # largest cosine: every direction counts as of length one
            m = torch.from_numpy(mu).cuda().double()
            dots = W.double() @ m.T
            over = dots.max(1).values - dots.gather(1, torch.from_numpy(got).cuda()[:, None])[:, 0]
            assert (over <= tol * W.double().norm(dim=1)).all(), over.max().item()
        else:
            _nearest(W, mu, got, tol)
        if (e["n"] == 0).any():                                  # an empty cluster keeps a centroid that the export does not show
            break
        mu = e["mu"]


# The same from seed rows: the first assignment's centroids are bf16 values and need no second look, the second's norms come from it.  A row with an infinity
# and one with a NaN get some label and disturb no other row's.
def test_first_assignment_from_rows_then_rounded_centroids():
    import paper_2511_21702_amd as csv
    V, d, C = 70001, 264, 1200
    gen = torch.Generator(device="cuda").manual_seed(3)
    W = (torch.randn(C, d, device="cuda", generator=gen)[torch.arange(V, device="cuda") % C] * (4.0 / d ** 0.5)
         + torch.randn(V, d, device="cuda", generator=gen) * (2.0 / d ** 0.5)).to(torch.bfloat16)
    first = np.arange(C, dtype=np.int32)
    log("first assignment from rows")
    tol, mu, want = 2.0 * (d / 8 + 16) * 2.0 ** -24, W[:C].float().cpu().numpy(), None
    for iters in (0, 1, 2):
        g = csv.csv_build_index(W, None, C, init_rows=first, iters=iters)
        e = g.export()
        g.free()
        want = _labels(e)
        _nearest(W, mu, want, tol)
        assert e["n"].min() > 0
        mu = e["mu"]
    W2 = W.clone()
    W2[60000, 5] = float("inf")
    W2[60001, 263] = float("nan")
    g = csv.csv_build_index(W2, None, C, init_rows=first, iters=0)
    once = _labels(g.export())
    g.free()
    g = csv.csv_build_index(W, None, C, init_rows=first, iters=0)
    clean = _labels(g.export())
    g.free()
    keep = np.ones(V, bool)
    keep[60000:60002] = False
    assert np.array_equal(once[keep], clean[keep])
    g = csv.csv_build_index(W2, None, C, init_rows=first, iters=2)
    e = g.export()
    g.free()
    assert sorted(e["perm"].tolist()) == list(range(V)) and e["n"].sum() == V


@pytest.mark.parametrize("V,seed_value", [(700, 4.0), (700, np.inf), (40000, 4.0)])                # 128 and 256 rows a tile
def test_sums_that_overflow_still_find_the_nearest(V, seed_value):
    """Finite rows whose products with a seed row overflow float32: minus infinity is the nearest, plus infinity farther than every finite score.  A row with
    a value that is not finite is nearest to none (the smallest id), a seed row with one is nobody's nearest."""
    import paper_2511_21702_amd as csv
    d, C = 264, 5
    W = np.zeros((V, d), np.float32)
    W[0, 0], W[1, 0], W[2, 1], W[4, 2] = 1e19, -1e19, 1.0, 8.0                   # seeds; ||1e19||^2 is finite
    W[3, 3], W[3, 4] = seed_value, 1.0
    kind = np.arange(V) % 4
    kind[:C] = -1
    W[kind == 0, 0], W[kind == 1, 0], W[kind == 2, 1], W[kind == 3, 2] = 1e20, -1e20, 2.0, 7.0
    W[100, 9], W[101, 260] = -np.inf, np.nan
    want = np.choose(np.maximum(kind, 0), [0, 1, 2, 4])
    want[:C] = [0, 1, 2, 3 if np.isfinite(seed_value) else 0, 4]
    want[100:102] = 0
    log(f"sums that overflow, seed {seed_value}")
    g = csv.csv_build_index(csv.bits_to_device(synth.f32_to_bf16_bits(W)), None, C, init_rows=np.arange(C, dtype=np.int32), iters=0)
    got = _labels(g.export())
    g.free()
    assert np.array_equal(got, want), np.flatnonzero(got != want)[:8]


def _both_ways(W, labels, C, iters, spherical=False):
    """Labels of the rows of W after `iters` iterations from the given labels (None: from the first C rows), found with rounded centroids first and with the exact product alone: the head
    once over is too small for the former, the same rows twice over, whose clusters have the same means, are not.  Bit for bit the same."""
    import paper_2511_21702_amd as csv
    V, d = W.shape
    assert C >= 384 and V * d * C < 20e9 <= 2 * V * d * C                         # assign_near_pays of the library
    out = []
    for n in (1, 2):
        start = {"init_rows": np.arange(C, dtype=np.int32)} if labels is None else {"init_labels": np.tile(labels, n)}
        g = csv.csv_build_index(torch.cat([W] * n), None, C, iters=iters, spherical=spherical, **start)
        out.append(_labels(g.export()))
        g.free()
    assert np.array_equal(out[1][:V], out[1][V:])
    bad = np.flatnonzero(out[0] != out[1][:V])
    assert bad.size == 0, (bad.size, bad[:8], out[0][bad[:8]], out[1][bad[:8]])
    return out[0]


def _planted(V, d, C, rng, gen, centre_of=lambda labels: labels, labels=None):
    """Rows around the centres that centre_of gives their labels; every cluster has a row.  (W bf16 on the device, labels)"""
    if labels is None:
        labels = rng.integers(0, C, V).astype(np.int32)
        labels[:C] = np.arange(C)
    centers = torch.randn(C, d, device="cuda", generator=gen) * (4.0 / d ** 0.5)
    noise = torch.randn(V, d, device="cuda", generator=gen) * (0.05 / d ** 0.5)
    return (centers[torch.from_numpy(centre_of(labels)).cuda().long()] + noise).to(torch.bfloat16).contiguous(), labels


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_a_centroid_that_is_not_finite_either_way(value):
    V, d, C = 24000, 520, 1500
    gen = torch.Generator(device="cuda").manual_seed(11)
    W, labels = _planted(V, d, C, np.random.default_rng(11), gen)
    W[7000, 13] = value
    log(f"a centroid of {value}")
    _both_ways(W, labels, C, 1)


def test_sums_that_drift_apart():
    """Products that move a float32 sum by a little less than half a unit each with the centroid's bf16 pieces and by a little more with the rounded centroid:
    d / 8 units apart in the end, which outweighs all else that the rounding leaves out.  The exact product's label is found all the same."""
    V, d, C = 3000, 16384, 384
    W = torch.zeros(V, d)
    W[:, 0] = 1.0
    labels = np.zeros(V, np.int32)
    x = torch.full((d,), 2.0 ** -7)
    x[:8] = 0.0
    x[:2] = 1.0
    # centroid 0: a quarter above the bf16 value 2^-20 by three quarters of its last bit, so that a group of eight products with x adds 2^-24 (the tie: 1 stays
    # 1) and 0.75 2^-31 (lost) by pieces, 2^-24 (1 + 2^-7) rounded (1 goes up by 2^-23)
    W[0:4, 8:] = 2.0 ** -20 * (1 + 2.0 ** -7)
    W[3, 8:] = 2.0 ** -20
    W[4:8, 1] = 2.0 ** -14                                                       # centroid 1: exactly representable, a score lower by 2^-13 than 0's
    labels[4:8] = 1
    W[8:208], W[8:108] = -3.0 * x, x                                             # the rows in question, from a cluster with mean -x
    labels[8:208] = 2
    rest = torch.arange(208, V)
    labels[208:] = 3 + (np.arange(208, V) - 208) % (C - 3)
    W[rest, 0] = 0.0
    W[rest, 8 + torch.from_numpy(labels[208:]).long()] = 8.0                     # far away
    log("sums that drift apart")
    got = _both_ways(W.to(torch.bfloat16).cuda(), labels, C, 1)
    assert (got[8:108] == 1).all()                                               # by pieces; the float64 sum lies between the two


def test_a_centroid_norm_that_rounds_by_the_order_of_its_sum():
    """||mu||^2 = 1 + 2^-24 and six terms of 2^-54, which in some orders are lost one by one in float64 and in others lift the sum over the float32 tie.  The
    score of centroid 0 is -1 or -1 + 2^-23, of centroid 1 exactly -1: the label must not depend on which kernel took the norm."""
    V, d, C = 24000, 520, 1500
    W = torch.zeros(V, d)
    labels = (np.arange(V) % C).astype(np.int32)
    far = torch.arange(V)
    W[far, 8 + torch.from_numpy(labels % 512).long()] = 8.0 * (1 + torch.from_numpy(labels // 512).float())
    W[labels == 0] = 0.0
    W[labels == 1] = 0.0
    W[labels == 0, 0] = W[labels == 1, 0] = 1.0
    W[labels == 0, 1] = 2.0 ** -12
    W[labels == 0, 2:8] = 2.0 ** -27
    log("a norm that rounds by the order of its sum")
    _both_ways(W.to(torch.bfloat16).cuda(), labels, C, 1)


def _second_look(W, labels, C, spherical, copies):
    """What the first look at the rounded scores finds, in float64: rows by the centroids in reach, pairs, and the cost that decides whether it is given up."""
    V, d = W.shape
    x, lab = W.double(), torch.from_numpy(labels).cuda().long()
    norm = x.norm(dim=1)
    rows = x / norm[:, None] if spherical else x
    mu = torch.zeros(C, d, dtype=torch.float64, device="cuda").index_add_(0, lab, rows)
    mu = (mu / mu.norm(dim=1, keepdim=True) if spherical else mu / torch.bincount(lab, minlength=C)[:, None]).float().double()
    near = mu.float().to(torch.bfloat16).double()
    left = 2.0 * ((mu - near).norm(dim=1) + (0.501 * d + 64.0) * 2.0 ** -24 * mu.norm(dim=1))       # round_centroids_kernel of the library
    low = (1.0 if spherical else (mu * mu).sum(1)) - 2.0 * x @ near.T - norm[:, None] * left
    reach = low <= (low + 2.0 * norm[:, None] * left).min(1, keepdim=True).values
    pad = torch.nn.functional.pad(reach, (0, -C % 64)).reshape(V, -1, 64).sum(2)                     # groups of 64 clusters
    size = torch.full((pad.shape[1],), 64, device="cuda")
    size[-1] -= -C % 64
    whole = (pad >= 3).any(1)
    total = torch.where(pad >= 3, size, pad).sum(1)
    n = {"settled": (total == 1) & ~whole, "few": (total > 1) & (total <= 16) & ~whole, "many": (total > 16) & (total <= 160) & ~whole,
         "whole": whole & (total <= 160), "wide": total > 160}                                       # AS_PAIRS_CHEAP, AS_PAIRS_ROW
    n = {k: copies * int(v.sum()) for k, v in n.items()}
    V *= copies
    cap = min(2 * V, V * C // 512)
    few, other = (copies * int(total[m].sum()) for m in ((total > 1) & (total <= 16) & ~whole, whole & (total <= 160) | (total > 16) & (total <= 160)))
    listed = n["wide"] + max(0, few + other - cap) / 2        # a row that finds the list full has two pairs at least
    cost = 0.4 + 6.5e9 / (V * d * C) + 100.0 * min(few + other, cap) / (V * C) + 1.15 * listed / V
    return n, few, cap, cost


# Rows with more than one centroid in reach, found by the exact scores of pairs, of whole groups and of rows with all centroids: the labels are those of the
# exact product, bit for bit.  "few": pairs of clusters, in one group of 64 and in two, share a centre; "many": twenty clusters do, two of a group at most;
# "whole": three of a group do; "wide": two hundred do (rows for all centroids); "full": more pairs than their list holds (the rest of the rows for all
# centroids).  The scratch of the shape with 4096 clusters does not fit into the index's copy of W.
@pytest.mark.parametrize("V,d,C,kind,spherical", [
    (24000, 1064, 750, "few", False), (24000, 1064, 750, "few", True), (24000, 1064, 750, "many", False), (24000, 1064, 750, "whole", False),
    (24000, 1064, 750, "wide", False), (6000, 8192, 400, "few", False), (6000, 8192, 400, "wide", False), (25000, 1992, 400, "full", False),
    (18000, 264, 4096, "few", False), (18000, 264, 4096, "wide", False)])
def test_rows_that_take_a_second_look(V, d, C, kind, spherical):
    import paper_2511_21702_amd as csv
    gen = torch.Generator(device="cuda").manual_seed(V)
    rng = np.random.default_rng(d)
    labels, centre = None, np.arange(C)
    if kind == "few":
        centre[1:32:8], centre[64:96] = centre[0:32:8], centre[0:32]
    elif kind == "many":
        centre[:640].reshape(10, 64)[:, :2] = 0
    elif kind == "whole":
        centre[[1, 2, 65, 66]] = [0, 0, 64, 64]
    elif kind == "wide":
        centre[:200] = 0
        small = np.repeat(np.arange(200, dtype=np.int32), 4)
        labels = np.concatenate([small, 200 + np.arange(V - small.size, dtype=np.int32) % (C - 200)])
    else:
        centre[1:int(0.42 * C):2] = centre[0:int(0.42 * C):2]
    W, labels = _planted(V, d, C, rng, gen, lambda l: centre[l], labels)
    n, pairs, cap, cost = _second_look(W, labels, C, spherical, 2)
    log(f"second look V={V} d={d} C={C} {kind} spherical={spherical}: {n}, {pairs} pairs of {cap}, cost {cost:.2f}")
    assert cost < 0.81 and n["settled"] > V / 2                                   # the rounded centroids are kept (given up: 0.85)
    assert n[{"full": "few"}.get(kind, kind)] > 100 and (pairs > 1.02 * cap) == (kind == "full")
    if C == 4096:
        assert C // 256 * 48 > 2 * d                                              # words a row / its share of the copy of W, bytes
    for iters in (1, 2):
        _both_ways(W, labels, C, iters, spherical)

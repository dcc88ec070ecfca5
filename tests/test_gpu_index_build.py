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

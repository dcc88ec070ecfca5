"""Cluster bounds: batches around the 64 sequences that one block of the batched product carries, and the few sequences that go by rows."""
import numpy as np
import pytest

import synth

from ._harness import Case, log

pytestmark = pytest.mark.gpu


# float32 sums of exact products: the bound's error is far below 1e-5 of |mu| |h| + R |h|
@pytest.mark.parametrize("B,bf16", [(64, False), (65, False), (65, True), (129, False), (256, False)])
def test_batched_bounds_match_float64(B, bf16):
    r = synth.small_recipe(f"bounds{B}", V=3000, d=520, C=75, B=B, steps=1, h_mode="mix", iso_frac=0.5)
    case = Case(r, seed=19, centroid_bf16=bf16, want_W64=False)
    h = case.hidden()[0]
    U = case.csv.csv_bounds(case.ws, case.gidx, case.csv.bits_to_device(h))
    U = (U[0] if isinstance(U, (tuple, list)) else U).double().cpu().numpy()
    h64 = (h.astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    mu, R, bmax = (np.asarray(x, np.float64) for x in (case.oidx.mu, case.oidx.R, case.oidx.bmax))
    hn = np.linalg.norm(h64, axis=1)
    want = h64 @ mu.T + hn[:, None] * R[None, :] + bmax[None, :]
    scale = hn[:, None] * (np.linalg.norm(mu, axis=1) + R)[None, :] + np.abs(bmax)[None, :]
    assert U.shape == want.shape and np.all(np.abs(U - want) <= 1e-5 * scale)
    case.close()


# Up to four sequences, a slice of a centroid row per wave: rows of one slice, of two and four, of a slice and a bit, a whole number of batches of
# loads; clusters that do not fill the last block.  bf16 rows of four sequences on both sides of the 4096 waves from which h goes through LDS.  An entry's error
# is at most that of a float32 sum of d exact products in lanes of d / 64: (d / 64 + 16) 2^-24 of |mu| |h|, and a few roundings of the sum.
@pytest.mark.parametrize("C,d,bf16", [(5, 8, False), (75, 520, False), (33, 1032, False), (131, 2056, False), (9, 4104, False), (70, 8192, False),
                                      (75, 520, True), (33, 4104, True), (1030, 4104, True), (1030, 2056, True), (2050, 2056, True)])
@pytest.mark.parametrize("B", [1, 2, 3, 4])
def test_bounds_of_a_few_sequences(B, C, d, bf16):
    _bounds_match_float64(B, C, d, bf16)


# Up to 16 sequences in one launch: rows shorter than a chunk of 1024 values, of one, of several and a bit; clusters inside a tile of 16; then shapes on the other
# side of the rule, which go by K slices.
@pytest.mark.parametrize("C,d,bf16", [(5, 8, False), (75, 520, False), (33, 1024, False), (131, 1032, False), (16, 2048, False), (3077, 3000, False), (17, 4104, True),
                                      (40, 5120, True), (4200, 1040, True), (131, 2056, False), (20, 8192, True)])
@pytest.mark.parametrize("B", [5, 11, 16, 17])
def test_bounds_of_a_small_batch(B, C, d, bf16):
    _bounds_match_float64(B, C, d, bf16)


def _slices(C, d, B, bf16):
    """(length, number) of the K slices of more than 64 sequences, and the most there may be: bound_mfma_plan of the library."""
    groups, nkb = -(-C // 128), -(-d // 32)
    n = min(-(-256 // groups), 32, nkb)
    most = -(-nkb // min(-(-nkb // (4 * n)) * 4, 12))
    plans = [(-(-groups * -(-nkb // k) * -(-B // 64) // 256) * k * (0.25 if bf16 else 0.5) + 2.2e-6 * -(-nkb // k) * B * C, -k) for k in (4, 8, 12, 16)
             if -(-nkb // k) <= most]
    k = -min(plans)[1]
    return k, -(-nkb // k), most


# More than 64 sequences: slices of 4, 8, 12 and 16 k-blocks, whole and partial last ones, as many as may be and fewer.  The slices' sums are added in
# float32, too, so the tolerance is that of the other batches.
@pytest.mark.parametrize("C,d,B,bf16,length", [(75, 8, 65, False, 4), (301, 1000, 70, False, 4), (1024, 4096, 65, False, 8), (260, 8192, 100, False, 8),
                                               (1031, 4104, 67, True, 12), (500, 4104, 200, False, 12), (1024, 4096, 256, False, 16), (1000, 4000, 250, True, 16)])
def test_bounds_of_many_sequences_by_slice_length(C, d, B, bf16, length):
    k, n, most = _slices(C, d, B, bf16)
    assert k == length and n <= most
    _bounds_match_float64(B, C, d, bf16, static=most * B * C * 4 <= 8 << 20)     # what csv_bounds_static has room for


def _bounds_match_float64(B, C, d, bf16, static=True):
    import paper_2511_21702_amd as csv
    torch = pytest.importorskip("torch")
    gen = torch.Generator(device="cuda").manual_seed(C + d)
    V = 2 * C + 1
    W = (torch.randn(V, d, device="cuda", generator=gen) * (4.0 / d ** 0.5)).to(torch.bfloat16)
    b = torch.randn(V, device="cuda", generator=gen) * 0.1
    labels = np.arange(V, dtype=np.int32) % C
    labels[labels == C // 2] = 0                                       # an empty cluster
    h = (torch.randn(B, d, device="cuda", generator=gen) * (8.0 / d ** 0.5)).to(torch.bfloat16)
    log(f"bounds B={B} C={C} d={d} bf16={bf16}")
    g = csv.csv_build_index(W, b, C, init_labels=labels, centroid_bf16=bf16)
    ws = csv.CsvWorkspace(g, B, V)
    U, hn = csv.csv_bounds(ws, g, h)
    U2, hn2 = torch.empty_like(U), torch.empty_like(hn)
    if static:
        csv.csv_bounds_static(g, h, U2, hn2)
        assert torch.equal(U, U2) and torch.equal(hn, hn2)
    else:
        with pytest.raises(csv.CsvError):
            csv.csv_bounds_static(g, h, U2, hn2)
    e = g.export()
    mu, R, bmax = (np.asarray(e[k], np.float64) for k in ("mu", "R", "bmax"))
    h64 = h.double().cpu().numpy()
    n = np.linalg.norm(h64, axis=1)
    want = h64 @ mu.T + n[:, None] * R[None, :] + bmax[None, :]
    full = e["n"] > 0
    tol = ((d / 64 + 16) * 2.0 ** -24) * n[:, None] * (np.linalg.norm(mu, axis=1) + R)[None, :] + 2.0 ** -22 * np.abs(want)
    got = U.double().cpu().numpy()
    assert np.isneginf(got[:, ~full]).all() and not full.all()
    assert (np.abs(got - want)[:, full] <= tol[:, full]).all()
    assert (np.abs(hn.double().cpu().numpy() - n) <= (d / 64 + 16) * 2.0 ** -24 * n).all()
    ws.free()
    g.free()

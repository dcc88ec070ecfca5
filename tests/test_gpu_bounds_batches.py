"""Cluster bounds of batches around the 64 sequences that one block of the batched product carries."""
import numpy as np
import pytest

import synth

from ._harness import Case

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

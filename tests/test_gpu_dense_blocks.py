"""Dense logits of up to four sequences where a block computes one tile of rows and where it computes several, and around the length that parts short from long rows."""
import numpy as np
import pytest

import synth

from ._harness import log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# d: 255, 256 and 257 pieces of 16 bytes, fewer than one per lane, a last trip that half the lanes make; V: one tile more than there are
# blocks (8 rows a tile, at least 2048 blocks), more than four tiles for each of them, three sequences from 12288 tiles on.
@pytest.mark.parametrize("V,d,B", [(16385, 776, 4), (16393, 2040, 1), (16385, 2048, 4), (20003, 2056, 3), (98305, 264, 3), (98305, 2048, 3),
                                   (131083, 72, 2), (70001, 1288, 4), (65537, 2048, 2)])
def test_dense_logits_by_blocks(V, d, B):
    import paper_2511_21702_amd as csv
    g0 = torch.Generator(device="cuda").manual_seed(V + d + B)
    W = torch.randn(V, d, generator=g0, device="cuda").bfloat16()
    h = torch.randn(B, d, generator=g0, device="cuda").bfloat16()
    b = torch.randn(V, generator=g0, device="cuda")
    labels = np.random.default_rng(V).integers(0, 5, V).astype(np.int32)
    log(f"dense logits V={V} d={d} B={B}")
    g = csv.csv_build_index(W, b, 5, init_labels=labels, iters=0)
    ws = csv.CsvWorkspace(g, B, 1)
    got = csv.csv_full_logits(ws, g, h, torch.full((B, V), float("nan"), dtype=torch.float32, device="cuda")).cpu().double()
    W64, h64, b64 = W.cpu().double(), h.cpu().double(), b.cpu().double()
    # exact products; at most d roundings of float32 sums, and the bias
    bound = (d + 1) * 2.0 ** -24 * (h64.abs() @ W64.abs().T + b64.abs())
    assert bool(((got - (h64 @ W64.T + b64)).abs() <= bound).all())
    ws.free()
    g.free()

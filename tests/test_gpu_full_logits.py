"""Dense logits at the edges of the product's tiles, of its K chunks and of the 64 x 64 tiles that bring the result into token order."""
import numpy as np
import pytest

import synth

from ._harness import log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# Vector product: 1..4 sequences, odd V (a tile's second row missing), rows of fewer pieces than one trip and with a remainder.
# MFMA product: 5.. sequences: sequence counts that are and are not a multiple of four, around 16, 32, 64 and two passes;
# V around a tile of 64 tokens and a group of 256 rows; one K chunk of 256, a ragged last one, several.
@pytest.mark.parametrize("V,d,B", [(1, 8, 1), (65, 2056, 1), (4099, 4096, 2), (1003, 520, 3), (513, 2552, 4),
                                   (63, 8, 5), (64, 256, 8), (65, 264, 15), (257, 512, 16), (3001, 520, 17), (511, 1288, 31), (1025, 256, 32),
                                   (515, 776, 33), (2049, 1032, 64), (700, 264, 65), (129, 2048, 100), (321, 520, 256)])
def test_full_logits_edges(V, d, B):
    import paper_2511_21702_amd as csv
    rng = np.random.default_rng(V + d + B)
    C = min(V, 7)
    W = synth.f32_to_bf16_bits(rng.normal(0, 1, (V, d)).astype(np.float32))
    h = synth.f32_to_bf16_bits(rng.normal(0, 1, (B, d)).astype(np.float32))
    b = rng.normal(0, 1, V).astype(np.float32)
    labels = rng.integers(0, C, V).astype(np.int32)
    log(f"full logits V={V} d={d} B={B}")
    g = csv.csv_build_index(csv.bits_to_device(W), torch.from_numpy(b).cuda(), C, init_labels=labels, iters=0)
    ws = csv.CsvWorkspace(g, B, 1)
    out = torch.full((B, V), float("nan"), dtype=torch.float32, device="cuda")
    got = csv.csv_full_logits(ws, g, csv.bits_to_device(h), out).cpu().numpy().astype(np.float64)
    W64, h64 = synth.bf16_bits_to_f32(W).astype(np.float64), synth.bf16_bits_to_f32(h).astype(np.float64)
    want = h64 @ W64.T + b
    # exact products; at most d roundings of float32 sums, and the bias
    bound = (d + 1) * 2.0 ** -24 * (np.abs(h64) @ np.abs(W64).T + np.abs(b))
    assert (np.abs(got - want) <= bound).all(), float((np.abs(got - want) / bound).max())
    ws.free()
    g.free()

"""The full-vocabulary product: a row's logit has the same bits whatever the launch form, the row's place and its neighbours."""
import numpy as np
import pytest

import synth
from oracle import csv_oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _head(V, d, B, C, seed, k):
    """A random head in which 3 k tokens, spread over the vocabulary, have the same row and bias, and hidden states near that row."""
    rng = np.random.default_rng(seed)
    W = rng.standard_normal((V, d), dtype=np.float32) / np.float32(np.sqrt(d))
    same = np.sort(rng.choice(V, 3 * k, replace=False))
    W[same] = W[same[0]]
    b = rng.normal(0, 0.1, V).astype(np.float32)
    b[same] = 0.25
    h = (4.0 * W[same[0]] + rng.normal(0, 1 / np.sqrt(d), (B, d))).astype(np.float32)
    labels = rng.permutation(np.arange(V) % C).astype(np.int32)
    return synth.f32_to_bf16_bits(W), b, synth.f32_to_bf16_bits(h), labels, same


# V and C such that seven sequences leave the fused launch 151 blocks for the product and the other forms 256, where groups of
# 256 rows suit the one and groups of 128 the other; rows of 4 and 8 KB (their K is cut into four parts), of 16 KB (eight), and of 4.5 KB (none).
@pytest.mark.parametrize("d", [2048, 2304, 4096, 8192])
def test_fallback_logits_do_not_depend_on_the_launch_form(d):
    import paper_2511_21702_amd as csv
    V, C, B, k = 24000, 480, 7, 10
    W, b, h, labels, same = _head(V, d, B, C, d, k)
    g = csv.csv_build_index(csv.bits_to_device(W), torch.from_numpy(b).cuda(), C, init_labels=labels)
    ws = csv.CsvWorkspace(g, B, 1)
    dh = csv.bits_to_device(h)
    got = {}
    for form in (1000, 1):                                          # one resident kernel, one launch per phase
        ws.set_tail_split(form)
        buf = csv.make_step_buffers(g, B, k, 1e-3, 0)               # a budget of no rows: every sequence falls back
        csv.csv_decode_step(ws, g, dh, buf)
        torch.cuda.synchronize()
        assert bool(((buf.flags & O.FLAG_FALLBACK) != 0).all())
        got[form] = {n: getattr(buf, n).cpu().numpy().copy() for n in ("ids", "logits", "lse")}
    dense = csv.csv_full_logits(ws, g, dh).cpu().numpy()
    for n in ("ids", "logits", "lse"):
        assert np.array_equal(got[1000][n].view(np.uint32), got[1][n].view(np.uint32)), n
    for x in got.values():
        assert np.array_equal(np.take_along_axis(dense, x["ids"].astype(np.int64), 1).view(np.uint32), x["logits"].view(np.uint32))
        assert np.array_equal(x["ids"], np.broadcast_to(same[:k], (B, k)))      # 3 k equal logits on top: the smallest ids, ascending
    ws.free()
    g.free()


# one, two and four tiles of 16 sequences, two passes; K of a single chunk, a ragged last one, cut into parts
@pytest.mark.parametrize("V,d,B", [(9000, 256, 8), (9001, 2056, 5), (9001, 2048, 17), (70003, 2048, 33), (33000, 4096, 64), (5003, 6144, 70), (6001, 8192, 40)])
def test_equal_rows_have_equal_logits(V, d, B):
    import paper_2511_21702_amd as csv
    W, b, h, labels, same = _head(V, d, B, 7, V + B, 60)
    g = csv.csv_build_index(csv.bits_to_device(W), torch.from_numpy(b).cuda(), 7, init_labels=labels)
    ws = csv.CsvWorkspace(g, B, 1)
    out = csv.csv_full_logits(ws, g, csv.bits_to_device(h)).cpu().numpy()[:, same].view(np.uint32)
    assert np.array_equal(out, np.broadcast_to(out[:, :1], out.shape)), int((out != out[:, :1]).sum())
    ws.free()
    g.free()

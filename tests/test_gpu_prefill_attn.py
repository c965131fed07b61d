"""Causal prefill attention around the edges of its tiles: 32 positions a wave, 64 tokens a step, up to four heads of a
group (or several position tiles) a workgroup, histories that start anywhere in a page.  Against the oracle's full
recompute, bar as for every logit comparison: max |dlogit| <= 3e-2 x per-row logit std."""
import numpy as np
import pytest

from oracle import decoder as od
from paper_2506_24119_amd import inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q_heads,kv_heads,head_dim,dtype", [
    (2, 2, 128, si.WEIGHT_BF16), (4, 2, 128, si.WEIGHT_BF16), (6, 2, 64, si.WEIGHT_BF16), (5, 1, 128, si.WEIGHT_BF16),
    (7, 1, 64, si.WEIGHT_BF16), (16, 1, 32, si.WEIGHT_BF16), (9, 3, 32, si.WEIGHT_FP32)])
def test_ragged_runs_and_histories(q_heads, kv_heads, head_dim, dtype):
    import torch
    from paper_2506_24119_amd import binding as sb
    g = si.ModelGeometry("attn-edges", 2, 128, q_heads, kv_heads, head_dim, 128, 256, 1e4, qk_norm=head_dim == 128,
                         weight_dtype=dtype)
    w = si.make_weights(g, seed=3)
    rng = np.random.Generator(np.random.PCG64(5))
    first = [1, 31, 33, 63, 65, 129, 200, 16]              # around 32, 64 and the page of 16
    second = [1, 33, 31, 65, 1, 64, 97, 140]
    seqs = [rng.integers(0, g.vocab, a + b).astype(np.int32) for a, b in zip(first, second)]
    ids = np.arange(len(seqs), dtype=np.int32)
    sess = sb.Session(g, sb.weights_to_device(w), 160, len(seqs), 24, 1024, 400, page_order=si.make_page_order(160, 2))
    got = [sess.prefill(ids, [s[:a] for s, a in zip(seqs, first)]).cpu().numpy()]
    got.append(sess.prefill(ids, [s[a:] for s, a in zip(seqs, first)]).cpu().numpy())
    torch.cuda.synchronize()
    sess.close()
    for b, s in enumerate(seqs):
        want = od.forward_full(g, w, s, logits_at=np.array([first[b] - 1, len(s) - 1]))
        for k in range(2):
            ratio = np.abs(got[k][b] - want[k]).max() / want[k].std()
            assert ratio <= 3e-2, (b, k, ratio)

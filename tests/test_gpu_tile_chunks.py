"""Tiled projections over one to eight chunks of 64 k, around the number of LDS slots that their loads run ahead by, on both tile heights,
against the float64 oracle: the scoring LM head (128 rows), whose logits are seen through log-probabilities (tolerance twice the logit bar of
3e-2 x per-row logit std, as in the other scoring tests), and gate/up in a prefill (256 rows; the logit bar)."""
import ctypes as C

import numpy as np
import pytest

from oracle import decoder as od
from oracle import scoring as osc
from paper_2506_24119_amd import inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 130, 600])
@pytest.mark.parametrize("d", [128, 256, 384, 512])
def test_few_chunks_of_k(d, rows):
    import torch
    from paper_2506_24119_amd import binding as sb
    g = si.ModelGeometry("chunks", 1, d, 2, 1, 64, 192, 1100, 1e6, qk_norm=True)       # 1,100 columns: a partly padded last tile
    host = si.make_weights(g, seed=d)
    rng = np.random.Generator(np.random.PCG64(rows))
    n = min(rows, 75)
    seqs = [rng.integers(0, g.vocab, n).astype(np.int32) for _ in range(rows // n)]
    seqs.append(rng.integers(0, g.vocab, rows - n * len(seqs) or 1).astype(np.int32))
    targets = np.concatenate([np.concatenate([s[1:], [-1]]) for s in seqs]).astype(np.int32)
    if rows > 1:
        targets[0] = g.vocab - 1                                    # the last column
    sess = sb.Session(g, sb.weights_to_device(host), 8 * len(seqs), len(seqs), 8, targets.size, 128, page_order=si.make_page_order(8 * len(seqs), 4))
    out = torch.full((targets.size,), 9.0, dtype=torch.float32, device="cuda")
    sb.spiral_score(sess.model, sess.pool, np.arange(len(seqs), dtype=np.int32), [len(s) for s in seqs],
                    torch.from_numpy(np.concatenate(seqs)).cuda(), torch.from_numpy(targets).cuda(), sess.ws, out)
    got = out.cpu().numpy()
    sess.close()
    off = 0
    for s in seqs:
        logits = od.forward_full(g, host, s, logits_at=np.arange(len(s)))
        t = targets[off:off + len(s)]
        want = np.where(t >= 0, osc.log_softmax_rows(logits)[np.arange(len(s)), t], 0.0)
        assert (np.abs(got[off:off + len(s)] - want) <= 6e-2 * logits.std(axis=-1)).all(), (d, rows, off)
        off += len(s)


def _tall_gate_up(d, ffn, n_seqs):
    """Rows enough that the tall tiles of gate/up fill the chip, which is where a d that is no multiple of 128 leaves the general kernel."""
    from paper_2506_24119_amd import binding as sb
    rule = sb.load_library()["_ZN6spiral16gemm_tile_heightEiiiiii"]
    rule.restype, rule.argtypes = C.c_int, [C.c_int] * 6
    g = si.ModelGeometry("chunks", 2, d, 2, 1, 64, ffn, 500, 1e6, qk_norm=True)
    host = si.make_weights(g, seed=3)
    seqs = si.make_prompts(g.vocab, n_seqs, 74, 78, seed=4)
    rows = sum(len(s) for s in seqs)
    assert rule(rows, g.ffn_dim, d, 1, 128, 128) == 256 and rows % 256
    ids = np.arange(n_seqs, dtype=np.int32)
    sess = sb.Session(g, sb.weights_to_device(host), n_seqs * 8, n_seqs, 8, rows, 128, page_order=si.make_page_order(n_seqs * 8, 4))
    got = sess.prefill(ids, seqs).cpu().numpy()
    sess.close()
    for b in (0, n_seqs // 2 - 1, n_seqs - 1):
        want = od.forward_full(g, host, seqs[b], logits_at=np.array([len(seqs[b]) - 1]))[0]
        assert np.abs(got[b] - want).max() <= 3e-2 * want.std(), (d, b)


def test_a_single_chunk_of_k():
    _tall_gate_up(64, 2048, 44)


@pytest.mark.parametrize("d,n_seqs", [(128, 12), (192, 15), (256, 12), (320, 15), (384, 12), (512, 12)])
def test_few_chunks_on_the_tall_tile(d, n_seqs):
    _tall_gate_up(d, 6144, n_seqs)

"""Decode steps on short contexts: a workgroup to a (row, kv head) pair up to 16, 32 or 96 pages (heads narrower than 128; those of 128
go by an estimate beyond 32 pages, see the tests of the rows' order), against the balanced stream (forced by
spiral_model_tune "chunk=") on either side of the rule, and the fp32 step of a few rows whose projections do the norms and the
residual's sums, against the oracle and at the edges of its rows."""
import numpy as np
import pytest

from oracle import decoder as od
from paper_2506_24119_amd import inputs as si

pytestmark = pytest.mark.gpu


def _step(g, w, lens, tune):
    import torch
    from paper_2506_24119_amd import binding as sb
    rng = np.random.Generator(np.random.PCG64(sum(lens)))
    B = len(lens)
    seqs = [rng.integers(0, g.vocab, n + 1).astype(np.int32) for n in lens]
    ids = np.arange(B, dtype=np.int32)
    nb = max(lens) // 16 + 2
    sess = sb.Session(g, w, nb * B + 2, B, nb, max(sum(lens), B), max(lens) + 4,
                      page_order=si.make_page_order(nb * B + 2, 3), tune=tune)
    sess.prefill(ids, [s[:-1] for s in seqs])
    sb.spiral_profile_begin(sess.model, sb.KERNEL_CLASSES.index("attn_combine"), 8)
    out = sess.decode_step(ids, torch.from_numpy(np.array([s[-1] for s in seqs])).cuda(), sess.new_logits(B)).cpu().numpy()
    merges = sb.spiral_profile_end(sess.model)[1]
    sess.close()
    return out, seqs, merges


def _compare(g, host, lens, direct, rows):
    from paper_2506_24119_amd import binding as sb
    w = sb.weights_to_device(host)
    got, seqs, merges = _step(g, w, lens, None)
    assert merges == (0 if direct else g.n_layers)
    stream, _, merges = _step(g, w, lens, "chunk=4")
    assert merges == g.n_layers
    for b in rows:
        want = od.forward_full(g, host, seqs[b], logits_at=np.array([len(seqs[b]) - 1]))[0]
        assert np.abs(got[b] - want).max() <= 3e-2 * want.std(), b
    scale = stream.std(axis=1, keepdims=True)
    assert (np.abs(got - stream) <= 1e-2 * scale).all()


@pytest.mark.parametrize("q_heads,kv_heads,head_dim,dtype", [
    (8, 2, 128, si.WEIGHT_BF16), (7, 1, 64, si.WEIGHT_BF16), (4, 4, 32, si.WEIGHT_BF16), (16, 1, 32, si.WEIGHT_FP32), (6, 2, 128, si.WEIGHT_FP32)])
@pytest.mark.parametrize("longest", [1, 16, 100, 255, 256])
def test_a_workgroup_to_a_pair(q_heads, kv_heads, head_dim, dtype, longest):
    """Contexts of two tokens to 256 (with the step's own; 16 pages), and 257, which few pairs leave to the balanced stream.  The two differ in the
    fp32 merge of the partial results, so by roundings of the half-precision attention output: 2^-11 of a value, in two layers; 1e-2 of the logits'
    deviation is five times what that can add up to over a head's 128 values.  The oracle's bar is the 3e-2 of every logits test."""
    g = si.ModelGeometry("short", 2, 128, q_heads, kv_heads, head_dim, 128, 256, 1e4, weight_dtype=dtype)
    lens = sorted({1, 15, 16, 17, 63, 64, 65, longest} & set(range(1, longest + 1)))
    _compare(g, si.make_weights(g, seed=81), lens, longest <= 255, range(len(lens)))


@pytest.mark.parametrize("longest", [256, 511, 512])
def test_many_pairs(longest):
    """130 pairs: the longest context may have 512 tokens (with the step's own)"""
    g = si.ModelGeometry("short", 2, 128, 4, 2, 64, 128, 256, 1e4)
    lens = [1 + (37 * b) % 90 for b in range(64)] + [longest]
    _compare(g, si.make_weights(g, seed=84), lens, longest <= 511, (0, 31, 64))


@pytest.mark.parametrize("shortest,longest,direct", [(850, 1535, True), (850, 1536, False), (60, 1535, False)])
def test_a_pair_for_every_cu(shortest, longest, direct):
    """264 pairs: 1,536 tokens, where the mean is at least half of the longest"""
    g = si.ModelGeometry("short", 2, 128, 8, 8, 32, 128, 256, 1e4)
    lens = [shortest + (29 * b) % 300 for b in range(32)] + [longest]
    _compare(g, si.make_weights(g, seed=85), lens, direct, (0, 32))


@pytest.mark.parametrize("q_heads,kv_heads,rows,longest,direct", [
    (8, 8, 64, 1100, True), (8, 8, 65, 511, True), (8, 8, 65, 512, False), (24, 8, 128, 1023, True), (32, 8, 65, 1024, False), (32, 8, 65, 1023, True), (24, 8, 128, 1100, False), (32, 8, 81, 1100, True), (32, 8, 79, 1100, False),
    (8, 8, 192, 1100, True)])
def test_a_pair_to_a_workgroup_in_rounds(q_heads, kv_heads, rows, longest, direct):
    """Pairs of a little more than two to a CU 1,024 tokens (512 with fewer than four query heads a pair), with fewer than four query heads up
    to six to a CU 1,024; else 1,536."""
    g = si.ModelGeometry("short", 1, 128, q_heads, kv_heads, 32, 128, 256, 1e4)
    lens = [longest - 300 + (29 * b) % 300 for b in range(rows - 1)] + [longest]
    _compare(g, si.make_weights(g, seed=86), lens, direct, (0, rows - 1))


@pytest.mark.parametrize("d,ffn,norm,B,vocab", [
    (128, 512, False, 1, 260), (128, 512, False, 4, 260), (128, 512, False, 5, 260), (128, 512, False, 32, 260), (128, 512, False, 33, 260),
    (128, 512, False, 32, 1100), (132, 200, True, 8, 260), (132, 200, True, 31, 260), (132, 200, True, 32, 260), (512, 96, False, 8, 260),
    (512, 1280, False, 16, 260), (768, 96, False, 5, 260), (1024, 96, False, 8, 260), (1024, 512, False, 16, 260), (1028, 96, False, 1, 260)])
def test_fp32_projections_that_norm(d, ffn, norm, B, vocab):
    """The last batch the rule takes and the first it leaves, remainders of four rows, widths that are and are not multiples of the 256 elements a
    wave reads at once.  Bar: q, k, v and the attention output round to half, 2^-11 each; all four in the same direction in two layers are 4e-3."""
    from paper_2506_24119_amd import binding as sb
    g = si.ModelGeometry("lean", 2, d, 4, 2, 32, ffn, vocab, 1e4, qk_norm=norm, qkv_bias=not norm, weight_dtype=si.WEIGHT_FP32)
    host = si.make_weights(g, seed=82)
    rng = np.random.Generator(np.random.PCG64(83))
    for lw in host["layers"]:
        for k in ("attn_norm", "mlp_norm"):
            lw[k] = rng.normal(1.0, 0.2, d).astype(np.float32)
    host["final_norm"] = rng.normal(1.0, 0.2, d).astype(np.float32)
    got, seqs, _ = _step(g, sb.weights_to_device(host), [3 + 7 * (b % 9) for b in range(B)], None)
    for b, s in enumerate(seqs):
        want = od.forward_full(g, host, s, logits_at=np.array([len(s) - 1]))[0]
        assert np.abs(got[b] - want).max() <= 4e-3 * want.std(), b


@pytest.mark.parametrize("d,ffn,vocab,B,norms", [
    (128, 512, 1024, 32, 0), (128, 512, 1024, 33, 4), (128, 512, 1028, 32, 1), (128, 512, 8192, 1, 0), (128, 512, 8196, 1, 1), (128, 512, 151936, 4, 1),
    (256, 768, 260, 32, 0), (256, 772, 260, 32, 4), (512, 1280, 260, 16, 0), (512, 1284, 260, 16, 4), (512, 1280, 260, 17, 4),
    (1024, 512, 260, 16, 0), (1028, 96, 260, 1, 4), (132, 200, 260, 32, 0)])
def test_which_fp32_steps_keep_their_norms(d, ffn, vocab, B, norms):
    """By the norm launches of a step of two layers: none, the one before the head, all.  Where every wave of a wide projection norms its
    rows for itself the step is slower (a vocabulary of 151,936, d 128, 32 rows 410 -> 700 us)."""
    import torch
    from paper_2506_24119_amd import binding as sb
    g = si.ModelGeometry("lean", 2, d, 4, 2, 32, ffn, vocab, 1e4, weight_dtype=si.WEIGHT_FP32)
    ids = np.arange(B, dtype=np.int32)
    sess = sb.Session(g, si.make_weights_torch(g, 1, "cuda:0"), B, B, 1, B, 16)
    sess.prefill(ids, [np.zeros(1, dtype=np.int32)] * B)
    sb.spiral_profile_begin(sess.model, sb.KERNEL_CLASSES.index("norm"), 16)
    sess.decode_step(ids, torch.zeros(B, dtype=torch.int32, device="cuda"), sess.new_logits(B))
    assert sb.spiral_profile_end(sess.model)[1] == norms
    sess.close()

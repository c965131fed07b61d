"""Decode attention of a few rows is cut into up to 16 pieces a (row, kv head) pair, down to single pages, with the partial
results in borrowed memory.  Contexts around the page and piece boundaries, one row and a few ragged ones, against the oracle
(bar 3e-2 x per-row logit std) and against the coarse cut (16 pages a workgroup at least): the two differ in the fp32
merge of the pieces, so by roundings of the half-precision attention output - 2^-11 of a value, in two layers; 1e-2 x std is
five times what that can add up to over one head's 128 values.  Contexts of up to 256 tokens are not cut unless "wgs" is set, here
to the number of workgroups that is the default (three to each of 256 CUs)."""
import numpy as np
import pytest

from oracle import decoder as od
from paper_2506_24119_amd import inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens", [[1], [15], [16], [17], [255], [256], [257], [272], [513], [1, 40, 300], [700, 3, 16, 129, 250]])
@pytest.mark.parametrize("dtype", [si.WEIGHT_BF16, si.WEIGHT_FP32])
def test_pieces_match_the_coarse_cut_and_the_oracle(lens, dtype):
    import torch
    from paper_2506_24119_amd import binding as sb
    hd = 128 if dtype == si.WEIGHT_BF16 else 32
    g = si.ModelGeometry("pieces", 2, 256, 8, 2, hd, 256, 512, 1e6, qk_norm=True, weight_dtype=dtype)
    host = si.make_weights(g, seed=21)
    w = sb.weights_to_device(host)
    rng = np.random.Generator(np.random.PCG64(sum(lens)))
    B = len(lens)
    seqs = [rng.integers(0, g.vocab, n).astype(np.int32) for n in lens]
    steps = rng.integers(0, g.vocab, (2, B)).astype(np.int32)
    ids = np.arange(B, dtype=np.int32)
    got = []
    for tune in ("wgs=768", "chunk=16", None):
        sess = sb.Session(g, w, 100, B, 48, max(B, sum(lens)), 720, page_order=si.make_page_order(100, 3), tune=tune)
        sess.prefill(ids, seqs)
        sb.spiral_profile_begin(sess.model, sb.KERNEL_CLASSES.index("attn_combine"), 8)
        got.append([sess.decode_step(ids, torch.from_numpy(s).cuda(), sess.new_logits(B)).cpu().numpy() for s in steps])
        assert sb.spiral_profile_end(sess.model)[1] == (0 if tune is None and max(lens) + 2 <= 256 else 2 if tune is None and max(lens) + 1 <= 256 else 4)
        sess.close()
    for b, s in enumerate(seqs):
        want = od.forward_full(g, host, np.concatenate([s, steps[:, b]]), logits_at=np.array([len(s), len(s) + 1]))
        for k in range(2):
            std = want[k].std()
            for form in (0, 2):
                assert np.abs(got[form][k][b] - want[k]).max() <= 3e-2 * std, (b, k)
                assert np.abs(got[form][k][b] - got[1][k][b]).max() <= 1e-2 * std, (b, k)


@pytest.mark.parametrize("q_heads,kv_heads,head_dim,dtype", [(8, 2, 128, si.WEIGHT_BF16), (6, 3, 64, si.WEIGHT_BF16), (4, 4, 32, si.WEIGHT_FP32)])
@pytest.mark.parametrize("lens", [[257], [700, 3, 16, 129, 250], [15, 16, 17, 512, 513], [300 + 25 * i for i in range(16)], [4200, 100]])
def test_pieces_are_cut_where_the_equal_ranges_are(lens, q_heads, kv_heads, head_dim, dtype):
    """A workgroup to each piece and the equal ranges of the whole batch (which setting "wgs" to its default keeps) add the same partial sums in
    the same order: the same bits, whichever form a batch's size takes.  One row and ragged ones, pairs that start anywhere in a range, pieces of one
    page to 16, and contexts so long that the pieces are not shortened (4,200 tokens)."""
    import ctypes as C
    import torch
    from paper_2506_24119_amd import binding as sb
    g = si.ModelGeometry("pieces", 2, 256, q_heads, kv_heads, head_dim, 256, 512, 1e6, qk_norm=True, weight_dtype=dtype)
    w = sb.weights_to_device(si.make_weights(g, seed=22))
    rng = np.random.Generator(np.random.PCG64(sum(lens)))
    B, blocks = len(lens), max(lens) // 16 + 2
    n_pages = sum(n // 16 + 2 for n in lens)
    rule = sb.load_library()["_ZN6spiral16decode_in_piecesEiiii"]
    rule.restype, rule.argtypes = C.c_bool, [C.c_int] * 4
    pages = [(n + 1 + 15) // 16 for n in lens]
    per = min(16, max((sum(pages) * kv_heads + 767) // 768, (max(pages) + 15) // 16))
    assert rule(sum(pages) * kv_heads, per, B * kv_heads, 768)
    seqs = [rng.integers(0, g.vocab, n).astype(np.int32) for n in lens]
    tok = torch.from_numpy(rng.integers(0, g.vocab, B).astype(np.int32)).cuda()
    ids, got = np.arange(B, dtype=np.int32), []
    for tune in (None, "wgs=768"):
        sess = sb.Session(g, w, n_pages, B, blocks, sum(lens), max(lens) + 4, page_order=si.make_page_order(n_pages, 3), tune=tune)
        sess.prefill(ids, seqs)
        sb.spiral_profile_begin(sess.model, sb.KERNEL_CLASSES.index("attn_combine"), 8)
        got.append(sess.decode_step(ids, tok, sess.new_logits(B)).cpu().numpy())
        assert sb.spiral_profile_end(sess.model)[1] == g.n_layers                # partial results in both
        sess.close()
    assert np.isfinite(got[0]).all() and np.array_equal(got[0], got[1])

"""Projections over more than 128 rows: tiles of 256 x 256 or 128 x 256 or the streaming kernel, K split or not, q/k/v
post-processing inside the projection or behind it - chosen from the shape.  Row counts around the tile heights, on a
geometry whose O and down projections are split; repacked weights must give the bits that row-major ones give, and both
the oracle's logits within the bar of every logit comparison (3e-2 x per-row logit std)."""
import numpy as np
import pytest

from oracle import decoder as od
from paper_2506_24119_amd import inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [129, 255, 257, 520, 900])
@pytest.mark.parametrize("head_dim,q_heads", [(128, 8), (64, 14)])
def test_row_counts_around_the_tiles(rows, head_dim, q_heads):
    import torch
    from paper_2506_24119_amd import binding as sb
    g = si.ModelGeometry("wide", 2, 1024, q_heads, 2, head_dim, 2048, 512, 1e6, qk_norm=head_dim == 128, qkv_bias=head_dim == 64)
    host = si.make_weights(g, seed=11)
    w = sb.weights_to_device(host)
    rng = np.random.Generator(np.random.PCG64(rows))
    lens = [rows - 2 * (rows // 3), rows // 3, rows // 3]
    seqs = [rng.integers(0, g.vocab, n).astype(np.int32) for n in lens]
    step = rng.integers(0, g.vocab, 3).astype(np.int32)
    ids = np.arange(3, dtype=np.int32)
    got = []
    for repack in (True, False):
        sess = sb.Session(g, w, 80, 3, 40, rows, 400, page_order=si.make_page_order(80, 4), repack=repack)
        first = sess.prefill(ids, seqs).cpu().numpy()
        second = sess.decode_step(ids, torch.from_numpy(step).cuda(), sess.new_logits(3)).cpu().numpy()      # reads the appended k, v
        got.append((first, second))
        sess.close()
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
    for b, s in enumerate(seqs):
        want = od.forward_full(g, host, np.concatenate([s, step[b:b + 1]]), logits_at=np.array([len(s) - 1, len(s)]))
        for k in range(2):
            ratio = np.abs(got[0][k][b] - want[k]).max() / want[k].std()
            assert ratio <= 3e-2, (b, k, ratio)


@pytest.mark.parametrize("key", ["o", "down", "qkv"])
def test_tuned_splits_reach_calls_of_many_rows(key):
    """spiral_model_tune "key=R:S" above 128 rows: one and three K splits of a projection add in different orders, so some
    logit differs in its last bits (all of them would be equal if the setting were dropped), and both stay within the bar."""
    from paper_2506_24119_amd import binding as sb
    g = si.ModelGeometry("wide", 2, 1024, 8, 2, 64, 2048, 512, 1e6)
    host = si.make_weights(g, seed=11)
    w = sb.weights_to_device(host)
    seqs = si.make_prompts(g.vocab, 3, 90, 120, seed=8)
    ids = np.arange(3, dtype=np.int32)
    got = []
    for splits in (1, 3):
        sess = sb.Session(g, w, 80, 3, 40, 400, 400, page_order=si.make_page_order(80, 4), tune=f"{key}=128:{splits}")
        got.append(sess.prefill(ids, seqs).cpu().numpy())
        sess.close()
    assert not np.array_equal(got[0], got[1])
    for b, s in enumerate(seqs):
        want = od.forward_full(g, host, s, logits_at=np.array([len(s) - 1]))[0]
        for k in range(2):
            assert np.abs(got[k][b] - want).max() <= 3e-2 * want.std(), (b, k)


def test_fused_qkv_epilogue_at_odd_multiples_of_64():
    """d_model % 128 == 64 (the streaming kernel does not take it): the q/k/v projection does its post-processing itself once
    its tiles fill the chip, an odd number of 64-wide chunks.  Against the two-kernel form: the same order of sums in
    both, so the same bits; and against the oracle."""
    from paper_2506_24119_amd import binding as sb
    g = si.ModelGeometry("k64", 1, 192, 20, 5, 128, 256, 512, 1e6, qk_norm=True)
    host = si.make_weights(g, seed=12)
    w = sb.weights_to_device(host)
    seqs = si.make_prompts(g.vocab, 9, 480, 520, seed=9)
    seqs[0] = seqs[0][:61]
    ids = np.arange(9, dtype=np.int32)
    rows = sum(len(s) for s in seqs)
    assert (rows + 255) // 256 * 15 >= 200 and rows % 128
    got = []
    for tune in ("fuse_qkv=1", "fuse_qkv=0"):
        sess = sb.Session(g, w, 320, 9, 40, rows, 640, page_order=si.make_page_order(320, 4), tune=tune)
        sb.spiral_profile_begin(sess.model, sb.KERNEL_CLASSES.index("qkv_post"), 10)
        got.append(sess.prefill(ids, seqs).cpu().numpy())
        _, n_post = sb.spiral_profile_end(sess.model)
        assert n_post == (0 if tune == "fuse_qkv=1" else 1)
        sess.close()
    assert np.array_equal(got[0], got[1])
    want = od.forward_full(g, host, seqs[0], logits_at=np.array([len(seqs[0]) - 1]))[0]
    assert np.abs(got[0][0] - want).max() <= 3e-2 * want.std()

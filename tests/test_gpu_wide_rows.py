"""Projections over more than 128 rows: tiles of 256 x 256 or 128 x 256 or the streaming kernel, K split or not, q/k/v
post-processing inside the projection or behind it - chosen from the shape.  Repacked weights must give the bits that
row-major ones (always the streaming kernel) give, and both the oracle's logits within the bar of every logit comparison
(3e-2 x per-row logit std).  test_row_counts_around_the_tiles is the streaming kernel with either weights, its O and down
projections split; the tests behind it name the tile that their shapes reach and check the rule for it."""
import ctypes as C

import numpy as np
import pytest

from oracle import decoder as od
from paper_2506_24119_amd import inputs as si

pytestmark = pytest.mark.gpu


def tile_height(M, N, K, splits, cols=256):
    """Rows of the tiles that a projection with fragment-ordered weights takes, 0 for the streaming kernel."""
    from paper_2506_24119_amd import binding as sb
    f = sb.load_library()["_ZN6spiral16gemm_tile_heightEiiiiii"]
    f.restype, f.argtypes = C.c_int, [C.c_int] * 6
    return f(M, N, K, splits, cols, 128)


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


TILED = dict(d_model=1024, n_q_heads=16, n_kv_heads=4, head_dim=128, ffn_dim=8192, vocab=512, rope_theta=1e6)


def _prefill_and_step(g, w, rows, tune, repack):
    import torch
    from paper_2506_24119_amd import binding as sb
    rng = np.random.Generator(np.random.PCG64(rows))
    lens = [rows - 2 * (rows // 3), rows // 3, rows // 3]
    seqs = [rng.integers(0, g.vocab, n).astype(np.int32) for n in lens]
    step = rng.integers(0, g.vocab, 3).astype(np.int32)
    ids = np.arange(3, dtype=np.int32)
    sess = sb.Session(g, w, 150, 3, 50, rows, 600, page_order=si.make_page_order(150, 4), repack=repack, tune=tune)
    out = [sess.prefill(ids, seqs).cpu().numpy()]
    sb.spiral_model_tune(sess.model, "qkv=0:0,o=0:0,down=0:0")                # the step that reads the appended k, v: as it comes
    out.append(sess.decode_step(ids, torch.from_numpy(step).cuda(), sess.new_logits(3)).cpu().numpy())
    sess.close()
    return seqs, step, out


# rows; K splits of O, down, q/k/v; tile heights of O, down, q/k/v and gate/up that these reach
@pytest.mark.parametrize("rows,splits,heights", [
    (129, (1, 3, 1), (128, 128, 0, 0)), (255, (1, 2, 1), (128, 128, 0, 0)), (257, (1, 2, 5), (128, 128, 128, 128)),
    (520, (1, 1, 3), (0, 128, 128, 256)), (1000, (5, 5, 2), (128, 128, 128, 256)), (1300, (3, 3, 1), (128, 128, 128, 128)),
    (1600, (5, 5, 1), (256, 256, 128, 256))])
def test_tiles_against_the_streaming_kernel(rows, splits, heights):
    """Both tile heights, split (64 and 8 chunks of K in 3 and 5 uneven parts) and whole, with and without SwiGLU, at row counts
    that leave remainders of 1, 127 and more rows in the last tile."""
    g = si.ModelGeometry("tiles", 1, qk_norm=True, **TILED)
    d, qw, nqkv, ffn = 1024, 2048, 3072, 8192
    assert (tile_height(rows, d, qw, splits[0]), tile_height(rows, d, ffn, splits[1]), tile_height(rows, nqkv, d, splits[2]),
            tile_height(rows, ffn, d, 1, 128)) == heights
    from paper_2506_24119_amd import binding as sb
    host = si.make_weights(g, seed=14)
    w = sb.weights_to_device(host)
    tune = "fuse_qkv=0,o=128:%d,down=128:%d,qkv=128:%d" % splits
    seqs, step, tiled = _prefill_and_step(g, w, rows, tune, True)
    _, _, streamed = _prefill_and_step(g, w, rows, tune, False)
    assert np.array_equal(tiled[0], streamed[0]) and np.array_equal(tiled[1], streamed[1])
    want = od.forward_full(g, host, np.concatenate([seqs[2], step[2:]]), logits_at=np.array([len(seqs[2]) - 1, len(seqs[2])]))
    for k in range(2):
        assert np.abs(tiled[k][2] - want[k]).max() <= 3e-2 * want[k].std()


@pytest.mark.parametrize("rows", [900, 1281])
@pytest.mark.parametrize("variant", ["qk_norm", "qkv_bias"])
def test_fused_qkv_epilogue_rounds_like_the_post_kernel(rows, variant):
    """The q/k/v projection's own epilogue, qkv_post_kernel behind the tiled projection and qkv_post_kernel behind the streaming
    one (row-major weights): the same bits in the logits, and in the k and v that a decode step reads."""
    from paper_2506_24119_amd import binding as sb
    g = si.ModelGeometry("tiles", 2, qk_norm=variant == "qk_norm", qkv_bias=variant == "qkv_bias", **dict(TILED, ffn_dim=1024))
    host = si.make_weights(g, seed=15)
    w = sb.weights_to_device(host)
    got = []
    for tune, repack in ((None, True), ("fuse_qkv=0,qkv=128:1", True), (None, False)):
        got.append(_prefill_and_step(g, w, rows, tune, repack)[2])
    for other in got[1:]:
        assert np.array_equal(got[0][0], other[0]) and np.array_equal(got[0][1], other[1])
    # the default form is the fused one here: no post-processing launches in a prefill
    sess = sb.Session(g, w, 150, 3, 100, rows, 1500, page_order=si.make_page_order(150, 4))
    sb.spiral_profile_begin(sess.model, sb.KERNEL_CLASSES.index("qkv_post"), 10)
    sess.prefill([0], [np.zeros(rows, dtype=np.int32)])
    assert sb.spiral_profile_end(sess.model)[1] == 0
    sess.close()


def test_a_sequence_among_others_stays_close_to_itself_alone():
    """Above 128 rows the K splits, and so the order of fp32 sums, follow from the rows of the whole call: a sequence of 300
    tokens alone (300 rows) and among others (1,600) differs by roundings of half-precision activations, 2^-11 of a
    value, in two layers: 1e-2 x std, the bound of the decode-attention pieces, which differ for the same reason."""
    import torch
    from paper_2506_24119_amd import binding as sb
    g = si.ModelGeometry("tiles", 2, qk_norm=True, **TILED)
    w = sb.weights_to_device(si.make_weights(g, seed=16))
    seqs = si.make_prompts(g.vocab, 4, 433, 434, seed=10)
    seqs[1] = seqs[1][:300]
    step = torch.arange(4, dtype=torch.int32, device="cuda")
    got = []
    for batch in ([0, 1, 2, 3], [1]):
        sess = sb.Session(g, w, 120, 4, 30, 1700, 480, page_order=si.make_page_order(120, 4))
        at = batch.index(1)
        out = [sess.prefill(batch, [seqs[b] for b in batch]).cpu().numpy()[at]]
        out.append(sess.decode_step(batch, step[torch.tensor(batch, device="cuda")].contiguous(), sess.new_logits(len(batch))).cpu().numpy()[at])
        got.append(out)
        sess.close()
    for k in range(2):
        assert np.abs(got[0][k] - got[1][k]).max() <= 1e-2 * got[1][k].std(), k

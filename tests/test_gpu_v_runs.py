"""V leaves the fused q/k/v projection in runs of four tokens of a page that start anywhere in a row tile; what a sequence's or a tile's end cuts off
goes token by token.  Appending runs of one token and more at every place of a page must leave the pages that qkv_post_kernel, which
writes element by element, leaves: the same bits in the logits of that call and of a step that reads them."""
import numpy as np
import pytest

from paper_2506_24119_amd import inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("longest,count", [(1, 1000), (3, 600), (7, 330), (60, 37)])
def test_runs_at_every_place_of_a_page(longest, count):
    import torch
    from paper_2506_24119_amd import binding as sb
    g = si.ModelGeometry("runs", 2, 1024, 16, 4, 128, 1024, 512, 1e6, qk_norm=True)
    w = sb.weights_to_device(si.make_weights(g, seed=21))
    rng = np.random.Generator(np.random.PCG64(longest))
    hist = [rng.integers(0, g.vocab, 1 + i % 16).astype(np.int32) for i in range(count)]
    new = [rng.integers(0, g.vocab, n).astype(np.int32) for n in rng.integers(1, longest + 1, count)]
    step = torch.from_numpy(rng.integers(0, g.vocab, count).astype(np.int32)).cuda()
    ids = np.arange(count, dtype=np.int32)
    rows = sum(len(n) for n in new)
    blocks = sum((len(h) + len(n) + 16) // 16 for h, n in zip(hist, new)) + 4
    got = []
    for fuse in (1, 0):                          # K unsplit in both, also in the histories' call, which may have too few rows to fuse
        tune = "fuse_qkv=%d,qkv=128:1" % fuse
        sess = sb.Session(g, w, blocks, count, 8, max(rows, sum(map(len, hist))), 128, page_order=si.make_page_order(blocks, 4), tune=tune)
        sess.prefill(ids, hist)
        sb.spiral_profile_begin(sess.model, sb.KERNEL_CLASSES.index("qkv_post"), 10)
        out = [sess.prefill(ids, new).cpu().numpy()]
        assert sb.spiral_profile_end(sess.model)[1] == (0 if fuse else 2), rows
        sb.spiral_model_tune(sess.model, "qkv=0:0")
        out.append(sess.decode_step(ids, step, sess.new_logits(count)).cpu().numpy())
        sess.close()
        got.append(out)
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])

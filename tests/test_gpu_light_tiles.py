"""Tiled projections whose last row tile of 128 is partly empty: its waves multiply the 32-row blocks that there are (none, one or two each),
and at most half full it is walked last.  Row counts on either side of each block, whole and split K, SwiGLU, the fused q/k/v epilogue and
the scoring head; repacked weights must give the bits that row-major ones give (the streaming kernel, which knows no such tiles)."""
import numpy as np
import pytest

from paper_2506_24119_amd import inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [129, 160, 161, 192, 193, 224, 225, 256, 257, 289, 321, 353, 385, 641, 800])
def test_partly_empty_row_tiles(rows):
    import torch
    from paper_2506_24119_amd import binding as sb
    g = si.ModelGeometry("light", 2, 1024, 8, 2, 128, 3072, 3000, 1e6, qk_norm=True)
    w = si.make_weights_torch(g, 6, "cuda:0")
    rng = np.random.Generator(np.random.PCG64(rows))
    n = [rows - rows // 3, rows // 3]
    seqs = [rng.integers(0, g.vocab, k).astype(np.int32) for k in n]
    tok = torch.from_numpy(np.concatenate(seqs)).cuda()
    targets = torch.from_numpy(rng.integers(0, g.vocab, rows).astype(np.int32)).cuda()
    step = torch.from_numpy(rng.integers(0, g.vocab, 2).astype(np.int32)).cuda()
    ids, got = np.arange(2, dtype=np.int32), []
    for repack in (True, False):
        for tune in (None, "o=128:3,down=128:2,qkv=128:1"):
            sess = sb.Session(g, w, 120, 2, 60, rows, rows + 8, page_order=si.make_page_order(120, 2), repack=repack, tune=tune)
            logp = torch.zeros(rows, dtype=torch.float32, device="cuda")
            sb.spiral_score(sess.model, sess.pool, ids, n, tok, targets, sess.ws, logp)
            out = [logp.cpu().numpy(), sess.decode_step(ids, step, sess.new_logits(2)).cpu().numpy()]      # reads the appended k, v
            sb.spiral_seq_truncate(sess.pool, ids, np.zeros(2, dtype=np.int32))
            out.append(sess.prefill(ids, seqs).cpu().numpy())
            got.append(out)
            sess.close()
    for tune in range(2):
        for a, b in zip(got[tune], got[2 + tune]):
            assert np.isfinite(a).all() and np.array_equal(a, b), (tune, rows)

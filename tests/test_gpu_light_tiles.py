"""Tiled projections whose last row tile of 128 is partly empty: its waves multiply the 32-row blocks that there are (none, one or two each),
and at most half full it is walked last.  Row counts on either side of each block, at which every projection takes such tiles: O and down with
K split, q/k/v whole, behind it either its own kernel or the fused epilogue, SwiGLU, and the scoring head; repacked weights must give the bits
that row-major ones give (the streaming kernel, which knows no such tiles)."""
import ctypes as C

import numpy as np
import pytest

from paper_2506_24119_amd import inputs as si
from test_gpu_wide_rows import TILED, tile_height

pytestmark = pytest.mark.gpu


def _wide_splits(M, N, K):
    from paper_2506_24119_amd import binding as sb
    f = sb.load_library()["_ZN6spiral15gemm_wide_shapeEiiiiRiS0_"]
    f.restype, f.argtypes = C.c_float, [C.c_int] * 4 + [C.POINTER(C.c_int)] * 2
    bn, splits = C.c_int(), C.c_int()
    f(M, N, K, 16, C.byref(bn), C.byref(splits))
    return splits.value


@pytest.mark.parametrize("tune", [None, "fuse_qkv=0,qkv=128:1,o=128:3,down=128:3"])
@pytest.mark.parametrize("rows", [1281, 1312, 1313, 1344, 1345, 1376, 1377, 1408, 1409])
def test_partly_empty_row_tiles(rows, tune):
    import torch
    from paper_2506_24119_amd import binding as sb
    g = si.ModelGeometry("light", 2, qk_norm=True, **dict(TILED, vocab=3000))
    d, qw, nqkv, ffn = g.d_model, g.n_q_heads * 128, (g.n_q_heads + 2 * g.n_kv_heads) * 128, g.ffn_dim
    s_o, s_down = (3, 3) if tune else (_wide_splits(rows, d, qw), _wide_splits(rows, d, ffn))
    assert s_o > 1 and s_down > 1
    assert (tile_height(rows, d, qw, s_o), tile_height(rows, d, ffn, s_down), tile_height(rows, nqkv, d, 1), tile_height(rows, ffn, d, 1, 128)) == (128,) * 4
    w = si.make_weights_torch(g, 6, "cuda:0")
    rng = np.random.Generator(np.random.PCG64(rows))
    n = [rows - rows // 3, rows // 3]
    seqs = [rng.integers(0, g.vocab, k).astype(np.int32) for k in n]
    tok = torch.from_numpy(np.concatenate(seqs)).cuda()
    targets = torch.from_numpy(rng.integers(0, g.vocab, rows).astype(np.int32)).cuda()
    step = torch.from_numpy(rng.integers(0, g.vocab, 2).astype(np.int32)).cuda()
    ids, got = np.arange(2, dtype=np.int32), []
    for repack in (True, False):
        sess = sb.Session(g, w, 120, 2, 60, rows, rows + 8, page_order=si.make_page_order(120, 2), repack=repack, tune=tune)
        logp = torch.zeros(rows, dtype=torch.float32, device="cuda")
        sb.spiral_profile_begin(sess.model, sb.KERNEL_CLASSES.index("qkv_post"), 8)
        sb.spiral_score(sess.model, sess.pool, ids, n, tok, targets, sess.ws, logp)
        assert sb.spiral_profile_end(sess.model)[1] == (0 if repack and tune is None else g.n_layers)
        out = [logp.cpu().numpy(), sess.decode_step(ids, step, sess.new_logits(2)).cpu().numpy()]      # reads the appended k, v
        sb.spiral_seq_truncate(sess.pool, ids, np.zeros(2, dtype=np.int32))
        out.append(sess.prefill(ids, seqs).cpu().numpy())
        got.append(out)
        sess.close()
    for a, b in zip(*got):
        assert np.isfinite(a).all() and np.array_equal(a, b), rows

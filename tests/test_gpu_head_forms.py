"""The LM head of a decode step by rows and vocabulary: gemm_decode_kernel (at most 32 rows, or a small head up to 128), the streaming
kernel, tiles of 128 rows (from 65 rows and 65,536 columns on; the sampler's winners of up to 128 rows only from a d_model of 2,048 on).  Repacked weights give the bits of row-major ones, whose head is never
tiled, and the fused step's tokens are those of the sampler on the stored logits."""
import numpy as np
import pytest

from paper_2506_24119_amd import inputs as si

pytestmark = pytest.mark.gpu


def _step(g, w, rows, repack, T):
    import torch
    from paper_2506_24119_amd import binding as sb
    ids = np.arange(rows, dtype=np.int32)
    rng = np.random.Generator(np.random.PCG64(rows))
    tok = torch.from_numpy(rng.integers(0, g.vocab, rows).astype(np.int32)).cuda()
    steps = (np.arange(rows, dtype=np.int32) * 5 + 2).astype(np.int32)
    sess = sb.Session(g, w, rows, rows, 1, 5 * rows, 16, repack=repack)
    sess.prefill(ids, [rng.integers(0, g.vocab, 1 + b % 5).astype(np.int32) for b in range(rows)])
    lens = np.array([1 + b % 5 for b in range(rows)], dtype=np.int32)
    logits = sess.decode_step(ids, tok, sess.new_logits(rows))
    stored, fused = (torch.full((rows,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
    sb.spiral_sample(logits, rows, g.vocab, T, 9, ids, steps, None, stored)
    if repack:
        sb.spiral_seq_truncate(sess.pool, ids, lens)
        sess.decode_sample_step(ids, tok, T, 9, steps, fused)
    out = logits.cpu().numpy(), stored.cpu().numpy(), fused.cpu().numpy()
    sess.close()
    return out


@pytest.mark.parametrize("d,vocab,rows", [
    (128, 1008, 33), (128, 1008, 128), (2560, 8192, 65), (2560, 13104, 96),                            # small heads: up to 2^25 weights, eight columns to a k
    (2560, 13120, 128), (128, 65520, 65), (640, 65536, 64),                                            # more weights, more columns: the streaming kernel
    (640, 65536, 65), (640, 65552, 128), (640, 65536, 129),                                            # tiles of the logits, up to 128 rows; winners streamed up to there
    (2048, 65552, 65), (2048, 65536, 100), (128, 70000, 257)])                                         # tiles with winners, one and three rows of them
def test_forms_of_the_head_agree(d, vocab, rows):
    g = si.ModelGeometry("head", 1, d, 4, 2, 64, 256, vocab, 1e6, qk_norm=True)
    w = si.make_weights_torch(g, 5, "cuda:0")
    tiled, stored, fused = _step(g, w, rows, True, 1.0)
    plain, other, _ = _step(g, w, rows, False, 1.0)
    assert np.array_equal(tiled, plain) and np.array_equal(stored, other)
    assert np.array_equal(fused, stored) and len(set(fused)) > rows // 8
    logits, greedy, fused = _step(g, w, rows, True, 0.0)
    assert np.array_equal(greedy, logits.argmax(1)) and np.array_equal(fused, greedy)


@pytest.mark.parametrize("d,vocab,rows", [(1024, 65536, 65), (1920, 65552, 128)])
def test_tiled_logits_and_streamed_winners_agree(d, vocab, rows):
    """Up to 128 rows and d_model below 2,048 the logits come from tiles, the sampler's winners from the streaming kernel."""
    import ctypes as C
    from paper_2506_24119_amd import binding as sb
    tiled = sb.load_library()["_ZN6spiral15gemm_head_tiledEiiii"]
    tiled.restype, tiled.argtypes = C.c_bool, [C.c_int] * 4
    assert tiled(rows, vocab, d, 0) and not tiled(rows, vocab, d, 2)
    g = si.ModelGeometry("head", 1, d, 4, 2, 64, 256, vocab, 1e6, qk_norm=True)
    w = si.make_weights_torch(g, 5, "cuda:0")
    for T in (1.0, 0.0):
        logits, stored, fused = _step(g, w, rows, True, T)
        assert np.array_equal(fused, stored) and len(set(fused)) > rows // 8
    assert np.array_equal(fused, logits.argmax(1))


@pytest.mark.parametrize("d,vocab", [(576, 65536), (640, 65540), (96, 70004)])
@pytest.mark.parametrize("rows", [64, 65, 100, 128, 129])
def test_large_heads_of_other_widths_agree(d, vocab, rows):
    """d_model not a multiple of 128, or a vocabulary not one of 16: neither the streaming kernel nor tiles, with either weights."""
    import torch
    from paper_2506_24119_amd import binding as sb
    g = si.ModelGeometry("head", 1, d, 4, 2, 64, 256, vocab, 1e6, qk_norm=True)
    w = si.make_weights_torch(g, 5, "cuda:0")
    ids = np.arange(rows, dtype=np.int32)
    rng = np.random.Generator(np.random.PCG64(rows))
    seqs = [rng.integers(0, vocab, 1 + b % 5).astype(np.int32) for b in range(rows)]
    tok = torch.from_numpy(rng.integers(0, vocab, rows).astype(np.int32)).cuda()
    got = []
    for repack in (True, False):
        sess = sb.Session(g, w, rows, rows, 1, 5 * rows, 16, repack=repack)
        got.append([sess.prefill(ids, seqs).cpu().numpy(), sess.decode_step(ids, tok, sess.new_logits(rows)).cpu().numpy()])
        sess.close()
    for a, b in zip(*got):
        assert np.isfinite(a).all() and np.array_equal(a, b)

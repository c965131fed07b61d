"""The projections of at most 128 rows (gemm_decode_kernel): a decode step and a short prefill at the edges of its row tiles, weight
tiles and K splits, against the oracle; repacked and row-major weights give the same bits, a sequence's logits do not depend on
how many others are in the call, and the fused sampler draws what the stored logits give on either side of 32 rows."""
import ctypes

import numpy as np
import pytest

from oracle import decoder as od
from paper_2506_24119_amd import inputs as si

LOGIT_TOL = 3e-2          # the bar of every logit comparison: half-precision activations

# K = 128 (the least, no split to make), widths that leave a remainder in the last weight tile (176 q/k/v heads x 32; ffn 416 and
# vocabulary 2,512 are 26 and 78.5 tiles), and a wide one whose projections split K
NARROW = si.ModelGeometry("narrow", 2, 128, 4, 1, 32, 384, 2512, 1e4, qkv_bias=True, tie_lm_head=False)
WIDE = si.ModelGeometry("wide", 2, 640, 10, 2, 128, 1408, 2512, 1e6, qk_norm=True)
# gate/up on the streaming kernel (776 tiles of 16 columns; up to 512 do not go there), which writes what the down projection reads
FFN = si.ModelGeometry("ffn", 2, 128, 4, 2, 32, 12416, 512, 1e4)


def _run(g, w, B, repack, ids=None, sample=False, tune=None):
    import torch
    from paper_2506_24119_amd import binding as sb
    rng = np.random.Generator(np.random.PCG64(7))
    lens = rng.integers(1, 20, 128)
    prompts = [rng.integers(0, g.vocab, int(n)).astype(np.int32) for n in lens]
    step = rng.integers(0, g.vocab, 128).astype(np.int32)
    ids = np.arange(B) if ids is None else np.array(ids)
    n = len(ids)
    sess = sb.Session(g, w, 3 * n + 2, n, 3, 128, 40, page_order=si.make_page_order(3 * n + 2, 3), repack=repack, tune=tune)
    seqs = np.arange(n, dtype=np.int32)
    for i in range(0, n, 6):                               # at most 6 x 19 rows: every projection of the prompts is a small one, too
        sess.prefill(seqs[i:i + 6], [prompts[b] for b in ids[i:i + 6]])
    tin = torch.from_numpy(step[ids]).cuda()
    out = sess.decode_step(seqs, tin, sess.new_logits(n)).cpu().numpy()
    if sample:
        at = np.full(n, 4, dtype=np.int32)
        a, b = torch.empty(n, dtype=torch.int32, device="cuda"), torch.empty(n, dtype=torch.int32, device="cuda")
        sess.sample(torch.from_numpy(out).cuda(), 1.0, 5, seqs, at, a)
        sb.spiral_seq_truncate(sess.pool, seqs, np.array([len(prompts[b]) for b in ids], dtype=np.int32))
        sess.decode_sample_step(seqs, tin, 1.0, 5, at, b)
        assert torch.equal(a, b)
    assert sess.saturation_count() == 0
    sess.close()
    return out, prompts, step


@pytest.mark.gpu
@pytest.mark.parametrize("g", [NARROW, WIDE, FFN], ids=["narrow", "wide", "ffn"])
@pytest.mark.parametrize("B", [1, 7, 31, 32, 33, 64, 65, 96, 97, 128])
def test_rows_against_oracle_and_row_major(g, B):
    from paper_2506_24119_amd import binding as sb
    host = si.make_weights(g, seed=71)
    w = sb.weights_to_device(host)
    got, prompts, step = _run(g, w, B, True, sample=B in (32, 33))
    assert np.array_equal(got, _run(g, w, B, False)[0])
    for b in {0, B // 2, B - 1}:
        toks = np.concatenate([prompts[b], step[b:b + 1]]).astype(np.int64)
        want = od.forward_full(g, host, toks, logits_at=np.array([len(toks) - 1]))[0]
        assert np.abs(got[b] - want).max() <= LOGIT_TOL * want.std(), b


@pytest.mark.gpu
def test_a_sequence_does_not_depend_on_the_rows_of_its_step():
    """The same K splits and order of sums at every row count up to 128: only the LM head changes kernels (at 33 rows), and nothing
    rounds its fp32 sums, so logits differ by a few units in the last place of a sum of 640 products (1e-6 of their size)."""
    from paper_2506_24119_amd import binding as sb
    w = sb.weights_to_device(si.make_weights(WIDE, seed=72))
    full = _run(WIDE, w, 128, True)[0]
    for ids in ([5], list(range(3, 33)), list(range(40)), list(range(30, 100))):
        got = _run(WIDE, w, None, True, ids=ids)[0]
        assert np.abs(got - full[ids]).max() <= 1e-5 * np.abs(full[ids]).max(), len(ids)


@pytest.mark.gpu
@pytest.mark.parametrize("tune", ["gu=64", "gu=96", "gu=160"])
def test_every_form_of_a_wide_gate_up(tune):
    """The streaming kernel's other workgroups hand the down projection the same bits."""
    from paper_2506_24119_amd import binding as sb
    w = sb.weights_to_device(si.make_weights(FFN, seed=73))
    for B in (7, 64, 128):
        for repack in (True, False):
            assert np.array_equal(_run(FFN, w, B, repack, tune=tune)[0], _run(FFN, w, B, repack)[0]), B


def test_gate_up_and_down_agree_on_the_order_between_them():
    """Down projections that read rows where they could read the operands' order take up to 1.7 times as long."""
    from paper_2506_24119_amd import binding
    lib = binding.load_library()
    frag, takes = lib._ZN6spiral16gemm_mlp_in_fragEiii, lib._ZN6spiral17gemm_decode_takesEiiiib
    for f, args in ((frag, [ctypes.c_int] * 3), (takes, [ctypes.c_int] * 4 + [ctypes.c_bool])):
        f.argtypes, f.restype = args, ctypes.c_bool
    for d, ffn in ((1024, 3072), (2560, 9728), (2048, 11008)):
        for M in (1, 32, 33, 128):
            assert takes(M, d, ffn, 0, False) and frag(M, d, ffn)
        assert not frag(129, d, ffn)
    assert not frag(8, 1088, 2176) and not frag(8, 1024, 1088) and not frag(8, 3584, 18944)          # gate/up, down on another kernel


def test_which_projections_are_small():
    from paper_2506_24119_amd import binding
    takes = binding.load_library()._ZN6spiral17gemm_decode_takesEiiiib
    takes.argtypes = [ctypes.c_int] * 4 + [ctypes.c_bool]
    takes.restype = ctypes.c_bool
    assert takes(1, 16, 128, 0, False) and takes(128, 16, 128, 0, False) and not takes(129, 16, 128, 0, False) and not takes(0, 16, 128, 0, False)
    assert not takes(8, 24, 128, 0, False) and not takes(8, 32, 192, 0, False)
    # where row-major weights, which take the same kernel as repacked ones, are slow on it: gate/up of more than two tiles a unit, 64 MB
    assert takes(128, 8192, 128, 1, False) and not takes(128, 8208, 128, 1, False) and not takes(1, 9728, 2560, 1, False)
    assert takes(128, 8192, 4096, 0, False) and not takes(1, 8208, 4096, 0, False) and not takes(1, 3584, 18944, 0, False)
    assert takes(32, 151936, 1024, 0, True) and not takes(33, 151936, 1024, 0, True)


def test_splits_are_those_of_the_shape():
    """The K splits by the projection alone, at least 128 k each; measured choices of three shapes."""
    from paper_2506_24119_amd import binding
    splits = binding.load_library()._ZN6spiral18gemm_decode_splitsEiii
    assert [splits(n, k, 16) for n, k in ((4096, 1024), (1024, 2048), (1024, 3072))] == [2, 8, 8]
    assert [splits(n, k, 16) for n, k in ((6144, 2560), (2560, 4096), (2560, 9728))] == [4, 3, 6]
    assert [splits(n, k, 16) for n, k in ((4608, 3584), (3584, 3584), (3584, 18944))] == [3, 4, 6]
    for n in (16, 48, 640, 6144):
        for k in (128, 256, 1408, 9728):
            assert 1 <= splits(n, k, 16) <= k // 128


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [31, 33, 97, 128])
@pytest.mark.parametrize("repack", [True, False])
def test_prefill_attention_writes_what_the_projection_reads(rows, repack):
    """Prefills of at most 128 rows: the attention's output goes to O in the operands' order, at row counts that leave remainders of
    a tile of 32, with runs that start inside a tile; against the oracle, and the same bits with either order of the weights."""
    from paper_2506_24119_amd import binding as sb
    host = si.make_weights(WIDE, seed=74)
    w = sb.weights_to_device(host)
    rng = np.random.Generator(np.random.PCG64(rows))
    seqs = [rng.integers(0, WIDE.vocab, n).astype(np.int32) for n in (5, rows - 22, 17)]
    sess = sb.Session(WIDE, w, 30, 3, 10, 128, 140, page_order=si.make_page_order(30, 3), repack=repack)
    got = sess.prefill(np.arange(3, dtype=np.int32), seqs).cpu().numpy()
    sess.close()
    for b, s in enumerate(seqs):
        want = od.forward_full(WIDE, host, s, logits_at=np.array([len(s) - 1]))[0]
        assert np.abs(got[b] - want).max() <= LOGIT_TOL * want.std(), b


@pytest.mark.gpu
def test_output_projection_of_a_prefill_takes_as_long_as_that_of_a_step():
    """The same projection of 128 rows on the 4B shape, in a prefill and in a decode step: 1.75 times as long when the prefill's
    attention left its output in rows.  The shortest of 20 launches each, between events."""
    import torch
    from paper_2506_24119_amd import binding as sb
    g = si.scaled_geometry("qwen3-4b", n_layers=1, vocab=512)
    sess = sb.Session(g, si.make_weights_torch(g, 1, "cuda:0"), 2 * 128 + 8, 128, 2, 128, 32, page_order=si.make_page_order(264, 3))
    ids = np.arange(128, dtype=np.int32)
    tok = torch.zeros(128, dtype=torch.int32, device="cuda")
    logits = sess.new_logits(128)
    runs = {"prefill": lambda: sb.spiral_prefill(sess.model, sess.pool, ids, np.ones(128, dtype=np.int32), tok, sess.ws, logits),
            "step": lambda: sess.decode_step(ids, tok, logits)}
    best = {}
    for name, run in runs.items():
        for _ in range(20):
            sb.spiral_seq_reset(sess.pool, ids)
            runs["prefill"]()
            sb.spiral_profile_begin(sess.model, sb.KERNEL_CLASSES.index("gemm_o"), 1)
            run()
            best[name] = min(best.get(name, 1e9), sb.spiral_profile_end(sess.model)[0])
    sess.close()
    assert best["prefill"] <= 1.35 * best["step"], best


@pytest.mark.gpu
@pytest.mark.parametrize("key", ["qkv", "o", "down"])
def test_tuned_rows_and_splits_of_small_calls(key):
    """spiral_model_tune "key=R:S" up to 128 rows: any R gives the same bits, one and three K splits add in different orders."""
    from paper_2506_24119_amd import binding as sb
    w = sb.weights_to_device(si.make_weights(WIDE, seed=75))
    for B in (5, 100):
        one = _run(WIDE, w, B, True, tune=f"{key}=32:1")[0]
        for R in (16, 64, 96, 128, 160):
            assert np.array_equal(one, _run(WIDE, w, B, True, tune=f"{key}={R}:1")[0]), (B, R)
        three = _run(WIDE, w, B, True, tune=f"{key}=64:3")[0]
        assert not np.array_equal(one, three) and np.abs(one - three).max() <= 1e-2 * one.std(), B


@pytest.mark.gpu
@pytest.mark.parametrize("repack", [True, False])
def test_widths_on_either_side_of_the_large_projections(repack):
    """q/k/v (7,168 x 5,120) and down (5,120 x 6,656) of more than 64 MB stay on the streaming kernel, q alone, O and gate/up do not: whoever
    writes their input has to know.  A decode step, a prefill of few rows and one whose last layer has one row a sequence."""
    import torch
    from paper_2506_24119_amd import binding as sb
    g = si.ModelGeometry("large", 1, 5120, 40, 8, 128, 6656, 512, 1e6)
    host = si.make_weights(g, seed=76)
    w = sb.weights_to_device(host)
    rng = np.random.Generator(np.random.PCG64(77))
    sess = sb.Session(g, w, 60, 4, 14, 200, 220, page_order=si.make_page_order(60, 3), repack=repack)
    seqs = [rng.integers(0, g.vocab, n).astype(np.int32) for n in (9, 14)]
    got = list(sess.prefill(np.arange(2, dtype=np.int32), seqs).cpu().numpy())
    long = [rng.integers(0, g.vocab, n).astype(np.int32) for n in (60, 75)]
    got += list(sess.prefill(np.array([2, 3], dtype=np.int32), long).cpu().numpy())
    step = rng.integers(0, g.vocab, 4).astype(np.int32)
    got += list(sess.decode_step(np.arange(4, dtype=np.int32), torch.from_numpy(step).cuda(), sess.new_logits(4)).cpu().numpy())
    sess.close()
    seqs += long
    for b, s in enumerate(seqs):
        want = od.forward_full(g, host, np.concatenate([s, step[b:b + 1]]), logits_at=np.array([len(s) - 1, len(s)]))
        for k in range(2):
            assert np.abs(got[4 * k + b] - want[k]).max() <= LOGIT_TOL * want[k].std(), (b, k)

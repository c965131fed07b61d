"""Causal prefill attention around the edges of its tiles: 32 positions a wave, 64 tokens a step, up to four heads of a
group (or several position tiles) a workgroup, histories that start anywhere in a page.  Against the oracle's full
recompute, bar as for every logit comparison: max |dlogit| <= 3e-2 x per-row logit std."""
import numpy as np
import pytest

from oracle import decoder as od
from paper_2506_24119_amd import inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q_heads,kv_heads,head_dim,dtype", [
    (2, 2, 128, si.WEIGHT_BF16), (4, 2, 128, si.WEIGHT_BF16), (6, 2, 64, si.WEIGHT_BF16), (5, 1, 128, si.WEIGHT_BF16),
    (7, 1, 64, si.WEIGHT_BF16), (16, 1, 32, si.WEIGHT_BF16), (9, 3, 32, si.WEIGHT_FP32)])
@pytest.mark.parametrize("tune", [None, "trim=0"])
def test_ragged_runs_and_histories(q_heads, kv_heads, head_dim, dtype, tune):
    """"trim=0": the last layer's attention goes through the prefill kernel, too, and its output for the last rows to the logits."""
    import torch
    from paper_2506_24119_amd import binding as sb
    g = si.ModelGeometry("attn-edges", 2, 128, q_heads, kv_heads, head_dim, 128, 256, 1e4, qk_norm=head_dim == 128,
                         weight_dtype=dtype)
    w = si.make_weights(g, seed=3)
    rng = np.random.Generator(np.random.PCG64(5))
    first = [1, 31, 33, 63, 65, 129, 200, 16]              # around 32, 64 and the page of 16
    second = [1, 33, 31, 65, 1, 64, 97, 140]
    seqs = [rng.integers(0, g.vocab, a + b).astype(np.int32) for a, b in zip(first, second)]
    ids = np.arange(len(seqs), dtype=np.int32)
    sess = sb.Session(g, sb.weights_to_device(w), 160, len(seqs), 24, 1024, 400, page_order=si.make_page_order(160, 2), tune=tune)
    got = [sess.prefill(ids, [s[:a] for s, a in zip(seqs, first)]).cpu().numpy()]
    got.append(sess.prefill(ids, [s[a:] for s, a in zip(seqs, first)]).cpu().numpy())
    torch.cuda.synchronize()
    sess.close()
    for b, s in enumerate(seqs):
        want = od.forward_full(g, w, s, logits_at=np.array([first[b] - 1, len(s) - 1]))
        for k in range(2):
            ratio = np.abs(got[k][b] - want[k]).max() / want[k].std()
            assert ratio <= 3e-2, (b, k, ratio)


def test_one_very_long_run_beside_a_thousand_short_ones():
    """1,023 runs of one token beside one of 65,632: 8,192 (sequence, kv head) pairs x 2,051 blocks of 32 positions are more
    workgroups than one dimension of a launch may have threads for.  Every sequence must get the logits that it gets without the
    others (fp32 weights: nothing but attention sees more than one row), bit for bit."""
    import torch
    from paper_2506_24119_amd import binding as sb
    g = si.ModelGeometry("long", 1, 64, 32, 8, 32, 64, 64, 1e4, weight_dtype=si.WEIGHT_FP32)
    w = sb.weights_to_device(si.make_weights(g, seed=4))
    rng = np.random.Generator(np.random.PCG64(6))
    B, n = 1024, 65632
    seqs = [rng.integers(0, g.vocab, n if b == 5 else 1).astype(np.int32) for b in range(B)]
    assert (n + 31) // 32 * B * g.n_kv_heads * 256 > 1 << 32
    ids = np.arange(B, dtype=np.int32)
    sess = sb.Session(g, w, 4103 + B, B, 4103, n + B, n + 1, page_order=None)
    together = sess.prefill(ids, seqs).cpu().numpy()
    sb.spiral_seq_reset(sess.pool, ids)
    assert np.array_equal(together[5:6], sess.prefill(ids[5:6], seqs[5:6]).cpu().numpy())
    rest = np.delete(ids, 5)
    assert np.array_equal(together[rest], sess.prefill(rest, [seqs[b] for b in rest]).cpu().numpy())
    torch.cuda.synchronize()
    sess.close()


@pytest.mark.parametrize("q_heads,kv_heads,head_dim", [(4, 2, 128), (6, 2, 64), (8, 1, 32)])
@pytest.mark.parametrize("at", [16, 40, 63, 64, 90, 149])
def test_a_nan_stays_out_of_earlier_positions(q_heads, kv_heads, head_dim, at):
    """A token whose embedding is NaN leaves NaN in its K and V.  No earlier position sees it, so their log-probabilities must
    stay what they are with an ordinary token there; the position itself and the later ones are NaN.  Rows that share a
    64-token step with it are summed by another routine (fp32 sums in another order, the same half-precision weights): bound as
    for every log-probability, 6e-2 x logit std, here 1e-2 absolute at a logit std of about 0.3."""
    import torch
    from paper_2506_24119_amd import binding as sb
    g = si.ModelGeometry("nan", 2, 128, q_heads, kv_heads, head_dim, 256, 256, 1e4, tie_lm_head=False)
    w = si.make_weights(g, seed=13)
    w["embed"][7] = 0x7FC0                                  # bf16 NaN
    wd = sb.weights_to_device(w)
    rng = np.random.Generator(np.random.PCG64(7))
    seqs = [rng.integers(8, g.vocab, n).astype(np.int32) for n in (150, 33)]
    got = []
    for tok in (7, 9):
        seqs[0][at] = tok
        sess = sb.Session(g, wd, 40, 2, 16, 256, 200, page_order=si.make_page_order(40, 2))
        toks = torch.from_numpy(np.concatenate(seqs)).cuda()
        tg = torch.from_numpy(rng.permutation(183).astype(np.int32)).cuda() % g.vocab if not got else tg
        out = torch.empty(183, dtype=torch.float32, device="cuda")
        sb.spiral_score(sess.model, sess.pool, [0, 1], [150, 33], toks, tg, sess.ws, out)
        got.append(out.cpu().numpy())
        sess.close()
    assert np.isnan(got[0][at:150]).all() and not np.isnan(got[1]).any()
    assert not np.isnan(got[0][:at]).any() and not np.isnan(got[0][150:]).any()
    assert np.abs(got[0][:at] - got[1][:at]).max() <= 1e-2 and np.array_equal(got[0][150:], got[1][150:])
    assert np.array_equal(got[0][:max(0, at - 63)], got[1][:max(0, at - 63)])      # out of reach: not summed again


@pytest.mark.parametrize("q_heads,kv_heads", [(12, 12), (18, 6), (15, 3), (32, 2), (64, 4), (11, 11)])
def test_head_groups_and_sequence_counts(q_heads, kv_heads):
    """Workgroups find their sequence, kv head and head group by multiplication with reciprocals: group sizes 1 to 16 over kv
    head counts that are and are not powers of two, 1 and 37 sequences, against the oracle."""
    from paper_2506_24119_amd import binding as sb
    g = si.ModelGeometry("groups", 1, 64, q_heads, kv_heads, 32, 64, 128, 1e4, weight_dtype=si.WEIGHT_FP32)
    host = si.make_weights(g, seed=5)
    w = sb.weights_to_device(host)
    for n_seqs in (1, 37):
        seqs = si.make_prompts(g.vocab, n_seqs, 1, 90, seed=n_seqs)
        sess = sb.Session(g, w, 7 * n_seqs, n_seqs, 7, 90 * n_seqs, 100, page_order=si.make_page_order(7 * n_seqs, 2))
        got = sess.prefill(np.arange(n_seqs, dtype=np.int32), seqs).cpu().numpy()
        sess.close()
        for b, s in enumerate(seqs):
            want = od.forward_full(g, host, s, logits_at=np.array([len(s) - 1]))[0]
            assert np.abs(got[b] - want).max() <= 3e-2 * want.std(), (n_seqs, b)


@pytest.mark.parametrize("head_dim,dtype", [(32, si.WEIGHT_FP32), (128, si.WEIGHT_FP32), (64, si.WEIGHT_BF16)])
def test_a_nan_token_can_be_dropped(head_dim, dtype):
    """A run with a NaN token in it, cut back to the tokens before it and continued: the kept K and V of the second layer, which
    earlier positions' attention produced, hold no NaN.  Bound as for a sequence among others: 1e-2 x std."""
    from paper_2506_24119_amd import binding as sb
    g = si.ModelGeometry("nan", 2, 64, 8, 2, head_dim, 128, 256, 1e4, tie_lm_head=False, weight_dtype=dtype)
    w = si.make_weights(g, seed=17)
    w["embed"][7] = 0x7FC0 if dtype == si.WEIGHT_BF16 else np.nan
    wd = sb.weights_to_device(w)
    rng = np.random.Generator(np.random.PCG64(8))
    seq, more = rng.integers(8, g.vocab, 100).astype(np.int32), rng.integers(8, g.vocab, 3).astype(np.int32)
    seq[70] = 7
    got = []
    for run in (seq, seq[:70]):
        sess = sb.Session(g, wd, 16, 1, 16, 128, 200, page_order=si.make_page_order(16, 2))
        sess.prefill([0], [run])
        sb.spiral_seq_truncate(sess.pool, [0], [70])
        got.append(sess.prefill([0], [more]).cpu().numpy()[0])
        sess.close()
    assert np.abs(got[0] - got[1]).max() <= 1e-2 * got[1].std()


@pytest.mark.parametrize("gain", [0.25, 3.0, 6.0])
def test_maxima_that_rise_by_less_and_by_more_than_the_rescale_threshold(gain):
    """Unmasked steps keep a row's weights relative to a maximum that they follow only when it has risen by 2^8: scores of a
    standard deviation of 0.4, 4 and 9 (in powers of two) over 13 steps, so that rows never rescale after the first step, do so
    now and then, and do so often; runs that end in a step, on its edge and one token behind it.  Bar as above."""
    from paper_2506_24119_amd import binding as sb
    g = si.ModelGeometry("rise", 1, 128, 4, 2, 128, 128, 256, 1e4, qk_norm=True)
    w = si.make_weights(g, seed=17)
    w["layers"][0]["q_norm"] = (w["layers"][0]["q_norm"] * gain).astype(np.float32)
    rng = np.random.Generator(np.random.PCG64(18))
    lens, hist = [832, 833, 700, 64, 127], [0, 300, 64, 63, 1]
    seqs = [rng.integers(0, g.vocab, n).astype(np.int32) for n in lens]
    ids = np.arange(len(seqs), dtype=np.int32)
    sess = sb.Session(g, sb.weights_to_device(w), 180, len(seqs), 56, 3000, 860, page_order=si.make_page_order(180, 2), tune="trim=0")
    old = [b for b in range(len(seqs)) if hist[b]]
    sess.prefill(ids[old], [seqs[b][:hist[b]] for b in old])
    got = sess.prefill(ids, [s[h:] for s, h in zip(seqs, hist)]).cpu().numpy()
    sess.close()
    for b, s in enumerate(seqs):
        want = od.forward_full(g, w, s, logits_at=np.array([len(s) - 1]))[0]
        assert np.abs(got[b] - want).max() <= 3e-2 * want.std(), b


@pytest.mark.parametrize("head_dim,dtype", [(32, si.WEIGHT_FP32), (128, si.WEIGHT_BF16), (64, si.WEIGHT_BF16)])
@pytest.mark.parametrize("run,at,keep,more,tune", [
    (200, 186, 30, 150, None), (300, 286, 100, 185, None), (300, 286, 100, 185, "trim=0"),
    (60, 46, 40, 1, None), (300, 286, 280, 1, None), (300, 286, 280, 1, "chunk=16"), (300, 286, 285, 1, "wgs=768")])
def test_a_nan_behind_the_last_token(head_dim, dtype, run, at, keep, more, tune):
    """A run with a NaN token, cut back to before it and continued up to the same page, by a prefill whose last layer has one row and by a decode
    step, in every form of their attention: pages are not cleared, and a weight of zero does not stop a NaN.  Bound as above."""
    import torch
    from paper_2506_24119_amd import binding as sb
    assert at < run and keep <= at and keep + more <= at and (keep + more - 1) // 16 == at // 16
    g = si.ModelGeometry("nan", 2, 128, 256 // head_dim, 2, head_dim, 128, 256, 1e4, tie_lm_head=False, weight_dtype=dtype)
    w = si.make_weights(g, seed=17)
    w["embed"][7] = 0x7FC0 if dtype == si.WEIGHT_BF16 else np.nan
    wd = sb.weights_to_device(w)
    rng = np.random.Generator(np.random.PCG64(run + more))
    seq, new = rng.integers(8, g.vocab, run).astype(np.int32), rng.integers(8, g.vocab, more).astype(np.int32)
    got = []
    for tok in (7, 9):
        seq[at] = tok
        sess = sb.Session(g, wd, 24, 1, 24, 320, 320, page_order=si.make_page_order(24, 2), tune=tune)
        sess.prefill([0], [seq])
        sb.spiral_seq_truncate(sess.pool, [0], [keep])
        if more > 1:
            got.append(sess.prefill([0], [new]).cpu().numpy()[0])
        else:
            got.append(sess.decode_step(np.zeros(1, dtype=np.int32), torch.from_numpy(new).cuda(), sess.new_logits(1)).cpu().numpy()[0])
        sess.close()
    assert np.isfinite(got[0]).all()
    assert np.abs(got[0] - got[1]).max() <= 1e-2 * got[1].std()

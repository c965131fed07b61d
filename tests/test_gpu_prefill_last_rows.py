"""A prefill's last layer computes queries, attention, O and MLP for the last token of each sequence only: against the same call
with every row computed (spiral_model_tune "trim=0") and against the oracle, at the edges of the rule and where the two forms
differ most - one layer, a run of one token, histories, runs that end on a page boundary, more than 128 sequences."""
import numpy as np
import pytest

from oracle import decoder as od
from paper_2506_24119_amd import inputs as si

pytestmark = pytest.mark.gpu

LOGIT_TOL = 3e-2          # the bar of every logit comparison: half-precision activations


def _runs(total, B, rng):
    """B run lengths that add up to `total`, the first a single token, the second a multiple of the page size where there is room."""
    if B == 1:
        return [total]
    lens = rng.multinomial(total - B, np.full(B, 1.0 / B)) + 1
    lens[-1] += lens[0] - 1
    lens[0] = 1
    if B > 2 and lens[-1] > 16:
        d = 16 - lens[1] % 16
        lens[1] += d
        lens[-1] -= d
    return [int(n) for n in lens]


@pytest.mark.parametrize("layers,hd,rows,B,history,norm", [
    (2, 128, 129, 1, 0, True), (1, 128, 129, 3, 40, True), (2, 64, 131, 32, 20, False), (2, 128, 300, 75, 0, False),
    (3, 128, 700, 5, 300, True), (2, 128, 640, 160, 33, True)])
@pytest.mark.parametrize("repack", [True, False])
def test_last_rows_only(layers, hd, rows, B, history, norm, repack):
    import torch
    from paper_2506_24119_amd import binding as sb
    g = si.ModelGeometry("last", layers, 256, 512 // hd, 256 // hd, hd, 384, 512, 1e6, qk_norm=norm, qkv_bias=not norm)
    host = si.make_weights(g, seed=61)
    w = sb.weights_to_device(host)
    rng = np.random.Generator(np.random.PCG64(1000 * rows + B))
    lens = _runs(rows, B, rng)
    hist = [rng.integers(0, g.vocab, int(n)).astype(np.int32) for n in rng.integers(0, history + 1, B)]
    new = [rng.integers(0, g.vocab, n).astype(np.int32) for n in lens]
    ids = rng.permutation(B).astype(np.int32)
    step = rng.integers(0, g.vocab, B).astype(np.int32)
    blocks = [(len(h) + len(n) + 16) // 16 + 1 for h, n in zip(hist, new)]
    got, attn = [], []
    for tune in ("trim=1", "trim=0"):
        sess = sb.Session(g, w, sum(blocks), B, max(blocks), max(rows, sum(len(h) for h in hist)), 1100,
                          page_order=si.make_page_order(sum(blocks), 6), repack=repack, tune=tune)
        old = [i for i in range(B) if len(hist[i])]
        if old:
            sess.prefill(ids[old], [hist[i] for i in old])
        sb.spiral_profile_begin(sess.model, sb.KERNEL_CLASSES.index("attn_prefill"), 16)
        out = [sess.prefill(ids, new).cpu().numpy()]
        attn.append(sb.spiral_profile_end(sess.model)[1])
        out.append(sess.decode_step(ids, torch.from_numpy(step).cuda(), sess.new_logits(B)).cpu().numpy())     # reads the appended k and v
        assert sess.saturation_count() == 0
        got.append(out)
        sess.close()
    assert attn == [layers - 1, layers]
    for b in {0, 1 % B, B // 2, B - 1}:
        toks = np.concatenate([hist[b], new[b], step[b:b + 1]]).astype(np.int64)
        want = od.forward_full(g, host, toks, logits_at=np.array([len(toks) - 2, len(toks) - 1]))
        for k in range(2):
            for form in got:
                assert np.abs(form[k][b] - want[k]).max() <= LOGIT_TOL * want[k].std(), (b, k)
    for k in range(2):        # every row: the two forms differ by roundings only, each within the bar of the oracle
        assert np.abs(got[0][k] - got[1][k]).max() <= 2 * LOGIT_TOL * got[1][k].std()


@pytest.mark.parametrize("rows,B", [(128, 4), (259, 65)])
def test_every_row_below_the_rule(rows, B):
    """128 rows, and less than four rows to a sequence: nothing is left out."""
    from paper_2506_24119_amd import binding as sb
    g = si.ModelGeometry("last", 2, 256, 4, 2, 128, 384, 512, 1e6)
    w = sb.weights_to_device(si.make_weights(g, seed=62))
    rng = np.random.Generator(np.random.PCG64(rows))
    new = [rng.integers(0, g.vocab, n).astype(np.int32) for n in _runs(rows, B, rng)]
    sess = sb.Session(g, w, 2 * B + 20, B, 20, rows, 320, page_order=si.make_page_order(2 * B + 20, 6))
    sb.spiral_profile_begin(sess.model, sb.KERNEL_CLASSES.index("attn_prefill"), 16)
    sess.prefill(np.arange(B, dtype=np.int32), new)
    assert sb.spiral_profile_end(sess.model)[1] == 2
    sess.close()


@pytest.mark.parametrize("repack", [True, False])
def test_a_sequence_does_not_depend_on_the_contexts_of_its_call(repack):
    """Copies of a run at several places of a call, and the same run among other lengths and histories (the same sum of rows, from which
    the projections' K splits follow): the last layer's attention is cut from the pair's own first page, so all get the same bits.  By
    contexts of one piece of 16 pages (250 tokens) and of three (700)."""
    from paper_2506_24119_amd import binding as sb
    g = si.ModelGeometry("last", 2, 256, 4, 2, 128, 384, 512, 1e6, qk_norm=True)
    w = sb.weights_to_device(si.make_weights(g, seed=63))
    rng = np.random.Generator(np.random.PCG64(64))
    probes = {n: rng.integers(0, g.vocab, n).astype(np.int32) for n in (250, 700)}
    want = {}
    # lengths of the runs of a call, and of the histories in front of them; all calls append 4,000 tokens
    for lens, hist in (([250, 700, 333, 250, 700, 417, 650, 700], [0] * 8),
                       ([700, 601, 250, 10, 700, 700, 38, 250, 700, 51], [0] * 10),
                       ([1100, 250, 700, 700, 250, 1000], [500, 0, 0, 0, 0, 1400]), ([250] * 16, [0] * 16)):
        assert sum(lens) == 4000
        B = len(lens)
        ids = rng.permutation(B).astype(np.int32)
        old = [rng.integers(0, g.vocab, n).astype(np.int32) for n in hist]
        new = [probes[n] if n in probes and not h else rng.integers(0, g.vocab, n).astype(np.int32) for n, h in zip(lens, hist)]
        sess = sb.Session(g, w, 600, B, 152, 4000, 2500, page_order=si.make_page_order(600, B), repack=repack)
        kept = [b for b in range(B) if hist[b]]
        if kept:
            sess.prefill(ids[kept], [old[b] for b in kept])
        got = sess.prefill(ids, new).cpu().numpy()
        sess.close()
        for b in range(B):
            if lens[b] in probes and not hist[b]:
                assert np.array_equal(got[b], want.setdefault(lens[b], got[b])), (lens, b)

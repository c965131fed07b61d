"""The categorical sampler cuts a row into slices and passes over entries that cannot win without computing their noise.
Its tokens must be those of the truncated sampler's kernel with nothing cut, which scores every entry of a row in one
workgroup with the same expression - bit for bit, at slice edges, with scores so large that rounding makes ties, and with
infinities and NaN among the logits."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _both(logits, T, seed):
    import torch
    from paper_2506_24119_amd import binding as sb
    B, V = logits.shape
    ids, steps = np.arange(B, dtype=np.int32), (np.arange(B, dtype=np.int32) * 3 + 1).astype(np.int32)
    a = torch.full((B,), -7, dtype=torch.int32, device="cuda")
    b = torch.full((B,), -7, dtype=torch.int32, device="cuda")
    tau = torch.empty(B, dtype=torch.float32, device="cuda")
    for _ in range(2):                                   # a second call on a used output buffer
        sb.spiral_sample(logits, B, V, T, seed, ids, steps, None, a)
    sb.spiral_sample_truncated(logits, B, V, T, 0, 1.0, seed, ids, steps, None, b, tau)
    torch.cuda.synchronize()
    return a.cpu().numpy(), b.cpu().numpy()


@pytest.mark.parametrize("B,V", [(1, 1), (3, 7), (2, 8193), (1, 16383), (5, 16385), (3, 40001), (1, 151936), (130, 20000), (300, 2500)])
@pytest.mark.parametrize("T", [1.0, 0.6, 0.013])
def test_slices_and_screen_keep_every_token(B, V, T):
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(B * 1000 + V)
    for scale, shift in ((1.0, 0.0), (30.0, 5.0), (0.01, 1e5), (0.0, -3.0)):
        logits = torch.empty((B, V), device="cuda").normal_(0.0, 1.0, generator=gen) * scale + shift
        a, b = _both(logits, T, 11)
        assert np.array_equal(a, b), (scale, shift, np.flatnonzero(a != b)[:5])


def test_infinities_and_nan():
    import torch
    V = 20000                                            # two slices of 10000
    logits = torch.zeros((7, V), device="cuda")
    logits[0] = float("-inf")                            # nothing to choose from: the lowest index
    logits[1] = float("nan")                             # no score at all: index 0
    logits[2, :] = float("-inf"); logits[2, 9999] = -1e30
    logits[3, 5000] = float("inf"); logits[3, 15000] = float("inf")
    logits[4, 0] = float("nan"); logits[4, 4000:] = float("-inf")
    logits[5, :12000] = float("nan")
    logits[6, :] = torch.finfo(torch.float32).min; logits[6, 3] = 0.0
    a, b = _both(logits, 1.0, 5)
    assert np.array_equal(a, b), (a, b)
    assert a[0] == 0 and a[1] == 0 and a[2] == 9999 and a[3] == 5000 and a[4] != 0 and a[5] >= 12000 and a[6] == 3


@pytest.mark.parametrize("B,V", [(2, 20479), (2, 20480), (1, 24575), (1, 24576), (130, 41001), (128, 60000), (1, 49152), (2, 98303), (2, 98304)])
def test_every_form_keeps_every_token(B, V):
    """The lengths at which a row is cut (98,304 greedy, 49,152 with a noise buffer, 24,576 with generated noise) and at which
    a slice is screened (20,480 entries), each side; greedy and buffered noise against a plain argmax of the same fp32 scores."""
    import torch
    from paper_2506_24119_amd import binding as sb
    gen = torch.Generator(device="cuda")
    gen.manual_seed(V)
    logits = torch.empty((B, V), device="cuda").normal_(0.0, 2.0, generator=gen)
    noise = torch.empty((B, V), device="cuda").normal_(0.0, 1.0, generator=gen)
    for T in (1.0, 0.6):
        a, b = _both(logits, T, 3)
        assert np.array_equal(a, b), np.flatnonzero(a != b)[:5]
    ids, out = np.arange(B, dtype=np.int32), torch.full((B,), V, dtype=torch.int32, device="cuda")
    host, nz = logits.cpu().numpy(), noise.cpu().numpy()
    sb.spiral_sample(logits, B, V, 0.0, 1, ids, ids, None, out)
    assert np.array_equal(out.cpu().numpy(), host.argmax(1))
    sb.spiral_sample(logits, B, V, 0.6, 1, ids, ids, noise, out)
    assert np.array_equal(out.cpu().numpy(), (host / np.float32(0.6) + nz).argmax(1))


@pytest.mark.parametrize("B", [1, 128])
def test_infinities_and_nan_across_slices(B):
    """As above with rows that are cut: 18 slices of 8,441 entries (one row), two screened ones (128 rows)."""
    import torch
    V, half = 151936, 75968
    logits = torch.zeros((max(B, 7), V), device="cuda")
    logits[0] = float("-inf")
    logits[1] = float("nan")
    logits[2, :] = float("-inf"); logits[2, half - 1] = -1e30
    logits[3, 5000] = float("inf"); logits[3, half + 5000] = float("inf")
    logits[4, 0] = float("nan"); logits[4, 4000:] = float("-inf")
    logits[5, :half + 4000] = float("nan")
    logits[6, :] = torch.finfo(torch.float32).min; logits[6, half + 3] = 0.0
    want = {0: 0, 1: 0, 2: half - 1, 3: 5000, 6: half + 3}
    rows = [logits[i:i + 1].contiguous() for i in range(7)] if B == 1 else [logits]
    for i, r in enumerate(rows):
        a, b = _both(r, 1.0, 5)
        assert np.array_equal(a, b), (i, a, b)
        if B == 1:
            assert a[0] == want.get(i, a[0]) and (i != 4 or a[0] != 0) and (i != 5 or a[0] >= half + 4000)
        else:
            assert all(a[k] == v for k, v in want.items()) and a[4] != 0 and a[5] >= half + 4000

"""The categorical sampler reads four entries at once where the rows are 16-byte aligned and their length is a multiple of four, one
otherwise; its screen works on scaled logits, which overflow where the temperature is next to nothing.  Tokens must be those of the
truncated sampler's kernel with nothing cut, which does neither."""
import numpy as np
import pytest

from test_gpu_sample_slices import _both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [4, 12, 4096, 8200, 24580, 151936])
@pytest.mark.parametrize("shift", [0, 1, 3])
def test_rows_that_are_not_aligned(V, shift):
    import torch
    from paper_2506_24119_amd import binding as sb
    B = 3
    gen = torch.Generator(device="cuda")
    gen.manual_seed(V)
    store = torch.empty(B * V + 4, device="cuda").normal_(0.0, 2.0, generator=gen)
    logits = store[shift:shift + B * V].view(B, V)
    a, b = _both(logits, 1.0, 4)
    assert np.array_equal(a, b)
    ids, out = np.arange(B, dtype=np.int32), torch.full((B,), V, dtype=torch.int32, device="cuda")
    noise = torch.empty(B * V + 4, device="cuda").normal_(0.0, 1.0, generator=gen)[:B * V].view(B, V)
    host = logits.cpu().numpy()
    sb.spiral_sample(logits, B, V, 0.0, 1, ids, ids, None, out)
    assert np.array_equal(out.cpu().numpy(), host.argmax(1))
    sb.spiral_sample(logits, B, V, 0.6, 1, ids, ids, noise, out)
    assert np.array_equal(out.cpu().numpy(), (host / np.float32(0.6) + noise.cpu().numpy()).argmax(1))


@pytest.mark.parametrize("T", [1e-39, 3e-39, 1e-37, 1e-30, 1e30])
@pytest.mark.parametrize("scale", [1e-5, 1.0, 1e30])
def test_temperatures_at_the_ends(T, scale):
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    for V in (151936, 24576):
        logits = torch.empty((2, V), device="cuda").normal_(0.0, 1.0, generator=gen) * scale
        logits[1] = -logits[1].abs()                       # scores of one sign, most of them beyond the range
        a, b = _both(logits, T, 4)
        assert np.array_equal(a, b), (V, a, b)


@pytest.mark.parametrize("V", [2 ** 31 - 1, 2 ** 31 - 4])
def test_the_longest_rows(V):
    """The loads of the sampler and of the truncated one run a step ahead: past the end of a row whose length is the largest that the entry
    points take, in loads of one entry and of four.  All but the last 20,000 entries are -inf, whose noise never counts."""
    import torch
    from oracle import sampling as osp
    from oracle import truncated as otr
    from paper_2506_24119_amd import binding as sb
    n = 20000
    rng = np.random.Generator(np.random.PCG64(V % 1000))
    tail = rng.standard_normal(n).astype(np.float32)
    logits = torch.full((1, V), -float("inf"), dtype=torch.float32, device="cuda")
    logits[0, V - n:] = torch.from_numpy(tail).cuda()
    ids, steps = np.array([3], dtype=np.int32), np.array([8], dtype=np.int32)
    with np.errstate(over="ignore"):
        key = osp._mix(osp._mix(np.uint64(5) ^ osp._GOLD) + ((np.uint64(3) << np.uint64(32)) | np.uint64(8)))
        r = (osp._mix(key + np.arange(V - n, V, dtype=np.uint64) * osp._GOLD) >> np.uint64(32)).astype(np.uint32)
    noise = -np.log(-np.log(osp.uniform_from_bits(r), dtype=np.float32), dtype=np.float32)
    out = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    sb.spiral_sample(logits, 1, V, 0.0, 5, ids, steps, None, out)
    assert int(out) == V - n + int(tail.argmax())
    sb.spiral_sample(logits, 1, V, 1.0, 5, ids, steps, None, out)
    tok, margin = osp.sample_row(tail, 1.0, noise)
    assert margin > 1e-5 and int(out) == V - n + tok
    need = sb.spiral_sample_truncated_workspace_bytes(1, V)
    work = torch.empty(need, dtype=torch.uint8, device="cuda")
    for top_k, top_p in ((0, 0.9), (50, 1.0), (20, 0.9)):
        out.fill_(-1)
        sb.spiral_sample_truncated_ws(logits, 1, V, 1.0, top_k, top_p, 5, ids, steps, None, out, None, work, need)
        tok, margin, _, slack = otr.sample_row(tail, 1.0, top_k, top_p, noise)
        assert margin > 1e-5 and slack > 1e-6 and int(out) == V - n + tok, (top_k, top_p)

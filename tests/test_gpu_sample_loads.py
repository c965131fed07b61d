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

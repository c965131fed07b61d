"""The rules that choose a launch form from sizes, read from the library on the CPU (no GPU work): calls that one form serves
faster must not be sent to another."""
import ctypes as C

import pytest


@pytest.fixture(scope="module")
def lib():
    from paper_2506_24119_amd import binding
    return binding.load_library()


def rule(lib, mangled, restype, *argtypes):
    f = lib[mangled]
    f.restype, f.argtypes = restype, list(argtypes)
    return f


GREEDY, GENERATED, BUFFER = 0, 1, 2


def test_short_rows_of_the_categorical_sampler_stay_in_one_workgroup(lib):
    """Cutting a row costs a second launch (3 us): one workgroup a row is faster for greedy rows of 65,536 entries, buffered
    noise of 40,000 and generated noise of 20,000, whatever the number of rows."""
    slices = rule(lib, "_ZN6spiral13sample_slicesEiii", C.c_int, C.c_int, C.c_int, C.c_int)
    for rows in (1, 16, 72, 128):
        for mode, longest in ((GREEDY, 65536), (BUFFER, 40000), (GENERATED, 20000)):
            assert all(slices(rows, V, mode) == 1 for V in (1, 500, 4000, 16384, 20000, longest) if V <= longest)
        for mode in (GREEDY, GENERATED, BUFFER):
            assert slices(rows, 151936, mode) > 1 and slices(rows, 151936, mode) * 8192 <= 151936


def test_short_slices_are_not_screened(lib):
    """The screen visits one entry a thread in full first: 1.5 times the time at 4,000 entries, a gain from 24,576 on."""
    screens = rule(lib, "_ZN6spiral14sample_screensEi", C.c_bool, C.c_int)
    assert not any(screens(n) for n in (1, 4000, 9496, 16384)) and all(screens(n) for n in (24576, 75968))


def test_scoring_pairs_of_narrow_head_models_fit(lib):
    """The tiled LM head of the scoring pass needs a pair per row and 128 columns; a vocabulary of 151,936 on 12 + 2 + 2 heads of 128
    or 14 + 2 + 2 of 64 leaves room for them in the layers' products.  70,000 entries on one head of a 256-wide model do not."""
    fit = rule(lib, "_ZN6spiral15score_pairs_fitEiiiii", C.c_bool, *[C.c_int] * 5)
    assert fit(151936, 1536, 8960, 12 * 128, 2 * 128) and fit(151936, 896, 4864, 14 * 64, 2 * 64)
    assert fit(30000, 256, 384, 128, 128) and not fit(70000, 256, 384, 128, 128)


def test_both_forms_of_the_head_add_in_the_same_order(lib):
    """A step with the sampler inside draws the tokens of the sampler on that step's logits, bit for bit: the LM head of either comes
    from gemm_decode_kernel, whose order of sums is its own, or of neither.  The rule may not look at the epilogue; that the other kernels (of
    which the two forms may take different ones) add in one order is seen on the GPU.  Its lines: 32 rows, for small heads 128; those have at most
    2^25 weights and eight columns to a k."""
    takes = rule(lib, "_ZN6spiral17gemm_decode_takesEiiiib", C.c_bool, *[C.c_int] * 4, C.c_bool)
    STORE, SAMPLE = 0, 2
    for rows in (1, 32, 33, 64, 65, 96, 97, 128, 129, 500):
        for d in (128, 640, 1024, 2560, 3584):
            for vocab in (1008, 8192, 13120, 65520, 65536, 151936):
                assert takes(rows, vocab, d, STORE, True) == takes(rows, vocab, d, SAMPLE, True), (rows, d, vocab)
    for epilogue in (STORE, SAMPLE):
        head = lambda rows, vocab, d: takes(rows, vocab, d, epilogue, True)
        assert head(32, 151936, 1024) and not head(33, 151936, 1024) and not head(128, 151936, 2560)
        assert head(128, 8192, 2560) and not head(129, 8192, 2560) and not head(129, 1008, 128)
        assert head(128, 8192, 1024) and not head(33, 8208, 1024)                # eight columns to a k
        assert head(128, 16384, 2048) and not head(33, 16400, 2048) and head(128, 13104, 2560) and not head(33, 13120, 2560)      # 2^25 weights
        assert not head(32, 8192, 1088) and not head(32, 8196, 1024)             # widths that it does not take


def test_tiles_of_the_head_keep_to_the_streaming_kernels_shapes(lib):
    """Repacked heads may be tiled only where row-major ones go to the streaming kernel, which adds in the tiles' order: d_model a multiple of
    128 and a vocabulary of 16.  (Others go to a kernel that splits d_model over four waves.)"""
    tiled = rule(lib, "_ZN6spiral15gemm_head_tiledEiiii", C.c_bool, *[C.c_int] * 4)
    STORE, SAMPLE = 0, 2
    for rows in (64, 65, 100, 128, 129):
        for vocab, d in ((65536, 1088), (65540, 2560), (151944, 1024), (65536, 64), (151936, 2080)):
            assert not tiled(rows, vocab, d, STORE) and not tiled(rows, vocab, d, SAMPLE), (rows, vocab, d)
        assert tiled(rows, 151936, 2560, STORE) == (65 <= rows <= 128) and tiled(rows, 151936, 2560, SAMPLE) == (rows >= 65)

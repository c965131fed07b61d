"""Host-only guard on the register budget of the decode attention kernel: it runs three workgroups per compute unit
(three waves per SIMD), which holds only while a wave needs at most 168 vector registers and spills nothing.  An
innocent-looking source change can cost that occupancy (and a fifth of the kernel's bandwidth) without failing any
numerical test, so the compiler's own resource report is checked here."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_decode_attention_fits_three_waves_per_simd(tmp_path):
    from paper_2506_24119_amd import build as B
    if not (os.path.exists(B.HIPCC) or shutil.which(B.HIPCC)):
        pytest.skip("hipcc not available")
    src = os.path.join(B.CSRC, "kernels_attn.hip")
    cmd = [B.HIPCC] + B._flags() + ["-x", "hip", "--cuda-device-only", "-S", src, "-o", str(tmp_path / "attn.s")]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-2000:]
    asm = open(tmp_path / "attn.s").read()
    found = {}
    for m in re.finditer(r"\.name:\s+(\S+)\n(?:.*\n)*?\s+\.vgpr_count:\s+(\d+)\n\s+\.vgpr_spill_count:\s+(\d+)", asm):
        found[m.group(1)] = (int(m.group(2)), int(m.group(3)))
    stream = {k: v for k, v in found.items() if "attn_stream_kernel" in k}
    assert len(stream) >= 6, sorted(found)                      # head_dim 32 / 64 / 128 x two activation types
    for name, (vgprs, spills) in stream.items():
        assert vgprs <= 168 and spills == 0, (name, vgprs, spills)


def _resources(tmp_path, source):
    """{kernel: (vector registers, vector spills)} as the compiler reports them"""
    from paper_2506_24119_amd import build as B
    if not (os.path.exists(B.HIPCC) or shutil.which(B.HIPCC)):
        pytest.skip("hipcc not available")
    src = os.path.join(B.CSRC, source)
    cmd = [B.HIPCC] + B._flags() + ["-x", "hip", "--cuda-device-only", "-S", src, "-o", str(tmp_path / "k.s")]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-2000:]
    asm = open(tmp_path / "k.s").read()
    found = {}
    for m in re.finditer(r"\.name:\s+(\S+)\n(?:.*\n)*?\s+\.vgpr_count:\s+(\d+)\n\s+\.vgpr_spill_count:\s+(\d+)", asm):
        found[m.group(1)] = (int(m.group(2)), int(m.group(3)))
    return found


def test_prefill_attention_fits_two_waves_per_simd(tmp_path):
    prefill = {k: v for k, v in _resources(tmp_path, "kernels_attn.hip").items() if "attn_prefill_kernel" in k}
    assert len(prefill) == 6, sorted(prefill)                   # head_dim 32 / 64 / 128 x two activation types
    for name, (vgprs, spills) in prefill.items():
        assert vgprs <= 256 and spills == 0, (name, vgprs, spills)


def test_tiled_projections_keep_their_accumulators_in_registers(tmp_path):
    """One wave per SIMD has 512 registers, a 256-row tile's accumulators take half of them.  Tiles of 128 rows share a compute unit by two,
    which holds only up to 256.  Nothing spills.  Every kernel of the file is one of these, whatever it is called."""
    tile = _resources(tmp_path, "kernels_gemm_tile.hip")
    assert len([k for k in tile if "gemm_tile_kernel" in k]) == 6, sorted(tile)      # plain and SwiGLU of both heights, the fused q/k/v and the scoring head
    assert len([k for k in tile if "head_tile_kernel" in k]) == 3 and len(tile) == 9, sorted(tile)      # logits; winners of one row tile and of more
    for name, (vgprs, spills) in tile.items():
        tall = re.search(r"gemm_tile_kernelILi\d+ELi256E", name)
        assert vgprs <= (512 if tall else 256) and spills == 0, (name, vgprs, spills)


def test_projections_of_few_rows_keep_to_the_waves_they_are_built_for(tmp_path):
    """gemm_decode_kernel is built for one or two waves per SIMD (its last parameter): 512 or 256 registers, nothing spilled."""
    decode = _resources(tmp_path, "kernels_gemm_decode.hip")
    assert all("gemm_decode_kernel" in k for k in decode) and len(decode) == 52, sorted(decode)
    # 4 row tiles x 3 weight tiles x 2 epilogues x 2 weight orders, and the sampler's 4 row tiles
    for name, (vgprs, spills) in decode.items():
        waves = int(re.search(r"Li(\d+)EEEvNS", name).group(1))
        assert vgprs <= 512 // waves and spills == 0, (name, vgprs, spills)

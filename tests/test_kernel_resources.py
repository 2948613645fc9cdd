"""Registers of the compiled kernels: none spills to scratch memory.

A launch bound that the compiler cannot meet without spilling costs more than
the waves it buys; the compiler says nothing about it.  The device code is
compiled here as the library's is, with its resource remarks on."""

import os
import re
import subprocess

import pytest

from paper_2312_06827_amd import _build as B


def _scratch(source):
    """Kernel -> bytes of scratch memory per lane."""
    r = subprocess.run([B.HIPCC, *B.FLAGS, "--cuda-device-only",
                        "-Rpass-analysis=kernel-resource-usage", "-c",
                        os.path.join(B.CSRC, source), "-o", os.devnull],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    names = re.findall(r"Function Name: (\S+)", r.stderr)
    sizes = re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", r.stderr)
    assert names and len(names) == len(sizes)
    return {n: int(b) for n, b in zip(names, sizes)}


@pytest.mark.skipif(not os.path.exists(B.HIPCC), reason="no HIP compiler")
@pytest.mark.parametrize("source", ["variance.hip", "mlp.hip"])
def test_no_scratch_memory(source):
    spilled = {k: v for k, v in _scratch(source).items() if v}
    assert not spilled


@pytest.mark.skipif(not os.path.exists(B.HIPCC), reason="no HIP compiler")
@pytest.mark.parametrize("source", ["atrous_f32_2d.hip", "atrous_f16_2d.hip"])
def test_small_frame_level_has_no_scratch_memory(source):
    """Step 1 with one row per thread, as small frames and batches run it."""
    one_row = re.compile(r"(13atrous_tile_kI(f|DF16_)Li1ELi1E.*Lb0EEE|14atrous_batch_kI(f|DF16_)Li1ELi1E)")
    kernels = {k: v for k, v in _scratch(source).items() if one_row.search(k)}
    assert kernels
    assert not {k: v for k, v in kernels.items() if v}

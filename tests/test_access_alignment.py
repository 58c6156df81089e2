"""Rows of odd width put 16-bit vectors at 2-byte and fp32 vectors at 4-byte addresses. The vector types say
so, and the compiler reports where one reaches code that assumes the vector's own alignment: no source may."""
import os
import subprocess

import pytest

from paper_2404_03019_amd import build


@pytest.mark.parametrize("source", ["bwd_kernels.hip", "ep_bf16_i32.hip", "ep_f16_i64.hip", "ep_f32_i64.hip",
                                    "ep_join.hip"])
def test_vector_types_keep_their_alignment(source):
    flags = [f for f in build.FLAGS if not f.startswith("-W")]
    proc = subprocess.run([build.HIPCC, *flags, "-Walign-mismatch", "-fsyntax-only", os.path.join(build.CSRC, source)],
                          capture_output=True, text=True, timeout=300)
    assert proc.returncode == 0, proc.stderr[-2000:]
    assert "align-mismatch" not in proc.stderr, proc.stderr[-2000:]

"""Layout of the device code's shared structures, checked by compiling the
header (no GPU)."""

import os
import subprocess

import pytest

from paper_2207_03936_amd import build

WIDTHS = (64, 128, 256, 512, 1024)


@pytest.mark.parametrize("B", WIDTHS)
def test_vector_reads_of_the_shared_block_are_aligned(B, tmp_path):
    """Members that the stages read as one 16-byte vector lie on a multiple of
    16 bytes, in every width (the 64-lane events' blocks lie in dynamic LDS,
    each a multiple of 16 bytes long)."""
    src = tmp_path / "layout.hip"
    src.write_text(
        '#include <cstddef>\n#include "sbt_device.h"\nusing namespace sbt;\n'
        f"using S = Shared<{B}>;\n"
        'static_assert(alignof(S) % 16 == 0, "block");\n'
        'static_assert(offsetof(S, ctl) % 16 == 0, "step counters");\n'
        'static_assert(offsetof(S, mt) % 16 == 0, "module table");\n'
        f'static_assert(shared_block_bytes<{B}>() % 16 == 0, "region");\n')
    cmd = [build.hipcc()] + build.FLAGS + ["--offload-host-only", "-fsyntax-only", "-I", build.INCLUDE, "-I", build.CSRC,
                                           str(src)]
    res = subprocess.run(cmd, capture_output=True, text=True, cwd=os.path.dirname(src))
    assert res.returncode == 0, res.stderr

"""Layout of the device code's shared structures, checked by compiling the
header (no GPU)."""

import os
import subprocess

import pytest

from paper_2207_03936_amd import build

WIDTHS = (64, 128, 256, 512, 1024)
SLOTS = (256, 448, 480, 672, 768, 1024, 1536)


def _holds(tmp_path, head, conditions):
    """Compiles the device header with each condition as a static assertion."""
    src = tmp_path / "layout.hip"
    src.write_text('#include <cstddef>\n#include "sbt_device.h"\nusing namespace sbt;\n' + head +
                   "".join(f'static_assert({c}, "{c}");\n' for c in conditions))
    cmd = [build.hipcc()] + build.FLAGS + ["--offload-host-only", "-fsyntax-only", "-I", build.INCLUDE, "-I", build.CSRC,
                                           str(src)]
    res = subprocess.run(cmd, capture_output=True, text=True, cwd=os.path.dirname(src))
    assert res.returncode == 0, res.stderr


@pytest.mark.parametrize("B", WIDTHS)
def test_vector_reads_of_the_shared_block_are_aligned(B, tmp_path):
    """Members that the stages read as one 16-byte vector lie on a multiple of
    16 bytes, in every width (the 64-lane events' blocks lie in dynamic LDS,
    each a multiple of 16 bytes long)."""
    _holds(tmp_path, f"using S = Shared<{B}>;\n", [
        "alignof(S) % 16 == 0", "offsetof(S, ctl) % 16 == 0", "offsetof(S, mt) % 16 == 0",
        f"shared_block_bytes<{B}>() % 16 == 0"])


def test_forming_tracks_have_lanes_for_a_full_module(tmp_path):
    """In every compiled instance as many tracks fit the lanes' registers as a
    module of the slots' capacity has hits, or more."""
    _holds(tmp_path, "", [f"{B} * track_sets<{B}, {cap}>() >= {cap}" for B in WIDTHS for cap in SLOTS])


def test_grouped_events_fit_the_launch_bounds(tmp_path):
    """64-lane events: what a workgroup's LDS holds, its lanes may run."""
    _holds(tmp_path, "", [f"max_block_lanes<64, {cap}>() / 64 == 16 || "
                          f"(max_block_lanes<64, {cap}>() / 64 + 1) * event_region_bytes<64>({cap}, 0) > kMaxDynLds"
                          for cap in (0,) + SLOTS])


def test_compaction_reach_of_events_tracked_in_lds(tmp_path):
    """An event that the LDS form tracks names its hits by position, and its
    compaction still runs in LDS wherever links and tracks alone fit: in the
    plain form's 64 KiB and in each instance's LDS (26 full modules, at most
    16,384 hits)."""
    cases = [(65536, n) for n in (13900, 14100, 16384, 24400)]
    fits = [f"compact_form({n}, {lds}, true) != Compact::kMemory" for lds, n in cases]
    for cap in SLOTS:
        n, lds = min(26 * cap, 16384), f"(int)lds_bytes({cap}, 16384)"
        fits.append(f"compact_form({n}, {lds}, true) != Compact::kMemory || compact_form({n}, {lds}, false) == Compact::kMemory")
    _holds(tmp_path, "", fits + ["compact_form(13900, 65536, true) == Compact::kWhole",
                                 "compact_form(24700, 65536, true) == Compact::kMemory",
                                 "compact_form(24400, 65536, false) == Compact::kWhole"])

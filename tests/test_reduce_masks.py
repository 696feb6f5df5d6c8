"""The reduction of several slots at once (wave_reduce_slots, csrc/kernels.hpp) compiles only for the masks of sums
and maxima that its lane exchanges serve: with more than four slots, each pair of slots 2j and 2j + 1 alike."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1912_04263_amd", "csrc")


@pytest.mark.parametrize("slots,mask,served", [(6, 0x3F, True), (8, 0xF0, True), (5, 0x0, True), (8, 0x3C, True),
                                               (3, 0x5, True), (4, 0x2, True), (5, 0x1F, False), (8, 0x15, False),
                                               (6, 0x20, False)])
def test_masks(tmp_path, slots, mask, served):
    src = tmp_path / "mask.hip"
    src.write_text(f'#include "kernels.hpp"\n__device__ double probe(const double (&v)[{slots}]) '
                   f'{{ return qpg::wave_reduce_slots<{slots}, {mask}u>(v); }}\n')
    r = subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-arch=gfx950", "--cuda-device-only",
                        "-std=c++17", "-fsyntax-only", "-I", CSRC, str(src)], capture_output=True, text=True)
    assert (r.returncode == 0) == served, r.stderr
    if not served:
        assert "both sums or both maxima" in r.stderr

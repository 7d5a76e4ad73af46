"""The block layout that the segmented kernels' part form stages its runs in,
compiled for the host with the address and undefined-behaviour sanitizers
(tests/seg_blocks_units.cpp)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_block_layout_matches_the_flat_run(tmp_path):
    exe = str(tmp_path / "seg_blocks_units")
    subprocess.check_call([HIPCC, "-std=c++17", "-O1", "-g", "--offload-arch=gfx950", "--offload-host-only",
                           "-Xarch_host", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                           "-I", os.path.join(ROOT, "paper_1412_6862_amd", "csrc"), "-o", exe,
                           os.path.join(ROOT, "tests", "seg_blocks_units.cpp")], stderr=subprocess.DEVNULL)
    out = subprocess.run([exe], env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"), capture_output=True, text=True,
                         timeout=600)
    assert out.returncode == 0, out.stderr[-4000:]
    assert "seg blocks ok" in out.stdout

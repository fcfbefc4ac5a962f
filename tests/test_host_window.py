"""The staged step's 32-bit window at its edges (tests/native/window_edges.cpp), on the CPU:
with a window of all but 16 KB of the 4 GiB, a source in the first tiles was taken for one of
a workgroup's own where that lay within its own size of the window's end."""

import os
import subprocess

import pytest

from paper_1906_11925_amd import build as B

HERE = os.path.dirname(os.path.abspath(__file__))


def test_own_and_other_sources_at_the_windows_edges(tmp_path):
    try:
        cc = B.hipcc()
    except RuntimeError:
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "window_edges")
    subprocess.run([cc, "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17",
                    os.path.join(HERE, "native", "window_edges.cpp"), "-o", exe], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stdout

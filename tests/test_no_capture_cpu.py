"""The library captures no HIP graphs (runs without a GPU): two crashes of the host
process had a captured graph of a per-step context in play, and their cause was
not found."""
import subprocess

import pytest

sp = pytest.importorskip("paper_2303_07819_amd")


def test_library_uses_no_graph_or_capture_call():
    sp.load_library()
    names = subprocess.run(["nm", "-D", "--undefined-only", sp.LIB_PATH], capture_output=True, text=True,
                           check=True).stdout.split()
    assert "hipMalloc" in {n.split("@")[0] for n in names}
    assert not [n for n in names if n.startswith(("hipGraph", "hipStreamBeginCapture", "hipStreamEndCapture"))]

"""The plans that ordinary launches run, and what they are asked for on the host (no GPU)."""
import subprocess
import sys

import pytest

tc = pytest.importorskip("paper_1402_6601_amd")


@pytest.mark.parametrize("nb", [16, 128, 256, 512])
def test_workspace_of_an_empty_system(nb):
    """Order 0 is a valid size with nothing to do (in a process of its own: it
    used to end the process)."""
    try:
        tc.load()
    except ImportError as e:  # library not built
        pytest.skip(str(e))
    code = ("import paper_1402_6601_amd as tc; lib = tc.load(); "
            "print(lib.tchol_factor_solve_workspace_bytes(0, %d, 3), lib.tchol_workspace_bytes(0, 0, %d, 0))" % (nb, nb))
    r = subprocess.run([sys.executable, "-c", code], stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, timeout=120)
    assert r.returncode == 0, (r.returncode, r.stderr[-500:])
    both, factor = map(int, r.stdout.split())
    assert 0 < factor <= both < 1 << 20

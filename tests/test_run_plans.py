"""The plans that ordinary launches run, and what they are asked for on the host (no GPU)."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1402_6601_amd", "csrc")

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


@pytest.fixture(scope="module")
def host_check(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    exe = str(tmp_path_factory.mktemp("run_plans") / "run_plan_host")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-Wall", "-fno-omit-frame-pointer", "-fsanitize=address,undefined",
           "-fno-sanitize-recover=undefined", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
           os.path.join(ROOT, "tests", "run_plan_host.cpp"), os.path.join(CSRC, "plan.cpp"), "-o", exe]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-4000:]
    return exe


def test_data_flow_claim_order_and_items(host_check):
    """Two tile sizes in one plan, merged updates, POTRF with its inverse, fine
    work items: conflicts ordered, claim orders topological, outputs covered."""
    r = subprocess.run([host_check], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-4000:]
    assert r.stdout.rstrip().endswith(", 0 failures")


@pytest.mark.parametrize("kind", [0, 1, 2, 3, 4, 5, 6, 7, 12, 19])
def test_the_check_notices_missing_edges(host_check, kind):
    """Without the edges into one kind of task the check must fail."""
    r = subprocess.run([host_check, str(kind)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 1 and "not ordered" in r.stdout


def _query(op, n, nb, policy):
    try:
        return tc.plan_query(op, n, nb, policy)
    except ImportError as e:  # library not built
        pytest.skip(str(e))


@pytest.mark.parametrize("policy", [tc.POLICY_LIST, tc.POLICY_RANK, tc.POLICY_FIFO, tc.POLICY_RANDOM])
def test_query_of_the_run_plan(policy):
    """PLAN_RUN: tiles of 128 in the factorization, the caller's in the solve."""
    n, nb = 1600, 512
    run = _query(tc.OP_FACTOR_SOLVE, n, nb, policy | tc.PLAN_RUN)
    kinds = [tc.KIND_NAMES[k] for k in run["kind"]]
    assert kinds.count("POTRF") == 13 and kinds.count("FTRSV") == 4 and kinds.count("GEMM4") > 0
    assert sorted(set(run["item_task"])) == list(range(run["ntask"]))
    factor = _query(tc.OP_FACTOR, n, nb, policy | tc.PLAN_RUN)
    assert [tc.KIND_NAMES[k] for k in factor["kind"]].count("POTRF") == 13
    # without the flag, and for the operations that have one plan only
    assert [tc.KIND_NAMES[k] for k in _query(tc.OP_FACTOR, n, nb, policy)["kind"]].count("POTRF") == 4
    with pytest.raises(tc.TcholError):
        _query(tc.OP_SOLVE, n, nb, policy | tc.PLAN_RUN)
    with pytest.raises(tc.TcholError):
        _query(tc.OP_FACTOR, n, nb, -1)

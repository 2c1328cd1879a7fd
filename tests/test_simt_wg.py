"""Workgroup-local sweeps on the CPU emulation (tests/simt) with one wave of the
workgroup left behind at every barrier: every wave must leave a solve by the
same round, whatever another one meets meanwhile."""
import json
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, os.path.join(HERE, "simt"))
import build as simt_build  # noqa: E402
import pytest  # noqa: E402
import wg_build  # noqa: E402


def run(which, cus=1):
    wg_build.build()
    env = dict(os.environ, SIMT_CUS=str(cus), SIMT_LAG="1")
    asan = simt_build.asan_runtime()
    if asan:
        env["LD_PRELOAD"] = asan
        env["ASAN_OPTIONS"] = "detect_leaks=0:detect_stack_use_after_return=0"
    r = subprocess.run([sys.executable, os.path.join(HERE, "simt", "wg_cases.py"), which], env=env,
                       capture_output=True, text=True, timeout=900)
    assert r.returncode == 0, r.stderr[-4000:]
    return [json.loads(x) for x in r.stdout.splitlines() if x.startswith("{")]


def test_batch_instances_after_a_malformed_one():
    rows = run("batch")
    assert len(rows) == 12
    for x in rows:
        assert x["code"] == 2, x                      # LLP_E_INPUT: the first nonzero instance status
        assert x["bad"] == [2] * 3 and x["good"] == [0] * 9 and x["equal"], x


@pytest.mark.parametrize("cus", [1, 64])
def test_closures_well_formed_and_not(cus):
    """In groups of 32 rows, and (as many groups as CUs) of 16."""
    rows = run("closure", cus)
    assert len(rows) == 3 * 7
    for x in rows:
        assert x["code"] == 0 and x["equal"] if x["case"].endswith("None") else x["code"] == 2, x

"""Marked pull rounds against rounds that list their candidates, and the
oracle, on the CPU emulation (tests/simt): zero weights, a row longer than a
wave evaluates, vertices without arcs, overflow and ids out of range."""
import json
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, os.path.join(HERE, "simt"))
import build as simt_build  # noqa: E402


def test_marked_rounds_equal_listed_ones():
    simt_build.build()
    env = dict(os.environ, SIMT_CUS="4")
    asan = simt_build.asan_runtime()
    if asan:
        env["LD_PRELOAD"] = asan
        env["ASAN_OPTIONS"] = "detect_leaks=0:detect_stack_use_after_return=0"
    r = subprocess.run([sys.executable, os.path.join(HERE, "simt", "marked_cases.py")], env=env, capture_output=True,
                       text=True, timeout=900)
    assert r.returncode == 0, r.stderr[-4000:]
    rows = [json.loads(x) for x in r.stdout.splitlines() if x.startswith("{")]
    assert len(rows) == 5
    for x in rows:
        assert x["status"][0] == x["status"][1], x
        if x["status"][0] == 0:
            assert x["equal"] and x.get("oracle", True), x
    by = {x["case"]: x["status"][0] for x in rows}
    assert by["overflow"] == 4                                # LLP_E_OVERFLOW
    assert by["bad-out-id"] == by["bad-in-id"] == 2           # LLP_E_INPUT

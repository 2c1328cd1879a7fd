"""Small graphs under the hybrid schedule: the one-workgroup solve against
the grid-wide sweep and the oracle on the CPU emulation (tests/simt), over
block and step edges, hubs, multi-arcs, zero and negative weights, overflow
and ids out of range."""
import json
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, os.path.join(HERE, "simt"))
import build as simt_build  # noqa: E402


def test_small_graphs_equal_the_grid_wide_sweep():
    simt_build.build()
    env = dict(os.environ, SIMT_CUS="4")
    asan = simt_build.asan_runtime()
    if asan:
        env["LD_PRELOAD"] = asan
        env["ASAN_OPTIONS"] = "detect_leaks=0:detect_stack_use_after_return=0"
    r = subprocess.run([sys.executable, os.path.join(HERE, "simt", "small_cases.py")], env=env, capture_output=True,
                       text=True, timeout=900)
    assert r.returncode == 0, r.stderr[-4000:]
    rows = [json.loads(x) for x in r.stdout.splitlines() if x.startswith("{")]
    assert len(rows) == 2 * 15
    for x in rows:
        assert x["status"][0] == x["status"][1], x
        if x["status"][0] == 0:
            assert x["equal"] and x.get("oracle", True), x
    by = {(x["case"], x["kind"]): x["status"][0] for x in rows}
    assert by["overflow", "sssp"] == 4 and by["overflow", "bfs"] == 0      # LLP_E_OVERFLOW
    assert by["bad-id", "sssp"] == by["bad-id-low", "bfs"] == 2            # LLP_E_INPUT

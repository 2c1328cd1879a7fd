"""Small graphs of long rows under the hybrid schedule on the CPU emulation
(tests/simt) against the oracle: few vertices up to the limit on their arcs
are one launch and past it grid-wide rounds; hubs, hubs side by side, and
several blocks of vertices per wave."""
import json
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, os.path.join(HERE, "simt"))
import build as simt_build  # noqa: E402


def test_long_rows_and_few_vertices():
    simt_build.build()
    env = dict(os.environ, SIMT_CUS="4", SIMT_LAG="1")
    asan = simt_build.asan_runtime()
    if asan:
        env["LD_PRELOAD"] = asan
        env["ASAN_OPTIONS"] = "detect_leaks=0:detect_stack_use_after_return=0"
    r = subprocess.run([sys.executable, os.path.join(HERE, "simt", "dense_cases.py")], env=env, capture_output=True,
                       text=True, timeout=900)
    assert r.returncode == 0, r.stderr[-4000:]
    rows = [json.loads(x) for x in r.stdout.splitlines() if x.startswith("{")]
    assert len(rows) == 2 * 17
    for x in rows:
        assert x["status"] == 0 and x["equal"], x
    launches = {(x["case"], x["kind"]): x["launches"] for x in rows}
    for kind in ("sssp", "bfs"):
        for n, m in ((3, 50150), (64, 53200), (300, 65000)):
            assert launches[f"limit-{n}-{m}", kind] == 1
            assert launches[f"limit-{n}-{m + 1}", kind] > 1
        assert launches["hub-9000", kind] == launches["hubs", kind] == launches["rmat", kind] == 1

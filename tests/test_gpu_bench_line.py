"""What bench.py's line says about the PCG's form is what the timed solves ran.  Needs an MI355X."""
import json
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# bench.py's main, with the form that the library reports printed when the problem is closed
RUN = """
import sys, bench
from paper_2510_15271_amd import ba
close = ba.Problem.close
def closing(p):
    if getattr(p, "_h", None):
        print("form at close", p.pcg_form(), file=sys.stderr, flush=True)
    close(p)
ba.Problem.close = closing
bench.main()
"""


@pytest.mark.parametrize("args,label", [([], "resident (one launch per linear solve)"),
                                        (["--per-launch-pcg"], "one launch per iteration")])
def test_pcg_label(balib, args, label):
    """A 500-camera drive of 3000 points, one step and no other leg."""
    cmd = [sys.executable, "-c", RUN, "--steps", "1", "--warmup", "1", "--points", "3000", "--no-cpu-baseline",
           "--no-config0", "--no-refine", "--no-rig", "--no-pose-graph", "--loop-precisions", "", "--serving", "-1"]
    print("running", cmd[3:] + args, flush=True)
    r = subprocess.run(cmd + args, cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    out = json.loads(r.stdout.strip().splitlines()[-1])
    assert out["config"]["pcg"] == label
    form = balib.PCG_PER_LAUNCH if args else balib.PCG_AUTO
    assert f"form at close {form}" in r.stderr

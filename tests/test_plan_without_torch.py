"""The host calls of the binding (plans, symbols) run where torch is absent."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SCRIPT = """
import sys
sys.modules["torch"] = None  # import torch raises ImportError
import numpy as np
from paper_2405_02508_amd import mer
P = mer.plan_init(np.array([[0, 0, 0, 0, 3, 20, 64, 48]], np.int64))
assert P.total_px == 64 * 48 and mer.lib().mer_version() == 1
print("plan ok")
"""


def test_plans_are_made_without_torch():
    from paper_2405_02508_amd import mer
    if not os.path.exists(mer.LIB_PATH):
        from paper_2405_02508_amd import build
        build.build()
    r = subprocess.run([sys.executable, "-c", SCRIPT], cwd=ROOT, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "plan ok" in r.stdout, r.stderr[-2000:]

"""Plans made and loaded in a forked child of a process that has made plans
itself, as a pre-forking server or a data loader's workers do: neither may wait
for threads that only the parent has.  A fresh interpreter makes and saves a
plan large enough to be worth several threads, forks, and the child makes and
loads the same one."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = """
import os, signal, sys
import numpy as np
import paper_2509_12086_amd as saq

D = 512
M = np.random.default_rng(0).standard_normal((D, D)).astype(np.float32)
make = lambda: saq.Plan.from_parts([D // 2] * 2, [5, 3], M, np.zeros(D, np.float32))
path = sys.argv[1]
p = make()
p.save(path)
q = saq.Plan.load(path)
pid = os.fork()
if pid == 0:
    signal.alarm(20)          # a child that waits for a thread that is not there ends here
    a, b = make(), saq.Plan.load(path)
    same = all(np.array_equal(x.arrays()[0], M) and x.device_bytes() == p.device_bytes() for x in (a, b))
    os._exit(0 if same else 1)
_, status = os.waitpid(pid, 0)
sys.exit(0 if status == 0 else 3)
"""


@pytest.mark.parametrize("threads", ["1", "4"])
def test_plans_in_a_forked_child(tmp_path, threads):
    env = dict(os.environ, OMP_NUM_THREADS=threads, PYTHONPATH=ROOT)
    r = subprocess.run([sys.executable, "-c", CHILD, str(tmp_path / "plan.bin")], env=env, cwd=ROOT,
                       timeout=90, capture_output=True, text=True)
    assert r.returncode == 0, (r.returncode, r.stderr[-2000:])

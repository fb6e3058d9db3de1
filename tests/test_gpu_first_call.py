"""The first attention call of a process sets its device up, whatever the batch: what runs after it finds the set-up done."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = """
import numpy as np, torch
import paper_2602_14516_amd as A
import workloads as W
from gpu_util import DevBatch
b = W.make_batch(%s, %s, 8, 2, 64, 16, seed=3)
db = DevBatch(b)
first = A.mixed_batch_attn(db.cache, b.ctx_len, b.incr_len, db.bt, db.q, db.k_new, db.v_new)
out = torch.zeros_like(first)
A.mixed_batch_attn_static(db.cache, b.ctx_len, b.incr_len, db.bt, db.q, db.k_new, db.v_new, out)   # no ampd_init before it
assert torch.equal(out, first)
print("same", flush=True)
"""


@pytest.mark.parametrize("C,L", [([70, 300], [1, 1]), ([70], [40]), ([70, 300], [1, 40])], ids=["decode rows", "tile", "mixed"])
def test_first_call_sets_the_device_up(C, L):
    print("case: first call,", C, L, flush=True)
    env = dict(os.environ, PYTHONPATH=os.pathsep.join([ROOT, os.path.join(ROOT, "tests"), os.environ.get("PYTHONPATH", "")]))
    r = subprocess.run([sys.executable, "-c", CHILD % (C, L)], cwd=ROOT, env=env, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "same" in r.stdout, r.stdout + r.stderr

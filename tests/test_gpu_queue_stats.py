"""The load-balance build's records of small tensors (at most 16 processes use the GPU:
this test starts one)."""
import os
import subprocess
import sys

import pytest

from paper_2507_15121_amd import build

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = """
import numpy as np, torch
from paper_2507_15121_amd import api, queue_balance
rng = np.random.default_rng(0)
dims = (50, 40, 30)
for nnz in (1, 3000, 100_000):
    idx = np.stack([rng.integers(0, d, nnz) for d in dims]).astype(np.int32)
    t = api.Tensor(idx, np.ones(nnz, np.float32), dims)
    fac = [torch.ones((d, 16), device="cuda") for d in dims]
    for d in range(3):
        api.mttkrp(t, d, fac)
        torch.cuda.synchronize()
        rec, waves, hz = queue_balance._records(api.lib())
        assert rec.shape[0] > 0 and int(rec[:, 1].sum()) == nnz, (nnz, d, rec.shape, rec[:, 1].sum())
        assert queue_balance.summarize(rec, waves, hz)["span_us"] > 0
    t.close()
print("records ok")
"""


def test_records_of_small_tensors():
    if not os.path.exists(build.QSTATS_LIB):
        pytest.skip("libamped_qstats.so is not built")
    r = subprocess.run([sys.executable, "-c", PROGRAM], capture_output=True, text=True, timeout=100, cwd=ROOT,
                       env=dict(os.environ, AMPED_LIB=build.QSTATS_LIB))
    assert r.returncode == 0 and "records ok" in r.stdout, r.stdout + r.stderr[-2000:]

"""CP-ALS sweeps with modes on both sides of the row counts up to which the R x R
kernel adds the Gram partials itself (8 slabs of 256 rows) and computes the
factor itself (256 blocks of 4 entries per thread), against the oracle.

Tolerances: as in the other sweep tests, fp32 MTTKRP and Gram products (about
1e-6 relative) times cond(V), which is O(1) for these random factors: 1e-4 for
factors and lambda, 1e-5 for the fit."""
import numpy as np
import pytest

import oracle
from oracle import als
from gpu_util import log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2507_15121_amd import api  # noqa: E402


@pytest.mark.parametrize("rank,dims", [
    (16, (2048, 2049, 255)),
    (16, (16384, 16385, 64)),
    (24, (256 * 42, 256 * 42 + 1, 43)),
    (48, (256 * 85, 256 * 85 + 1, 86)),
    (64, (16384, 300, 16385)),
])
def test_sweep_at_fold_edges(rank, dims):
    rng = np.random.default_rng(rank + dims[0])
    nnz = 200000
    idx = np.stack([rng.integers(0, d, nnz) for d in dims]).astype(np.int32)
    val = rng.uniform(0, 1, nnz).astype(np.float32)
    F0 = [rng.uniform(-1, 1, (d, rank)).astype(np.float32) for d in dims]
    t = api.Tensor(idx, val, dims)
    dF = [torch.from_numpy(f).cuda() for f in F0]
    lam, fit = api.cp_als_sweep(t, dF)
    Fo, lo, fo = als.cp_als_sweep(idx, val, dims, [f.astype(np.float64) for f in F0])
    errs = [oracle.rel_fro(f.cpu().numpy(), o) for f, o in zip(dF, Fo)]
    log("R=%d dims %s: factors %.1e lambda %.1e fit %.1e" % (rank, dims, max(errs),
                                                            oracle.rel_fro(lam.cpu().numpy(), lo), abs(float(fit) - fo)))
    assert max(errs) <= 1e-4
    assert oracle.rel_fro(lam.cpu().numpy(), lo) <= 1e-4
    assert abs(float(fit) - fo) <= 1e-5
    t.close()

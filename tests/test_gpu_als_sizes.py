"""CP-ALS sweeps at the edges of the R x R kernel's register tiles (16, 32, 64,
96, 128) and of the Gram slabs (256 rows), against the oracle.

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


def _problem(dims, nnz, rank, seed):
    rng = np.random.default_rng(seed)
    idx = np.stack([rng.integers(0, d, nnz) for d in dims]).astype(np.int32)
    val = rng.uniform(0, 1, nnz).astype(np.float32)
    return idx, val, [rng.uniform(-1, 1, (d, rank)).astype(np.float32) for d in dims]


@pytest.mark.parametrize("rank", [1, 2, 7, 15, 16, 17, 31, 32, 33, 48, 63, 64, 65, 95, 96, 97, 127, 128])
@pytest.mark.parametrize("dims", [(1030, 700, 513), (600, 511, 400, 256)])
def test_sweep_at_rank_edges(rank, dims):
    idx, val, F0 = _problem(dims, 30000, rank, rank)
    t = api.Tensor(idx, val, dims)
    dF = [torch.from_numpy(f).cuda() for f in F0]
    lam, fit = api.cp_als_sweep(t, dF)
    Fo, lo, fo = als.cp_als_sweep(idx, val, dims, [f.astype(np.float64) for f in F0])
    errs = [oracle.rel_fro(f.cpu().numpy(), o) for f, o in zip(dF, Fo)]
    log("R=%d order %d: factors %.1e lambda %.1e fit %.1e" % (rank, len(dims), max(errs), oracle.rel_fro(lam.cpu().numpy(), lo),
                                                             abs(float(fit) - fo)))
    assert max(errs) <= 1e-4
    assert oracle.rel_fro(lam.cpu().numpy(), lo) <= 1e-4
    assert abs(float(fit) - fo) <= 1e-5
    t.close()


@pytest.mark.parametrize("rank", [12, 40, 70, 110])
def test_zero_column_and_reused_grams(rank):
    """A zero factor column (V singular: the tiny pivot) and a second sweep on
    the kept Gram matrices."""
    dims = (400, 300, 350)
    idx, val, F0 = _problem(dims, 20000, rank, rank)
    F0[1][:, rank // 2] = 0.0
    t = api.Tensor(idx, val, dims)
    dF = [torch.from_numpy(f).cuda() for f in F0]
    Fo = [f.astype(np.float64) for f in F0]
    for sweep in range(2):
        lam, fit = api.cp_als_sweep(t, dF, reuse_grams=sweep > 0)
        Fo, lo, fo = als.cp_als_sweep(idx, val, dims, Fo)
        assert max(oracle.rel_fro(f.cpu().numpy(), o) for f, o in zip(dF, Fo)) <= 1e-4
        assert oracle.rel_fro(lam.cpu().numpy(), lo) <= 1e-4
        assert abs(float(fit) - fo) <= 1e-5
        Fo = [f.cpu().numpy().astype(np.float64) for f in dF]
    t.close()

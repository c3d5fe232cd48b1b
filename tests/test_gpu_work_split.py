"""How the nonzeros are handed to the waves, at the edges of the split: every
chunk exactly once whether the grid has a wave for each of them or takes them
from the counters.  Integer inputs, whose sums are exact in fp32 in any order,
so every result equals the oracle's bit for bit."""
import numpy as np
import pytest

import oracle
from gpu_util import dev_factors, hip_mttkrp, log, oracle_mttkrp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2507_15121_amd import api  # noqa: E402


def int_problem(dims, nnz, rank, seed, heavy=0.2):
    """nnz random coordinates (duplicates add), a share of them in one mode-0 row."""
    rng = np.random.default_rng(seed)
    idx = np.stack([rng.integers(0, d, nnz) for d in dims]).astype(np.int32)
    idx[0, rng.random(nnz) < heavy] = dims[0] // 2
    val = rng.integers(1, 4, nnz).astype(np.float32)
    factors = [rng.integers(-2, 3, (d, rank)).astype(np.float32) for d in dims]
    return idx, val, factors


@pytest.mark.parametrize("chunks", [1, 7, 255, 256, 257, 2047, 2048, 2049, 4097, 30011])
def test_every_chunk_once(chunks):
    """Chunk counts around a grid of 256 blocks of 8 waves (and of 512 or 768 of 4)."""
    dims, rank = (900, 400, 300), 32
    idx, val, factors = int_problem(dims, chunks * 4 - 1, rank, chunks)
    t = api.Tensor(idx, val, dims, chunk_nnz=4)
    dfac = dev_factors(factors)
    loss_ref, _ = oracle.cp_loss(idx, val, [f.astype(np.float64) for f in factors])
    for d in range(3):
        np.testing.assert_array_equal(hip_mttkrp(t, d, dfac), oracle_mttkrp(idx, val, dims, factors, d).astype(np.float32))
        grad = torch.full((dims[d], rank), float("nan"), device="cuda")
        loss, _ = api.cp_loss_grad(t, d, dfac, -2.0, out=grad)
        np.testing.assert_array_equal(grad.cpu().numpy(), oracle.cp_grad(idx, val, dims, factors, d).astype(np.float32))
        assert float(loss) == loss_ref
    assert float(api.cp_loss(t, dfac)) == loss_ref
    log("%d chunks: exact" % chunks)
    t.close()


@pytest.mark.parametrize("nnz", [1, 255, 256, 257, 256 * 2048, 256 * 2048 + 1, 512 * 2048 + 1])
@pytest.mark.parametrize("rank", [16, 32, 128])
def test_library_sized_units(nnz, rank):
    """Units that the library sizes, around whole tiles of 256 nonzeros and
    whole rounds of 2048 waves; rows shared by many units and by none."""
    dims = (40_000, 300, 200)
    idx, val, factors = int_problem(dims, nnz, rank, nnz % 1000 + rank)
    t = api.Tensor(idx, val, dims)
    assert t.chunk_nnz == 4096   # the layout contract's chunks are as before
    dfac = dev_factors(factors)
    for d in (0, 2):
        np.testing.assert_array_equal(hip_mttkrp(t, d, dfac), oracle_mttkrp(idx, val, dims, factors, d).astype(np.float32))
    t.close()


def test_rows_kept_in_lds():
    """Enough nonzeros (2^25 and a few) that the launch copies the most-used rows
    to LDS first; they mix with other rows."""
    dims, rank = (3000, 2000, 900), 16
    rng = np.random.default_rng(9)
    nnz = (1 << 25) + 77
    idx = np.stack([np.minimum((d * rng.random(nnz, dtype=np.float32) ** 4).astype(np.int32), d - 1) for d in dims])
    val = rng.integers(0, 2, nnz).astype(np.float32)
    factors = [rng.integers(-1, 2, (d, rank)).astype(np.float32) for d in dims]
    t = api.Tensor(idx, val, dims)
    dfac, bfac = dev_factors(factors), dev_factors(factors, torch.bfloat16)
    ref = oracle_mttkrp(idx, val, dims, factors, 1)
    assert np.abs(ref).max() < 2 ** 24
    np.testing.assert_array_equal(hip_mttkrp(t, 1, dfac), ref.astype(np.float32))
    np.testing.assert_array_equal(hip_mttkrp(t, 1, bfac, bf16=True), ref.astype(np.float32))
    t.close()


@pytest.mark.parametrize("order", [2, 3, 4, 5])
@pytest.mark.parametrize("rank", [1, 2, 3, 4, 5, 6, 7, 8, 9, 11, 12, 15, 17, 20, 25, 31, 33, 48, 63, 65, 100, 127, 129, 200, 255, 256,
                                  257, 300, 513])
def test_any_rank(rank, order):
    """Ranks around every lane count of a row and every lane width: the last
    lanes' columns overlap, the last launch of a wide rank is narrower.  fp32 and
    bfloat16 factors (small integers are exact in both), and the residual forms
    where they are taken (ranks up to 64)."""
    rng = np.random.default_rng(rank * 10 + order)
    dims = (37, 30, 23, 11, 9)[:order]
    nnz = 3000 if rank <= 64 else 700
    idx = np.stack([rng.integers(0, d, nnz) for d in dims]).astype(np.int32)
    idx[0, idx[0] == 5] = 6          # an untouched row
    val = rng.integers(1, 4, nnz).astype(np.float32)
    factors = [rng.integers(-1, 2, (d, rank)).astype(np.float32) for d in dims]
    t = api.Tensor(idx, val, dims)
    dfac = dev_factors(factors)
    bfac = dev_factors(factors, torch.bfloat16)
    for d in range(order):
        ref = oracle_mttkrp(idx, val, dims, factors, d)
        assert np.abs(ref).max() < 2 ** 24
        np.testing.assert_array_equal(hip_mttkrp(t, d, dfac), ref.astype(np.float32))
        np.testing.assert_array_equal(hip_mttkrp(t, d, bfac, bf16=True), ref.astype(np.float32))
        if rank <= 64:
            grad = torch.full((dims[d], rank), float("nan"), device="cuda")
            loss, _ = api.cp_loss_grad(t, d, dfac, -2.0, out=grad)
            gref = oracle.cp_grad(idx, val, dims, factors, d)
            assert np.abs(gref).max() < 2 ** 24
            np.testing.assert_array_equal(grad.cpu().numpy(), gref.astype(np.float32))
            assert float(loss) == oracle.cp_loss(idx, val, [f.astype(np.float64) for f in factors])[0]
    if rank <= 64:
        assert float(api.cp_loss(t, dfac)) == oracle.cp_loss(idx, val, [f.astype(np.float64) for f in factors])[0]
    t.close()


def test_infinities_stay_in_their_columns():
    """A rank whose last lanes overlap: an infinite factor value changes the
    columns and residuals that hold it and no other (a column that two lanes
    hold enters a sum once)."""
    dims, rank, nnz = (20, 15, 10), 22, 400
    rng = np.random.default_rng(22)
    idx = np.stack([rng.integers(0, d, nnz) for d in dims]).astype(np.int32)
    val = rng.random(nnz).astype(np.float32) + 0.5
    factors = [rng.random((d, rank)).astype(np.float32) + 0.5 for d in dims]
    factors[1][3, 19] = np.inf
    t = api.Tensor(idx, val, dims)
    dfac = dev_factors(factors)
    with np.errstate(invalid="ignore"):
        ref = oracle_mttkrp(idx, val, dims, factors, 0)
    got = hip_mttkrp(t, 0, dfac)
    np.testing.assert_array_equal(np.isinf(got), np.isinf(ref))
    assert not np.isnan(got).any()
    assert np.isinf(float(api.cp_loss(t, dfac)))   # the squared residual of a hit entry, not NaN
    t.close()

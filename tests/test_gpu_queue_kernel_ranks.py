"""The queue's MTTKRP kernel at any rank: given chunk lengths keep small tensors out of
the one-launch kernel, so the lanes' overlap, launches of more than 256 columns, every
lane count and width and both factor types are those of the kernel that large tensors
take.  Integer inputs, against the oracle bit for bit."""
import numpy as np
import pytest

from gpu_util import dev_factors, hip_mttkrp, oracle_mttkrp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2507_15121_amd import api  # noqa: E402


@pytest.mark.parametrize("order", [2, 3, 4, 5])
@pytest.mark.parametrize("rank", [1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 15, 16, 18, 20, 25, 31, 32, 33, 34, 48, 63, 64, 65, 66, 100, 126,
                                  127, 128, 130, 200, 252, 254, 255, 256, 257, 258, 300, 512, 513, 514])
def test_any_rank(rank, order):
    """Around every lane count, lane width and launch width."""
    rng = np.random.default_rng(rank * 10 + order)
    dims = (37, 30, 23, 11, 9)[:order]
    nnz = 3000 if rank <= 64 else 700
    idx = np.stack([rng.integers(0, d, nnz) for d in dims]).astype(np.int32)
    idx[0, idx[0] == 5] = 6          # an untouched row
    val = rng.integers(1, 4, nnz).astype(np.float32)
    factors = [rng.integers(-1, 2, (d, rank)).astype(np.float32) for d in dims]
    t = api.Tensor(idx, val, dims, chunk_nnz=64 if rank % 2 else 250)
    dfac = dev_factors(factors)
    bfac = dev_factors(factors, torch.bfloat16)
    for d in range(order):
        ref = oracle_mttkrp(idx, val, dims, factors, d)
        assert np.abs(ref).max() < 2 ** 24
        np.testing.assert_array_equal(hip_mttkrp(t, d, dfac), ref.astype(np.float32))
        np.testing.assert_array_equal(hip_mttkrp(t, d, bfac, bf16=True), ref.astype(np.float32))
    t.close()


@pytest.mark.parametrize("rank", [22, 38, 70, 262])
@pytest.mark.parametrize("bf16", [False, True])
def test_infinities_stay_in_their_columns(rank, bf16):
    """Ranks whose last lanes overlap: an infinite factor value changes the columns that
    hold it and no other."""
    dims, nnz = (20, 15, 10), 400
    rng = np.random.default_rng(rank)
    idx = np.stack([rng.integers(0, d, nnz) for d in dims]).astype(np.int32)
    val = rng.random(nnz).astype(np.float32) + 0.5
    factors = [rng.integers(1, 4, (d, rank)).astype(np.float32) for d in dims]
    factors[1][3, rank - 3] = np.inf
    t = api.Tensor(idx, val, dims, chunk_nnz=64)
    with np.errstate(invalid="ignore"):
        ref = oracle_mttkrp(idx, val, dims, factors, 0)
    got = hip_mttkrp(t, 0, dev_factors(factors, torch.bfloat16 if bf16 else None), bf16=bf16)
    np.testing.assert_array_equal(np.isinf(got), np.isinf(ref))
    assert not np.isnan(got).any()
    t.close()

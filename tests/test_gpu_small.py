"""MTTKRP in one launch (tensors of up to 2^18 nonzeros whose units the library
sizes): units cut at row starts, rows that span units, rows that span more units
than the launch takes, untouched rows.  Integer inputs, exact in any order, against
the oracle bit for bit; every output starts as NaN."""
import numpy as np
import pytest

from gpu_util import dev_factors, hip_mttkrp, oracle_mttkrp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2507_15121_amd import api  # noqa: E402


def _tensor(lengths, rows, dims, seed):
    """Mode 0 has the given row lengths, at the given rows."""
    rng = np.random.default_rng(seed)
    i0 = np.repeat(np.asarray(rows, np.int32), lengths)
    nnz = i0.size
    idx = np.stack([i0] + [rng.integers(0, d, nnz).astype(np.int32) for d in dims[1:]])
    idx = np.ascontiguousarray(idx[:, rng.permutation(nnz)])
    return idx, rng.integers(1, 4, nnz).astype(np.float32)


def _check(idx, val, dims, rank, seed=0, repeats=2):
    rng = np.random.default_rng(seed)
    factors = [rng.integers(-1, 2, (d, rank)).astype(np.float32) for d in dims]
    t = api.Tensor(idx, val, dims)
    dfac, bfac = dev_factors(factors), dev_factors(factors, torch.bfloat16)
    for d in range(len(dims)):
        ref = oracle_mttkrp(idx, val, dims, factors, d)
        assert np.abs(ref).max(initial=0) < 2 ** 24
        for _ in range(repeats):   # what a launch leaves for the next one
            np.testing.assert_array_equal(hip_mttkrp(t, d, dfac), ref.astype(np.float32))
            np.testing.assert_array_equal(hip_mttkrp(t, d, bfac, bf16=True), ref.astype(np.float32))
    t.close()


@pytest.mark.parametrize("lengths", [[1], [63, 1], [64], [65], [128, 64], [192], [193], [191, 2, 193, 1], [256, 256, 256],
                                     [1] * 300, [64] * 40, [10, 2000, 10], [300, 300, 300, 5, 192, 192, 193],
                                     [4096], [4097, 1], [5000], [63, 64 * 63 + 2, 700, 1, 1, 9000]])
@pytest.mark.parametrize("rank", [5, 16, 32, 100])
def test_row_lengths(lengths, rank):
    """Around a unit (64), the longest unsplit row (192), and the most units of a
    row (64: a longer one sends the mode to the other kernel)."""
    rows = np.cumsum(np.random.default_rng(len(lengths)).integers(1, 30, len(lengths)))
    dims = (int(rows[-1]) + 40, 30, 20)
    idx, val = _tensor(lengths, rows, dims, sum(lengths))
    _check(idx, val, dims, rank)


@pytest.mark.parametrize("order,rank", [(2, 32), (3, 200), (3, 300), (4, 20), (5, 64), (6, 16)])
def test_orders_and_wide_ranks(order, rank):
    rng = np.random.default_rng(order)
    dims = (60, 45, 33, 12, 9, 7)[:order]
    nnz = 6000
    idx = np.stack([rng.integers(0, d, nnz) for d in dims]).astype(np.int32)
    idx[0, rng.random(nnz) < 0.2] = 7
    _check(idx, rng.integers(1, 3, nnz).astype(np.float32), dims, rank)


@pytest.mark.parametrize("nnz", [(1 << 17) - 1, 1 << 17, (1 << 17) + 1, 1 << 18, (1 << 18) + 1])
@pytest.mark.parametrize("dims", [(3000, 900, 500), (30_000, 20_000, 10_000)])
def test_unit_sizes(nnz, dims):
    """The unit's nominal size, and whether rows may be split, change at these
    counts; above the last the large kernel takes over."""
    rng = np.random.default_rng(nnz)
    idx = np.stack([np.minimum((d * rng.random(nnz) ** 1.5).astype(np.int32), d - 1) for d in dims])
    _check(idx, rng.integers(0, 2, nnz).astype(np.float32), dims, 16)


def test_rows_untouched_around_few_nonzeros():
    dims = (300_000, 50, 40)
    idx, val = _tensor([3, 400, 2], [5, 150_000, 299_990], dims, 1)
    _check(idx, val, dims, 24)


def test_same_bits_every_time():
    """Split rows are added in unit order, whoever arrives last: real-valued
    results do not vary from launch to launch."""
    rng = np.random.default_rng(8)
    dims = (50, 400, 300)
    idx = np.stack([rng.integers(0, d, 60_000) for d in dims]).astype(np.int32)
    t = api.Tensor(idx, rng.random(60_000).astype(np.float32), dims)
    dfac = dev_factors([rng.random((d, 32)).astype(np.float32) for d in dims])
    first = hip_mttkrp(t, 0, dfac)
    for _ in range(20):
        np.testing.assert_array_equal(hip_mttkrp(t, 0, dfac).view(np.uint32), first.view(np.uint32))
    t.close()

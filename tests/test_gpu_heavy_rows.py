"""Rows that span many work units: their pieces are added in fp64, so their error
does not grow with the number of units.  All inputs positive, so every partial sum
grows and an fp32 sum of n pieces would be off by about sqrt(n / 36) * 2^-23."""
import numpy as np
import pytest

from gpu_util import dev_factors

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2507_15121_amd import api  # noqa: E402

# A result is rounded to fp32 once (2^-24 at most).  What a piece brings with it is a
# group's serial sum of up to 512 terms, sqrt(512 / 36) * 2^-23 = 4.5e-7 at the most,
# independent over the hundreds of groups' runs of a heavy row (8 or more units of 1 to
# 32 groups), which leaves 4.5e-7 / sqrt(8) at the least many and 3e-8 at 200.
ROUNDED = 2.0 ** -24


def _positive(nnz, share, rank, seed):
    rng = np.random.default_rng(seed)
    dims = (3000, 700, 500)
    idx = np.stack([rng.integers(0, d, nnz) for d in dims]).astype(np.int32)
    idx[0, rng.random(nnz) < share] = 1234
    val = rng.random(nnz, dtype=np.float32) + np.float32(0.1)
    return dims, idx, val, [rng.random((d, rank), dtype=np.float32) + np.float32(0.1) for d in dims]


def _row_in_fp64(idx, val, factors, row):
    at = np.flatnonzero(idx[0] == row)
    p = val[at].astype(np.float64)[:, None]
    return (p * factors[1][idx[1, at]].astype(np.float64) * factors[2][idx[2, at]].astype(np.float64)).sum(0), at


def _err(got, ref):
    return float(np.linalg.norm(got.astype(np.float64) - ref) / np.linalg.norm(ref))


# units of 256 (300k nonzeros), 1024 (2M, and 6M of the queue) and 2560 (5M) nonzeros
@pytest.mark.parametrize("nnz,share", [(300_000, 0.5), (2_000_000, 0.3), (5_000_000, 0.3), (6_000_000, 0.3)])
@pytest.mark.parametrize("rank", [8, 32, 50])
def test_heavy_row(nnz, share, rank):
    dims, idx, val, factors = _positive(nnz, share, rank, rank)
    t = api.Tensor(idx, val, dims)
    dfac = dev_factors(factors)
    ref, _ = _row_in_fp64(idx, val, factors, 1234)
    got = api.mttkrp(t, 0, dfac).cpu().numpy()[1234]
    again = api.mttkrp(t, 0, dfac).cpu().numpy()[1234]
    assert _err(got, ref) <= ROUNDED + 3e-8
    np.testing.assert_array_equal(got.view(np.uint32), again.view(np.uint32))   # one order of the pieces
    bf = [f.to(torch.bfloat16) for f in dfac]
    refb, _ = _row_in_fp64(idx, val, [f.float().cpu().numpy() for f in bf], 1234)
    assert _err(api.mttkrp_bf16(t, 0, bf).cpu().numpy()[1234], refb) <= ROUNDED + 3e-8
    t.close()


@pytest.mark.parametrize("nnz,share", [(300_000, 0.5), (6_000_000, 0.3), (9_000_000, 0.3)])
def test_heavy_row_of_a_gradient(nnz, share):
    """The residual forms take up to 5 units at a time.  Negative residuals all: their
    sums grow too.  A residual has the rounding of its own 32 products, at most 2^-23 of
    the model's value, which is at most twice its own size here."""
    rank = 32
    dims, idx, val, factors = _positive(nnz, share, rank, 3)
    t = api.Tensor(idx, val, dims)
    dfac = dev_factors(factors)
    _, at = _row_in_fp64(idx, val, factors, 1234)
    p = factors[1][idx[1, at]].astype(np.float64) * factors[2][idx[2, at]].astype(np.float64)
    e = val[at].astype(np.float64) - p @ factors[0][1234].astype(np.float64)
    assert e.max() < 0
    ref = -2.0 * (e[:, None] * p).sum(0)
    got = api.cp_grad(t, 0, dfac, -2.0).cpu().numpy()[1234]
    assert _err(got, ref) <= ROUNDED + 6e-8
    t.close()


def test_heavy_row_of_streamed_layouts():
    """Streamed shards add into the row one after the other, in units of 4096 where a row
    spans many units: 29 pieces here and 15 of the shards' rounding (sqrt(44 / 36) * 2^-23
    at most, and a serial sum of 512 over 8 groups)."""
    dims, idx, val, factors = _positive(400_000, 0.3, 32, 4)
    t = api.Tensor(idx, val, dims, host_layout=True, shard_nnz=1 << 15)
    dfac = dev_factors(factors)
    ref, _ = _row_in_fp64(idx, val, factors, 1234)
    assert _err(api.mttkrp(t, 0, dfac).cpu().numpy()[1234], ref) <= 2.2e-7
    t.close()


@pytest.mark.parametrize("lengths", [[2048], [2304], [2305, 1, 2048 + 255], [1, 5000, 7, 9000, 300, 4000, 2], [255, 2049, 2303]])
@pytest.mark.parametrize("rank", [3, 16, 100, 300])
def test_rows_around_the_least_units(lengths, rank):
    """Rows of just under and over 8 unit edges, next to each other, exact on integers:
    both kernels' rows of 256-nonzero units (order 6 and the gradients take the queue's
    kernel at this size)."""
    rng = np.random.default_rng(len(lengths))
    rows = np.cumsum(rng.integers(1, 4, len(lengths)))
    i0 = np.repeat(rows, lengths).astype(np.int32)
    dims = (int(rows[-1]) + 2, 5, 4, 3, 3, 2)
    nnz = i0.size
    idx = np.ascontiguousarray(np.stack([i0] + [rng.integers(0, d, nnz).astype(np.int32) for d in dims[1:]]))
    val = rng.integers(1, 3, nnz).astype(np.float32)
    factors = [rng.integers(-1, 2, (d, rank)).astype(np.float32) for d in dims]
    from gpu_util import hip_mttkrp, oracle_mttkrp
    import oracle
    t = api.Tensor(idx, val, dims)
    dfac = dev_factors(factors)
    for d in range(len(dims)):
        ref = oracle_mttkrp(idx, val, dims, factors, d)
        for _ in range(2):
            np.testing.assert_array_equal(hip_mttkrp(t, d, dfac), ref.astype(np.float32))
    t.close()
    if rank <= 64:
        t = api.Tensor(idx[:3], val, dims[:3])
        for d in range(3):
            got = torch.full((dims[d], rank), float("nan"), device="cuda")
            api.cp_grad(t, d, dfac[:3], -2.0, out=got)
            np.testing.assert_array_equal(got.cpu().numpy(), oracle.cp_grad(idx[:3], val, dims[:3], factors[:3], d).astype(np.float32))
        t.close()


def test_heavy_row_of_a_large_tensor():
    """Units of 4096 (from 2^26 nonzeros on): a row of 13.4M nonzeros spans 3280 of them.
    A unit's sum is 8 groups' of 512 terms each: sqrt(512 / 36) * 2^-23 / sqrt(8 * 3280) =
    2.8e-9 beside the rounding, and what little a group's sums are biased by."""
    nnz, rank = (1 << 26) + 100_001, 32
    gen = torch.Generator(device="cuda").manual_seed(5)
    dims = (40_000, 30_000, 20_000)
    idx = torch.stack([torch.randint(d, (nnz,), generator=gen, device="cuda", dtype=torch.int32) for d in dims])
    idx[0][torch.rand(nnz, generator=gen, device="cuda") < 0.2] = 777
    val = torch.rand(nnz, generator=gen, device="cuda") + 0.1
    dev = [torch.rand((d, rank), generator=gen, device="cuda") + 0.1 for d in dims]
    ref = torch.zeros(rank, dtype=torch.float64, device="cuda")
    for at in torch.nonzero(idx[0] == 777)[:, 0].split(1 << 20):
        ref += (val[at].double()[:, None] * dev[1][idx[1, at].long()].double() * dev[2][idx[2, at].long()].double()).sum(0)
    t = api.Tensor(idx.cpu().numpy(), val.cpu().numpy(), dims)
    got = api.mttkrp(t, 0, dev)[777]
    assert torch.equal(got, api.mttkrp(t, 0, dev)[777])
    assert float((got.double() - ref).norm() / ref.norm()) <= ROUNDED + 3e-8
    grad = api.cp_grad(t, 0, dev, -2.0)
    assert torch.equal(grad[777], api.cp_grad(t, 0, dev, -2.0)[777])
    t.close()

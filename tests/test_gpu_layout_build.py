"""The device layout build against the host builder (itself pinned to the oracle
on the CPU): the same permutation, arrays and chunk flags, bit for bit, on
every way through it."""
import numpy as np
import pytest

from gpu_util import dev_factors, hip_mttkrp, log, oracle_mttkrp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2507_15121_amd import api  # noqa: E402


def _check(idx, val, dims, chunk=64, **kw):
    t = api.Tensor(idx, val, dims, chunk_nnz=chunk, keep_perm=True, **kw)
    for d in range(len(dims)):
        perm, flags = api.layout_host(idx, dims, d, chunk)
        got = t.layout(d, perm=True)
        np.testing.assert_array_equal(got["perm"], perm)
        np.testing.assert_array_equal(got["flags"], flags)
        np.testing.assert_array_equal(got["out_idx"], idx[d][perm])
        np.testing.assert_array_equal(got["in_idx"], np.delete(idx, d, axis=0)[:, perm])
        np.testing.assert_array_equal(got["values"], val[perm])
        assert t.touched[d] == np.unique(idx[d]).size
    return t


def _coo(dims, nnz, seed, sort):
    rng = np.random.default_rng(seed)
    idx = np.stack([rng.integers(0, d, nnz) for d in dims]).astype(np.int32)
    if sort:
        idx = np.ascontiguousarray(idx[:, np.lexsort(idx[::-1])])
    return idx, rng.random(nnz).astype(np.float32)


@pytest.mark.parametrize("sort", [False, True])
@pytest.mark.parametrize("dims", [(70, 300), (5, 70000, 300), (1, 40, 1, 30), (300, 1, 70000), (20, 30, 10, 15, 12),
                                  (9, 8, 7, 6, 5, 4, 3), (5, 4, 3, 6, 5, 4, 3, 2), (1, 1, 1)])
@pytest.mark.parametrize("nnz", [1, 5000])
def test_orders_and_sort_passes(dims, nnz, sort):
    """Every number of sort passes per mode (0 to 3), records of 16, 32 and 48
    bytes, sorted and unsorted input with duplicates; with a byte cap, wide
    records give way to a copy of the columns."""
    idx, val = _coo(dims, nnz, nnz + len(dims), sort)
    _check(idx, val, dims).close()
    _check(idx, val, dims, device_byte_cap=1 << 30).close()


def test_input_sorted_at_first_only():
    """The first 20,000 entries are in order, the rest is not."""
    dims = (900, 80, 70)
    idx, val = _coo(dims, 60_000, 5, True)
    idx[:, 20_000:] = idx[:, 20_000:][:, ::-1]
    _check(idx, val, dims).close()


@pytest.mark.parametrize("sort", [False, True])
def test_columns_copied_in_pieces(sort):
    """Columns of more than one upload piece (8 MB)."""
    dims = (40_000, 3_000, 500)
    idx, val = _coo(dims, 4_400_003, 6, sort)
    _check(idx, val, dims, chunk=4096).close()


@pytest.mark.parametrize("mode,at", [(0, 0), (2, 49_999), (1, 17_000)])
@pytest.mark.parametrize("sort", [False, True])
def test_bad_index_named(mode, at, sort):
    dims = (100, 90, 80)
    idx, val = _coo(dims, 50_000, 7, sort)
    idx[mode, at] = dims[mode] if at else -1
    with pytest.raises(api.AmpedError) as e:
        api.Tensor(idx, val, dims)
    assert e.value.status == api.ERR_RANGE
    assert "indices[%d][%d] = %d outside [0, %d)" % (mode, at, idx[mode, at], dims[mode]) in e.value.message


@pytest.mark.parametrize("unit", [1, 5, 256])
def test_row_lists_cover_every_untouched_and_shared_row(unit):
    """Gaps of every kind before, between and after touched rows: single rows,
    15, 16 and 17 rows, and runs cut into many pieces; rows that span many work
    units.  Every output row must be written (the outputs start as NaN)."""
    rng = np.random.default_rng(unit)
    rows, r = [], 3
    for gap in list(range(1, 40)) + [2047, 2048, 2049, 4096, 300_000]:
        rows += [r] * int(rng.integers(1, 4))
        r += gap + 1
    rows += [r] * 700
    dims = (r + 5000, 40, 30)
    nnz = len(rows)
    idx = np.stack([np.array(rows), rng.integers(0, 40, nnz), rng.integers(0, 30, nnz)]).astype(np.int32)
    idx = idx[:, rng.permutation(nnz)]
    val = rng.integers(1, 4, nnz).astype(np.float32)
    factors = [rng.integers(-2, 3, (d, 16)).astype(np.float32) for d in dims]
    t = api.Tensor(idx, val, dims, chunk_nnz=unit)
    dfac = dev_factors(factors)
    for d in range(3):
        np.testing.assert_array_equal(hip_mttkrp(t, d, dfac), oracle_mttkrp(idx, val, dims, factors, d).astype(np.float32))
    log("units of %d: exact" % unit)
    t.close()

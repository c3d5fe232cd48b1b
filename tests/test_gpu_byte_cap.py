"""options.device_byte_cap is an upper bound: a tensor that is created under a cap holds
at most that many device bytes, whatever its calls would like to have beside the
layouts, and its results are those of one without a cap."""
import numpy as np
import pytest

from gpu_util import dev_factors, hip_mttkrp, oracle_mttkrp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2507_15121_amd import api  # noqa: E402


def _admitted(make, cap):
    try:
        return make(cap)
    except api.AmpedError as e:
        assert e.status == 3, e   # NOMEM
        return None


def _caps(make):
    """The least cap that is admitted, then others up to well above what is held without one."""
    free = make(0)
    top = 4 * free.device_bytes + (1 << 22)
    free.close()
    lo, hi = 0, top
    while hi - lo > 1:
        mid = (lo + hi) // 2
        t = _admitted(make, mid)
        if t is None:
            lo = mid
        else:
            t.close()
            hi = mid
    caps = [hi]
    while caps[-1] < top:
        caps.append(int(caps[-1] * 1.07) + 1)
    return caps


def _check(idx, val, dims, make, every=1):
    rng = np.random.default_rng(5)
    factors = [rng.integers(-1, 2, (d, 16)).astype(np.float32) for d in dims]
    dfac = dev_factors(factors)
    ref = [oracle_mttkrp(idx, val, dims, factors, d).astype(np.float32) for d in range(len(dims))]
    caps = _caps(make)
    for k, cap in enumerate(caps):
        t = make(cap)
        assert t.device_bytes <= cap, (t.device_bytes, cap)
        if k % every == 0:
            for d in range(len(dims)):
                np.testing.assert_array_equal(hip_mttkrp(t, d, dfac), ref[d])
        t.close()


def _problem(dims, nnz, seed, heavy=0.2):
    rng = np.random.default_rng(seed)
    idx = np.stack([rng.integers(0, d, nnz) for d in dims]).astype(np.int32)
    for w in range(len(dims)):
        idx[w, rng.random(nnz) < heavy / (w + 1)] = dims[w] // 2
    return idx, rng.integers(1, 3, nnz).astype(np.float32)


@pytest.mark.parametrize("order", [2, 3, 5, 8])
@pytest.mark.parametrize("nnz", [1, 300, 5000])
def test_small_tensors(order, nnz):
    dims = (40, 30, 9, 8, 7, 5, 3, 2)[:order]
    idx, val = _problem(dims, nnz, nnz + order)
    _check(idx, val, dims, lambda cap: api.Tensor(idx, val, dims, device_byte_cap=cap), every=4)


@pytest.mark.parametrize("nnz,rows", [(100_000, 400), (131_072, 3000), (300_000, 20_000)])
def test_split_and_heavy_rows(nnz, rows):
    """Shares of split rows and slots of heavy ones in every mode."""
    dims = (rows, rows // 2, rows // 4)
    idx, val = _problem(dims, nnz, rows, heavy=0.03)
    _check(idx, val, dims, lambda cap: api.Tensor(idx, val, dims, device_byte_cap=cap), every=6)


@pytest.mark.parametrize("order,nnz,shard,chunk", [(2, 3000, 1, 1), (3, 20_000, 300, 100), (3, 200_000, 4096, 0), (8, 5000, 256, 256)])
def test_streamed_layouts(order, nnz, shard, chunk):
    """Many more nonzeros than a shard holds: what grows with them stays on the host."""
    dims = (40, 30, 9, 8, 7, 5, 3, 2)[:order]
    idx, val = _problem(dims, nnz, nnz + order)
    _check(idx, val, dims, lambda cap: api.Tensor(idx, val, dims, host_layout=True, shard_nnz=shard, chunk_nnz=chunk,
                                                  device_byte_cap=cap), every=9)


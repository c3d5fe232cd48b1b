"""Host-resident layouts as packed blocks of 256 nonzeros: the layout that comes
back is the host builder's bit for bit, and streamed results equal the oracle on
integer inputs, with shards that start and end anywhere in a block."""
import numpy as np
import pytest

import oracle
from gpu_util import dev_factors, hip_mttkrp, oracle_mttkrp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2507_15121_amd import api  # noqa: E402


@pytest.mark.parametrize("dims", [(2 ** 31 - 1, 5, 70_000), (1, 1, 3), (33, 2 ** 20 + 1), (3, 4, 5, 6, 7, 8, 9, 10)])
@pytest.mark.parametrize("nnz", [1, 255, 256, 257, 5000])
def test_layout_comes_back(dims, nnz):
    """Index widths from 0 to 31 bits, whole and partial blocks."""
    rng = np.random.default_rng(nnz)
    idx = np.stack([rng.integers(0, d, nnz) for d in dims]).astype(np.int32)
    idx[0, 0] = dims[0] - 1
    val = rng.standard_normal(nnz).astype(np.float32)
    modes = [d for d in range(len(dims))]
    t = api.Tensor(idx, val, dims, chunk_nnz=100, keep_perm=True, host_layout=True, shard_nnz=300)
    for d in modes:
        perm, flags = api.layout_host(idx, dims, d, 100)
        got = t.layout(d, perm=True)
        np.testing.assert_array_equal(got["perm"], perm)
        np.testing.assert_array_equal(got["flags"], flags)
        np.testing.assert_array_equal(got["out_idx"], idx[d][perm])
        np.testing.assert_array_equal(got["in_idx"], np.delete(idx, d, axis=0)[:, perm])
        np.testing.assert_array_equal(got["values"].view(np.uint32), val[perm].view(np.uint32))
    t.close()


@pytest.mark.parametrize("chunk,shard", [(1, 1), (7, 100), (64, 192), (100, 300), (256, 256), (0, 5000), (0, 0)])
def test_calls_in_a_row_share_the_buffers(chunk, shard):
    """Modes, bfloat16 factors, gradients and the loss one after the other with no
    wait between them: a call's copies start while the previous one's kernels
    still run."""
    rng = np.random.default_rng(chunk + shard)
    dims, nnz, rank = (900, 300, 200), (600 if chunk == 1 else 9000), 32
    idx = np.stack([rng.integers(0, d, nnz) for d in dims]).astype(np.int32)
    idx[0, rng.random(nnz) < 0.2] = 450
    val = rng.integers(1, 4, nnz).astype(np.float32)
    factors = [rng.integers(-2, 3, (d, rank)).astype(np.float32) for d in dims]
    t = api.Tensor(idx, val, dims, chunk_nnz=chunk, host_layout=True, shard_nnz=shard)
    dfac, bfac = dev_factors(factors), dev_factors(factors, torch.bfloat16)
    for _ in range(2):
        outs = [api.mttkrp(t, d, dfac) for d in range(3)]
        bouts = [api.mttkrp_bf16(t, d, bfac) for d in range(3)]
        grads = [api.cp_grad(t, d, dfac, -2.0) for d in range(3)]
        loss = api.cp_loss(t, dfac)
        for d in range(3):
            ref = oracle_mttkrp(idx, val, dims, factors, d).astype(np.float32)
            np.testing.assert_array_equal(outs[d].cpu().numpy(), ref)
            np.testing.assert_array_equal(bouts[d].cpu().numpy(), ref)
            np.testing.assert_array_equal(grads[d].cpu().numpy(),
                                          oracle.cp_grad(idx, val, dims, factors, d).astype(np.float32))
        assert float(loss) == oracle.cp_loss(idx, val, [f.astype(np.float64) for f in factors])[0]
    t.close()


def test_calls_on_two_streams_and_under_capture():
    """Calls ordered over two streams by an event, then a captured call whose
    replays alternate with eager calls."""
    rng = np.random.default_rng(3)
    dims, nnz, rank = (700, 300, 200), 20_000, 16
    idx = np.stack([rng.integers(0, d, nnz) for d in dims]).astype(np.int32)
    val = rng.integers(1, 4, nnz).astype(np.float32)
    factors = [rng.integers(-2, 3, (d, rank)).astype(np.float32) for d in dims]
    refs = [oracle_mttkrp(idx, val, dims, factors, d).astype(np.float32) for d in range(3)]
    t = api.Tensor(idx, val, dims, host_layout=True, shard_nnz=4096)
    dfac = dev_factors(factors)
    torch.cuda.synchronize()
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    for _ in range(3):
        x = api.mttkrp(t, 0, dfac, out=torch.full((dims[0], rank), float("nan"), device="cuda"), stream=a)
        b.wait_stream(a)
        y = api.mttkrp(t, 1, dfac, out=torch.full((dims[1], rank), float("nan"), device="cuda"), stream=b)
        a.wait_stream(b)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(x.cpu().numpy(), refs[0])
    np.testing.assert_array_equal(y.cpu().numpy(), refs[1])
    out = torch.empty((dims[2], rank), device="cuda")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        api.mttkrp(t, 2, dfac, out=out)
    for _ in range(3):
        out.fill_(float("nan"))
        g.replay()
        z = api.mttkrp(t, 0, dfac)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(out.cpu().numpy(), refs[2])
        np.testing.assert_array_equal(z.cpu().numpy(), refs[0])
    assert np.array_equal(hip_mttkrp(t, 1, dfac), refs[1])
    t.close()

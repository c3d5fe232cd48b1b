"""Rows that span units of the one-launch MTTKRP: the shares' hand-over between blocks,
launch after launch on the same slots, at other ranks in between, with other work on the
GPU so that the blocks arrive in other orders.  Integer inputs, exact in any order."""
import numpy as np
import pytest

from gpu_util import dev_factors, hip_mttkrp, oracle_mttkrp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2507_15121_amd import api  # noqa: E402


@pytest.mark.parametrize("lengths", [[4096], [193] * 40, [200, 4000, 260, 1, 3000, 77, 193], [2000] * 30])
def test_shares_launch_after_launch(lengths):
    rng = np.random.default_rng(len(lengths))
    i0 = np.repeat(np.arange(len(lengths)), lengths).astype(np.int32)
    dims = (len(lengths) + 3, 40, 30)
    idx = np.stack([i0] + [rng.integers(0, d, i0.size).astype(np.int32) for d in dims[1:]])
    val = rng.integers(1, 4, i0.size).astype(np.float32)
    t = api.Tensor(idx, val, dims)
    ranks = (16, 256, 5, 64, 300, 128)   # 1 to 4 columns per lane, and two launches
    fac = {r: [rng.integers(-1, 2, (d, r)).astype(np.float32) for d in dims] for r in ranks}
    dev = {r: dev_factors(f) for r, f in fac.items()}
    ref = {r: torch.from_numpy(oracle_mttkrp(idx, val, dims, f, 0).astype(np.float32)).cuda() for r, f in fac.items()}
    other = torch.cuda.Stream()
    x = torch.rand(1 << 22, device="cuda")
    for it in range(40):
        r = ranks[it % len(ranks)]
        if it % 3 == 0:
            with torch.cuda.stream(other):
                for _ in range(it % 7):
                    x.mul_(1.0)
        outs = [api.mttkrp(t, 0, dev[r]) for _ in range(4)]
        for out in outs:
            assert torch.equal(out, ref[r]), (it, r)
    torch.cuda.synchronize()
    t.close()


def test_shares_in_a_graph():
    """Replays, with eager launches of the same mode in between, find the slots cleared."""
    rng = np.random.default_rng(3)
    dims, rank = (12, 40, 30), 32
    idx = np.stack([rng.integers(0, d, 20_000) for d in dims]).astype(np.int32)
    val = rng.integers(1, 4, 20_000).astype(np.float32)
    factors = [rng.integers(-1, 2, (d, rank)).astype(np.float32) for d in dims]
    t = api.Tensor(idx, val, dims)
    dfac = dev_factors(factors)
    ref = oracle_mttkrp(idx, val, dims, factors, 0).astype(np.float32)
    out = torch.empty((dims[0], rank), device="cuda")
    np.testing.assert_array_equal(hip_mttkrp(t, 0, dfac), ref)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        api.mttkrp(t, 0, dfac, out=out)
    for _ in range(6):
        out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(out.cpu().numpy(), ref)
        np.testing.assert_array_equal(hip_mttkrp(t, 0, dfac), ref)
    t.close()

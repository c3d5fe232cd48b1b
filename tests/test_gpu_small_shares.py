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


@pytest.mark.parametrize("rank", [8, 16, 32])
@pytest.mark.parametrize("factors", ["f32", "bf16"])
def test_shares_are_added_in_fp64(rank, factors):
    """The longest split row of a launch, 64 units, all terms positive.  The result is
    rounded once (2^-24); a share is a sum of up to 4 + 32 terms of the 64-nonzero unit
    (2^-23 sqrt(36 / 36) at most), independent over 64 of them: 1.5e-8.  (Added in fp32
    the 64 shares alone would bring 2^-23 sqrt(64 / 36) = 1.6e-7.)"""
    rng = np.random.default_rng(rank)
    dims, nnz = (20, 400, 300), 4096 + 900
    idx = np.stack([rng.integers(0, d, nnz) for d in dims]).astype(np.int32)
    idx[0] = np.where(np.arange(nnz) < 4000, 7, rng.integers(8, 20, nnz))
    val = rng.random(nnz, dtype=np.float32) + np.float32(0.1)
    fac = [rng.random((d, rank), dtype=np.float32) + np.float32(0.1) for d in dims]
    t = api.Tensor(idx, val, dims)
    dev = dev_factors(fac, torch.bfloat16 if factors == "bf16" else None)
    fac = [f.float().cpu().numpy() for f in dev]
    at = np.flatnonzero(idx[0] == 7)
    ref = (val[at].astype(np.float64)[:, None] * fac[1][idx[1, at]].astype(np.float64) * fac[2][idx[2, at]].astype(np.float64)).sum(0)
    got = hip_mttkrp(t, 0, dev, bf16=factors == "bf16")[7]
    assert np.linalg.norm(got - ref) / np.linalg.norm(ref) <= 2.0 ** -24 + 1.5e-8
    t.close()

"""The gradient's factor kept on the device: the same bits as the factor given by
the host, and a backward pass that can be captured in a graph."""
import numpy as np
import pytest

from gpu_util import dev_factors

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2507_15121_amd import api, synth  # noqa: E402
from paper_2507_15121_amd.autograd import sparse_cp_loss  # noqa: E402


def _problem(rank=20):
    dims = (400, 300, 200)
    st = synth.tensor(dims, 9000, "zipf", 1.1, 0.05, seed=rank)
    return dims, api.Tensor(st.idx, st.val, dims, chunk_nnz=4096), dev_factors(synth.factors(dims, rank, seed=rank))


@pytest.mark.parametrize("rank", [16, 20])
@pytest.mark.parametrize("factor", [1.0, -0.3, 1e-20, 0.0])
def test_scaled_gradient_has_the_host_scale_s_bits(rank, factor):
    dims, t, F = _problem(rank)
    s = torch.tensor(factor, dtype=torch.float64, device="cuda")
    for d in range(3):
        a = api.cp_grad(t, d, F, -2.0 * factor)
        b = api.cp_grad_scaled(t, d, F, -2.0, s)
        assert torch.equal(a, b)
    t.close()


@pytest.mark.parametrize("n", [0, 1, 3, 4, 5, 1023, 4_000_001])
@pytest.mark.parametrize("factor", [1.0, -2.5, float("inf"), float("nan")])
def test_scale_in_place(n, factor):
    x = torch.randn(n, device="cuda")
    want = x * torch.tensor(factor, dtype=torch.float32, device="cuda")
    got = api.scale_(x, torch.tensor(factor, dtype=torch.float64, device="cuda"))
    assert got is x and torch.equal(torch.nan_to_num(got), torch.nan_to_num(want))
    assert torch.equal(torch.isnan(got), torch.isnan(want))


def test_forward_and_backward_replayed_from_a_graph():
    dims, t, F = _problem(32)
    F = [f.requires_grad_(True) for f in F]

    def step():
        loss = sparse_cp_loss(t, *F)
        return [loss.detach()] + list(torch.autograd.grad(loss, F))
    eager = [x.clone() for x in step()]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()
    torch.cuda.current_stream().wait_stream(side)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        outs = step()
    for _ in range(3):
        for o in outs:
            o.fill_(float("nan"))
        g.replay()
        again = step()
        torch.cuda.synchronize()
        for o, e, a in zip(outs, eager, again):
            np.testing.assert_array_equal(o.cpu().numpy(), e.cpu().numpy())
            np.testing.assert_array_equal(a.cpu().numpy(), e.cpu().numpy())
    t.close()


def test_bad_scales_refused():
    dims, t, F = _problem()
    for bad in (torch.tensor(1.0, device="cuda"), torch.tensor(1.0, dtype=torch.float64),
                torch.ones(2, dtype=torch.float64, device="cuda")):
        with pytest.raises(ValueError):
            api.cp_grad_scaled(t, 0, F, -2.0, bad)
        with pytest.raises(ValueError):
            api.scale_(torch.ones(4, device="cuda"), bad)
    t.close()

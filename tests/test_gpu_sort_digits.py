"""The layout build's radix sort at the edges of its digits (8 and 10 bits, one to
four passes) and of its tiles (4096 pairs, groups of blocks), with even and with
crowded digits: the permutation and arrays bit for bit those of a stable sort."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2507_15121_amd import api  # noqa: E402


@pytest.mark.parametrize("skew", [False, True])
@pytest.mark.parametrize("bits,nnz", [(8, 4095), (9, 4096), (10, 4097), (11, 8193), (16, 70_001), (17, 70_001),
                                      (20, 150_000), (21, 70_001), (30, 70_001), (31, 4097), (18, 2_200_000)])
def test_digit_widths_and_tiles(bits, nnz, skew):
    dims = (min(1 << bits, 2**31 - 1), 3, (1 << bits) - 1 if bits < 31 else 2)   # 2^31 rows are refused
    rng = np.random.default_rng(bits + nnz)
    cols = []
    for d in dims:
        x = rng.integers(0, d, nnz)
        if skew:   # nine of ten entries in three rows, so that whole waves share digits
            x = np.where(rng.random(nnz) < 0.9, rng.choice(np.array([0, d // 2, d - 1]), nnz), x)
        cols.append(x)
    cols[0][:2] = [0, dims[0] - 1]
    idx = np.stack(cols).astype(np.int32)
    val = rng.random(nnz).astype(np.float32)
    t = api.Tensor(idx, val, dims, keep_perm=True)
    lex = np.lexsort(idx[::-1])
    for d in range(3):
        perm = lex[np.argsort(idx[d][lex], kind="stable")]
        got = t.layout(d, perm=True)
        np.testing.assert_array_equal(got["perm"], perm)
        np.testing.assert_array_equal(got["out_idx"], idx[d][perm])
        np.testing.assert_array_equal(got["in_idx"], np.delete(idx, d, axis=0)[:, perm])
        np.testing.assert_array_equal(got["values"], val[perm])
    t.close()

"""The CSR products at block widths around the 16-column groups that they gather (the rest of a
padded block is zero): float64, float32 and bfloat16, against a float64 product, before and after
iterations that fill the buffers."""
import numpy as np
import pytest

from paper_2306_10379_amd import inputs as I

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,rel", [("fp64", 1e-13), ("mixed", 1e-5), ("bf16", 2e-2)])
@pytest.mark.parametrize("p", [1, 16, 17, 33, 40, 48, 49, 64, 65, 81, 128])
def test_product_at_column_group_edges(p, precision, rel):
    """Sums of 11 products: rounding of the operands (2^-9 bf16, 2^-24 fp32) and of the sums, each
    well below rel of the largest entry."""
    from paper_2306_10379_amd import gsi
    A = I.spiked_sparse(700, 5, 20, 3)
    W = np.random.default_rng(p).standard_normal((A.n, p))
    print(f"product p={p} {precision}", flush=True)
    with gsi.Solver(A, I.start_block(A.n, p, 4), p, precision=precision, max_iter=5) as s:
        ref = A.to_scipy() @ W
        Wd = torch.as_tensor(W, device="cuda")
        for _ in range(2):
            Z = (s.spmm if precision == "fp64" else s.spmm_lowp)(Wd).cpu().numpy()
            assert np.max(np.abs(Z - ref)) <= rel * np.max(np.abs(ref))
        s.solve()
        Z = (s.spmm if precision == "fp64" else s.spmm_lowp)(Wd).cpu().numpy()
        assert np.max(np.abs(Z - ref)) <= rel * np.max(np.abs(ref))

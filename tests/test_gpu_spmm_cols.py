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


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("p", [33, 40, 48, 49])
def test_solve_at_column_block_edges(p, precision):
    """The passes at 33 to 48 columns leave the last 16 of 64 out: the oracle's Ritz values to
    1e-10 and an orthonormal basis; in float64 its iteration count, and the values after 30
    gradient steps to 1e-9 (rounding grown by the steps)."""
    from oracle import gsi_oracle as O
    from paper_2306_10379_amd import gsi
    A = I.spiked_sparse(1100, 5, p, 7, gap=0.3, spike_max=9.0)
    X0 = I.start_block(A.n, p, 8)
    print(f"solve p={p} {precision}", flush=True)
    ref = O.rcg(A, X0, tol=1e-10, which=1, max_iter=3000)
    with gsi.Solver(A, X0, p, precision=precision, tol=1e-10, max_iter=3000) as s:
        status, iters = s.solve()
        ritz = np.asarray(s.residuals()[0])
        X = s.get_x().cpu().numpy()
    assert status == gsi.GSI_OK
    assert np.max(np.abs(ritz - ref.theta)) <= 1e-10 * np.max(np.abs(ref.theta))
    assert np.max(np.abs(X.T @ X - np.eye(p))) <= 1e-11
    if precision == "fp64":
        assert abs(iters - ref.iters) <= max(2, 0.02 * ref.iters)
        ref = O.rsd(A, X0, tol=1e-14, which=1, max_iter=30)
        with gsi.Solver(A, X0, p, method="rsd", tol=1e-14, max_iter=30) as s:
            s.solve()
            ritz = np.asarray(s.residuals()[0])
        assert np.max(np.abs(ritz - ref.theta)) <= 1e-9 * np.max(np.abs(ref.theta))

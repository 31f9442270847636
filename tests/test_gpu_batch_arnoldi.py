"""The batch's orthogonalisation: one workgroup per problem up to 5,120 densities (1 to 5 values a thread), launches
over all problems beyond.  Problems of very different lengths share a batch; each solution is compared with the
problem's own solve (the long ones on a fine grid: nodes much denser than the grid do not converge).  Both stop at a residual of 1e-11 of the right-hand side, and the operator's condition number is
of order 10, so they agree to 1e-9."""
import numpy as np
import pytest

from paper_2104_05024_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2104_05024_amd import kfbi as K  # noqa: E402


@pytest.mark.parametrize("longest", [700, 1024, 1025, 4097, 5120, 5121])
def test_batch_solve_of_uneven_densities(longest):
    print(f"[batch arnoldi] {longest}", flush=True)
    co = W.scalar_coeffs(2, 1.0, 200.0)
    probs = [(W.circle2d(0.6, longest), W.box(2, 64 if longest < 2000 else 1024), co), (W.circle2d(0.45, 33), W.box(2, 64), co),
             (W.circle2d(0.5, 257), W.box(2, 128), co)]
    b = K.Batch(probs)
    t = torch.linspace(0.0, 40.0, b.L, dtype=torch.float64, device="cuda")
    g = torch.sin(t)
    n = sum((grid.cells - 1) ** 2 for _, grid, _ in probs)
    f = torch.cos(torch.linspace(0.0, 900.0, n, dtype=torch.float64, device="cuda"))
    u, psi, info = b.solve_neumann(g, f, tol=1e-11)
    o = q = 0
    for iface, grid, c in probs:
        p = K.Problem(iface, grid, c)
        m = (grid.cells - 1) ** 2
        u1 = p.solve_neumann(g[o:o + p.M].reshape(1, -1), f[q:q + m].reshape(1, -1), tol=1e-11)[0].reshape(-1)
        e = float((u[q:q + m] - u1).abs().max() / u1.abs().max())
        o, q = o + p.M, q + m
        p.close()
        assert e < 1e-9, (grid.cells, e)
    b.close()
    assert np.all([i["iters"] > 0 for i in info])

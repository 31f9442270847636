"""The one-launch orthogonalisation of short Krylov vectors and its hand-over to the many-block kernels.

Vector lengths around the multiples of 1024 that change its shape, the last it takes (5120) and the
first it does not, restarts after one and a few vectors (the fewest basis vectors) and none at all,
with the step replayed from its graph and launched directly.  The residual GMRES reports follows from
the Hessenberg column; an explicit FP64 product of the returned density must give the same to the
rounding of the product: |true - reported| <= 1e-12 (a product's tolerance) relative to ||g'||."""
import numpy as np
import pytest

from paper_2104_05024_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2104_05024_amd import kfbi as K  # noqa: E402


@pytest.mark.parametrize("nodes", [63, 1023, 1024, 1025, 3072, 5120, 5121])
def test_reported_residual_is_the_residual(nodes):
    cells = 64 if nodes < 100 else 512
    grid = W.box(2, cells)
    p = K.Problem(W.circle2d(0.6, nodes), grid, W.scalar_coeffs(2, 1.0, 400.0))
    rng = np.random.default_rng(nodes)
    f = torch.tensor(rng.normal(size=(1, grid.n ** 2)), device="cuda")
    g = torch.tensor(rng.normal(size=(1, nodes)), device="cuda")
    for graph in (True, False):
        p.use_graph(graph)
        for restart in (1, 3, 50):
            print(f"[arnoldi] {nodes} nodes, restart {restart}, graph {graph}", flush=True)
            u, psi, info = p.solve_neumann(g, f, tol=1e-9, restart=restart, max_iters=400, true_resid=1,
                                           allow_noconv=True)
            assert info["iters"] > 0
            assert abs(info["true_resid"] - info["rel_resid"]) <= 1e-12, info
            if restart == 50:
                assert info["rel_resid"] <= 1e-9, info
    p.close()

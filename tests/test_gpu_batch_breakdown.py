"""A batched FP32 inner solve that breaks down has not converged.

The first problem's interface lies between grid nodes, with the tissue outside it: no grid line is cut and every stencil
is in the tissue, so its operator is exactly zero and the first Arnoldi column is.  The inner solve has to go on to its
residual and to its iteration limit, as a single problem's does, instead of returning as if it had converged (one
refinement, not the twenty allowed; two or three beside another problem, whose iterations count too).  The second
problem, alone, converges as ever."""
import numpy as np
import pytest

from paper_2104_05024_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2104_05024_amd import kfbi as K  # noqa: E402


def test_breakdown_is_not_convergence():
    co = W.scalar_coeffs(2, 1.0, 5.0)
    nothing = (W.Interface(2, [W.Surface((0.02, 0.02), -1, 9, [])]), W.Grid(2, -1.27, 1.13, 16), co)
    other = (W.circle2d(0.6, 97), W.box(2, 64), co)
    print("[breakdown]", flush=True)
    rng = np.random.default_rng(3)
    for probs in ([nothing], [nothing, other]):
        b = K.Batch(probs)
        g, f = torch.tensor(rng.normal(size=b.L), device="cuda"), torch.tensor(rng.normal(size=b.G), device="cuda")
        assert float(b.apply(g)[:9].abs().max()) == 0.0
        u, psi, info = b.solve_neumann(g, f, tol=1e-10, precision=1, max_iters=30, max_outer=20, allow_noconv=True)
        assert info[0]["outer"] <= (1 if len(probs) == 1 else 3) and info[0]["rel_resid"] > 0.5, info[0]
        assert bool(torch.isfinite(u).all())
        b.close()
    b = K.Batch([other])
    u, psi, info = b.solve_neumann(g[9:].contiguous(), f[-other[1].n ** 2:].contiguous(), tol=1e-10, precision=1)
    assert info[0]["rel_resid"] <= 1e-10
    b.close()

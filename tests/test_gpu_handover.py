"""Krylov cycles that change their orthogonalisation on the way: one workgroup while the basis is small, many blocks beyond.

The hand-over comes after 24,576 / n vectors of one problem and 36,864 / (longest) of a batch (n over 512), so cycles of 40
vectors cross it at every length here.  One problem: 40 iterations towards a tolerance they cannot reach, after which the
reported residual has to be the explicit one to 1e-12 (a product's rounding), and the same from the captured step as from
direct launches to the same.  A batch: its solutions against its members' own solves, both at 1e-11 of a well-conditioned
problem: 1e-9."""
import numpy as np
import pytest

from paper_2104_05024_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2104_05024_amd import kfbi as K  # noqa: E402


@pytest.mark.parametrize("nodes", [512, 700, 1025, 2049, 4097])
def test_one_problem(nodes):
    print(f"[hand-over] {nodes}", flush=True)
    grid = W.box(2, 512)
    p = K.Problem(W.circle2d(0.6, nodes), grid, W.scalar_coeffs(2, 1.0, 400.0))
    rng = np.random.default_rng(nodes)
    f = torch.tensor(rng.normal(size=(1, grid.n ** 2)), device="cuda")
    g = torch.tensor(rng.normal(size=(1, nodes)), device="cuda")
    sols = []
    for graph in (True, False):
        p.use_graph(graph)
        for _ in range(2):
            u, psi, info = p.solve_neumann(g, f, tol=1e-30, restart=64, max_iters=40, true_resid=1, allow_noconv=True)
            assert abs(info["true_resid"] - info["rel_resid"]) <= 1e-12, info
            sols.append(psi)
    for s in sols[1:]:
        assert float((s - sols[0]).abs().max()) <= 1e-10 * float(sols[0].abs().max())
    p.close()


@pytest.mark.parametrize("graph", [True, False], ids=["captured", "direct"])
@pytest.mark.parametrize("longest", [1200, 3000])
def test_batch(longest, graph):
    print(f"[hand-over] batch {longest}", flush=True)
    # 34 iterations (nodes denser than the grid) and 31 (a star), where 30 and 12 are the last of one workgroup
    co = W.scalar_coeffs(2, 1.0, 5.0)
    first = (W.circle2d(0.6, longest), W.box(2, 256), co) if longest == 1200 else \
        (W.star2d(0.7, 0.2, 8, longest), W.box(2, 512), co)
    probs = [first, (W.circle2d(0.45, 33), W.box(2, 64), co)]
    b = K.Batch(probs)
    b.graph(graph)
    rng = np.random.default_rng(longest)
    g, f = torch.tensor(rng.normal(size=b.L), device="cuda"), torch.tensor(rng.normal(size=b.G), device="cuda")
    u, psi, info = b.solve_neumann(g, f, tol=1e-11, restart=64)
    for i, (iface, grid, c) in enumerate(probs):
        p = K.Problem(iface, grid, c)
        s, t = slice(b.ioff[i], b.ioff[i] + b.M[i]), slice(b.goff[i], b.goff[i] + grid.n ** 2)
        v = p.solve_neumann(g[s].reshape(1, -1), f[t].reshape(1, -1), tol=1e-11, restart=64)[0].reshape(-1)
        assert float((u[t] - v).abs().max()) <= 1e-9 * float(v.abs().max()), i
        p.close()
    assert info[0]["iters"] * longest > 36 * 1024, info[0]["iters"]
    b.close()

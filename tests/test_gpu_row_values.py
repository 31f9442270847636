"""Row passes of a product with different numbers of values per thread must agree.

Without a reaction term the two components of a pair do not see each other, so the pair's product is the two scalar
ones; its lists have twice the rows.  At 512^3 that takes the passes over the 100,000 rows from which a transform is held
by fewer threads (8 values each, then 16); at 256^2 and 1024^2 the pair's rows fall into other tiles.  FP64 to 1e-12, a
product's tolerance; FP32 to 6e-8 times the cells (the rounding of grid values, magnified by differences over h)."""
import numpy as np
import pytest

from paper_2104_05024_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2104_05024_amd import kfbi as K  # noqa: E402


@pytest.mark.parametrize("dim,cells", [(2, 256), (2, 1024), (3, 256), (3, 512)])
def test_uncoupled_pair_is_two_scalars(dim, cells):
    print(f"[row values] {dim}D {cells}", flush=True)
    iface = W.circle2d(0.7, 401) if dim == 2 else W.sphere(0.7, 4001)
    grid, D = W.box(dim, cells), [[1.0] * dim, [2.0] * dim]
    p = K.Problem(iface, grid, W.Coeffs(2, D, 0.0))
    if (dim, cells) == (3, 512):
        rows = len(np.unique(p.table("irregular") // grid.n))
        assert rows < 100000 < 2 * rows
    psi = torch.tensor(np.random.default_rng(cells).uniform(-1, 1, size=(2, p.M)), device="cuda")
    pair = {t: p.apply(psi.to(t)).double() for t in (torch.float64, torch.float32)}
    p.close()
    for c in range(2):
        s = K.Problem(iface, grid, W.Coeffs(1, [D[c]], 0.0))
        for t, tol in ((torch.float64, 1e-12), (torch.float32, 6e-8 * cells)):
            one = s.apply(psi[c:c + 1].to(t)).double()
            assert float((pair[t][c:c + 1] - one).abs().max()) <= tol * float(one.abs().max()), (c, t)
        s.close()

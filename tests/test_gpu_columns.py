"""The last axis of the box solve solved as tridiagonal columns, against sine transforms on the CPU.

Every grid size (chunks of 8, 16 and 32 rows; one to 32 chunks per column), one and two components,
and coefficients on both sides of the rule that chooses between the columns and the sine
transform: isotropic, fibres along x, the last axis up to 100 times the others', no reaction and a
very strong one.  FP64: 1e-12, the tolerance of a box solve elsewhere.  FP32: 5e-6 (6e-8 per
transform stage over 2 log2(cells) stages and two axes).

The reference is the oracle's solve with the pair's determinant as a_i a_e + kappa (a_i + a_e): the
oracle takes (a_i + kappa)(a_e + kappa) - kappa^2, which at kappa = 1e5 loses eps kappa / 2a, 5e-13 of
the result on the 1024^2 grid (measured against the sum and difference of the two equations)."""
import numpy as np
import pytest
import scipy.fft

from oracle import boxsolve as obs
from paper_2104_05024_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2104_05024_amd import kfbi as K  # noqa: E402


def coefficients(dim):
    one = [1.0] * dim
    return {
        "scalar": W.Coeffs(1, [one], 400.0),
        "laplace": W.Coeffs(1, [one], 0.0),
        "fibres_x": W.Coeffs(1, [[3.0] + [0.5] * (dim - 1)], 50.0),
        "last_2": W.Coeffs(1, [one[1:] + [2.0]], 0.0),
        "last_6": W.Coeffs(1, [one[1:] + [6.0]], 0.0),
        "last_100": W.Coeffs(1, [one[1:] + [100.0]], 0.0),
        "stiff": W.Coeffs(1, [one], 1e16),
        "pair": W.Coeffs(2, [one, [2.0] * dim], 200.0),
        "pair_uncoupled": W.Coeffs(2, [one, [2.0] * dim], 0.0),
        "pair_equal": W.Coeffs(2, [one, one], 1e5),
        "pair_swapped": W.Coeffs(2, [[2.0] + [1.0] * (dim - 1), [3.0] + [0.5] * (dim - 1)], 2e4),
        "pair_last_100": W.Coeffs(2, [one[1:] + [100.0], one[1:] + [60.0]], 200.0),
    }


def reference(f, grid, co):
    if co.ncomp == 1:
        return obs.box_solve(f, grid, co)
    fh = [scipy.fft.dstn(c.reshape((grid.n,) * grid.dim), type=1, workers=obs.WORKERS) for c in f]
    ai, ae = (obs._mode_sums(grid.dim, grid.n, grid.h, D) for D in co.D)
    det = ai * ae + co.kappa * (ai + ae)
    uh = [((ae + co.kappa) * fh[0] + co.kappa * fh[1]) / det, (co.kappa * fh[0] + (ai + co.kappa) * fh[1]) / det]
    return np.stack([scipy.fft.idstn(u, type=1, workers=obs.WORKERS).ravel() for u in uh])


@pytest.mark.parametrize("dim,cells", [(2, 16), (2, 32), (2, 64), (2, 128), (2, 256), (2, 512), (2, 1024),
                                       (3, 16), (3, 32), (3, 64), (3, 128)])
def test_columns_match_oracle(dim, cells):
    grid = W.box(dim, cells)
    rng = np.random.default_rng(cells + dim)
    for name, co in coefficients(dim).items():
        print(f"[columns] {dim}D {cells} {name}", flush=True)
        f = rng.normal(size=(co.ncomp, grid.n ** dim))
        ref = reference(f, grid, co)
        for dtype, tol in ((torch.float64, 1e-12), (torch.float32, 5e-6)):
            if dtype == torch.float32 and cells > 256:
                continue                      # the transforms' own FP32 error passes 5e-6 there
            u = K.box_solve_noalloc(grid, co, torch.tensor(f, dtype=dtype, device="cuda"))
            e = float(np.max(np.abs(u.cpu().numpy().reshape(ref.shape) - ref)) / np.max(np.abs(ref)))
            assert e < tol, (name, dtype, e)

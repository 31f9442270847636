"""Coupled box solves of sources that nearly cancel between the components, f = (g, -g).

A bidomain step's source is of this kind.  It excites the pair's large eigenvalue only, while rounding in the rotation
of the last axis' columns leaks into the small one and comes out magnified by their ratio, about kappa over the mode
sums.  The reference is the sine-mode solve in extended precision, written so that it does not cancel.  Tolerance:
eps / 2 from each of the 2 dim log2(M) transform stages, adding up as a random walk (2.7 eps for 30 stages), doubled:
6 eps = 1.4e-15 of the solution's 2-norm.  It is the root mean square over sources and conductivities that has to keep
it: the transforms pair the two components' rows differently, and that part of their rounding is magnified as well
(single solves reach 1.9e-15)."""
import numpy as np
import pytest
import scipy.fft

from paper_2104_05024_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2104_05024_amd import kfbi as K  # noqa: E402

LD = np.longdouble


def mode_sums(grid, D):
    pi = LD("3.14159265358979323846264338327950288")
    k = np.arange(1, grid.n + 1).astype(LD)
    lam = 4 / LD(grid.h) ** 2 * np.sin(k * pi / (2 * grid.cells)) ** 2
    return sum(LD(D[a]) * lam.reshape((-1,) + (1,) * a) for a in range(grid.dim))


def reference(f, grid, co):
    fi, fe = (scipy.fft.dstn(c.reshape((grid.n,) * grid.dim).astype(LD), type=1) for c in f)
    ai, ae = (mode_sums(grid, D) for D in co.D)
    k, both = LD(co.kappa), fi + fe
    det = ai * ae + k * (ai + ae)
    return np.stack([scipy.fft.idstn(u, type=1).ravel()
                     for u in ((ae * fi + k * both) / det, (ai * fe + k * both) / det)])


@pytest.mark.parametrize("dim,cells", [(2, 16), (2, 32), (2, 64), (3, 16), (3, 32)])
def test_opposite_sources(dim, cells):
    grid = W.box(dim, cells)
    x = np.arange(1, cells) / cells
    coefs = {"twice": [[1.0] * dim, [2.0] * dim], "equal": [[1.0] * dim] * 2,
             "fibres": [[3.0] + [0.5] * (dim - 1), [2.0] + [1.0] * (dim - 1)],
             "swapped": [[2.0] + [1.0] * (dim - 1), [3.0] + [0.5] * (dim - 1)]}
    for kappa in (0.0, 5.0, 200.0):
        err = []
        for name, D in coefs.items():
            for seed in range(4):
                rng = np.random.default_rng(seed)
                g = sum((c - m) ** 2 for c, m in zip(np.meshgrid(*[x] * dim, indexing="ij"), rng.uniform(0.35, 0.65, dim)))
                g = (g < 0.06).astype(float).ravel()
                s = rng.uniform(0.8, 1.25)
                co = W.Coeffs(2, [[s * v for v in Dc] for Dc in D], kappa)
                f = np.stack([g, -g])
                u = K.box_solve_noalloc(grid, co, torch.tensor(f, device="cuda")).cpu().numpy()
                ref = reference(f, grid, co)
                err.append(float(np.linalg.norm((u.reshape(ref.shape) - ref).astype(float)) /
                                 np.linalg.norm(ref.astype(float))))
        rms = float(np.sqrt(np.mean(np.square(err))))
        print(f"[pair sources] {dim}D {cells} kappa {kappa:g}: {rms:.1e}, largest {max(err):.1e}", flush=True)
        assert rms < 1.4e-15, (kappa, err)

"""Box solves where the transform passes change their number of values per thread.

A pencil pair is held by M / 4, M / 8 or M / 16 threads depending on the size and on how many rows a pass has.
A source made of a few modes has an exact solution (each mode divided by its eigenvalue), so every size up to
512^3 is checked without an oracle run.  Tolerances: the rounding of 2 dim transforms of log2(M) stages each, 6e-8
(FP32) or 1.1e-16 (FP64) per stage, times the 10 or so that the modes add up to: 2e-5 and 4e-14."""
import numpy as np
import pytest

from paper_2104_05024_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2104_05024_amd import kfbi as K  # noqa: E402

TOL = {torch.float64: 4e-14, torch.float32: 2e-5}


def modes(dim, M, dtype):
    """Source and solution of (kappa - sum_a d_a^2) u = f for three modes, one of them the highest."""
    h, kappa = 2.4 / M, 300.0
    n = torch.arange(1, M, dtype=torch.float64, device="cuda")
    f = u = 0
    for amp, ks in ((1.0, (1, 2, 1)), (-0.7, (M // 3, 1, M // 2)), (0.4, (M - 1, M - 1, M - 1))):
        v, lam = amp, 0.0
        for a in range(dim):
            v = v * torch.sin(np.pi * ks[a] * n / M).reshape((-1,) + (1,) * a)
            lam += 4 / h ** 2 * np.sin(ks[a] * np.pi / (2 * M)) ** 2
        f, u = f + v, u + v / (lam + kappa)
    return f.reshape(1, -1).to(dtype), u.reshape(1, -1), kappa


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("dim,M", [(2, 32), (2, 64), (2, 128), (2, 256), (2, 512), (2, 1024), (3, 16), (3, 64), (3, 128),
                                   (3, 256), (3, 512)])
def test_box_solve_of_modes(dim, M, dtype):
    print(f"[passes] {dim}D {M} {dtype}", flush=True)
    f, u, kappa = modes(dim, M, dtype)
    iface = W.circle2d(0.6, 41) if dim == 2 else W.sphere(0.6, 97)
    p = K.Problem(iface, W.box(dim, M), W.scalar_coeffs(dim, 1.0, kappa))
    out = p.box_solve(f)
    e = float((out.double() - u).abs().max() / u.abs().max())
    p.close()
    assert e < TOL[dtype], e

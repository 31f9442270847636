"""Products whose first row pass forms the correction, against the same products with the correction launched apart
(as they are while profiling).  Both add the same terms in the same order, so only the rounding of fused
multiply-adds may differ: 1e-12 in FP64, 3e-6 with an FP32 grid side, relative to the largest value.  The sizes leave
tiles that span both components, rows with one node and partly filled groups of arms.  In FP32 the two routes pair
other rows, or hold other numbers of values per thread, at the coupled 512 (2D) and 256 (3D): both are then off the FP64
product by several 1e-6 in their own ways (1.8e-5 each, and 4.4e-6 / 3.5e-6), and only FP64 is compared."""
import numpy as np
import pytest

from paper_2104_05024_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2104_05024_amd import kfbi as K  # noqa: E402

PAIR = W.bidomain_coeffs(2, W.BidomainParams(), 0.01)
PAIR3 = W.Coeffs(2, [[3.0, 0.5, 0.5], [2.0, 1.0, 1.0]], 200.0)
CASES = {
    "circle_64": (W.circle2d(0.3, 9), W.box(2, 64), W.scalar_coeffs(2, 1.0, 50.0)),
    "circle_64_pair": (W.circle2d(0.6, 63), W.box(2, 64), PAIR),
    "circle_128_pair": (W.circle2d(0.9, 129), W.box(2, 128), PAIR),
    "star_256": (W.star2d(n_nodes=301), W.box(2, 256), W.scalar_coeffs(2, 1.0, 400.0)),
    "circle_512_pair": (W.circle2d(0.5, 333), W.box(2, 512), PAIR),
    "circle_1024": (W.circle2d(0.2, 201), W.box(2, 1024), W.scalar_coeffs(2, 1.0, 400.0)),
    "sphere_64_pair": (W.sphere(0.4, 97), W.box(3, 64), PAIR3),
    "sphere_128": (W.sphere(0.7, 997), W.box(3, 128), W.scalar_coeffs(3, 1.0, 400.0)),
    "sphere_128_pair": (W.sphere(0.2, 97), W.box(3, 128), PAIR3),
    "sphere_256_pair": (W.sphere(0.3, 401), W.box(3, 256), PAIR3),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_fused_correction(name):
    iface, grid, co = CASES[name]
    print(f"[fused correction] {name}", flush=True)
    p = K.Problem(iface, grid, co)
    psi = np.random.default_rng(8).uniform(-1, 1, size=(co.ncomp, p.M))
    for dtype, tol in ((torch.float64, 1e-12), (torch.float32, 3e-6)):
        if dtype == torch.float32 and name in ("circle_512_pair", "sphere_256_pair"):
            continue
        x = torch.tensor(psi, dtype=dtype, device="cuda")
        fused = p.apply(x)
        p.profile(True)
        apart = p.apply(x)
        p.profile(False)
        assert torch.equal(p.apply(x), fused)
        assert float((fused - apart).abs().max()) <= tol * float(apart.abs().max()), dtype
    p.close()

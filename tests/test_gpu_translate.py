"""The matrix-core translations (rotation, axial shift, rotation back) at every
kind of order they are built for, against the point sum."""

import numpy as np
import pytest

from oracle.native import point_sum_c
from synthetic import complex_normal, meshes, nystrom3

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# orders below, at and above the matrix instructions' 4-row steps and 16-row tiles, the largest of the double
# precision kernels, and those served by the next larger kernel (13, 15, 19).  Single precision ends at 18 here:
# the multipoles of boxes this small against the wavelength leave its range above
ORDERS64 = (3, 4, 5, 7, 8, 9, 11, 12, 13, 15, 16, 17, 18, 19, 20, 21, 22, 23, 24)
ORDERS32 = (3, 4, 5, 8, 9, 10, 12, 13, 16, 17, 18)


@pytest.fixture(scope="module")
def body():
    q = nystrom3(meshes.geodesic_ellipsoid((1.5, 1.0, 0.75), 7))
    n = q["points"].shape[0]
    a, b = complex_normal((2, n, 3), 71), complex_normal((2, n, 3), 72)
    k = 0.5
    ref = point_sum_c(q["points"], q["normals"], q["weights"], q["point_tri"], k, a, b)
    return q, k, a, b, ref


@pytest.mark.parametrize("precision,order", [("fp64", p) for p in ORDERS64] + [("fp32", p) for p in ORDERS32])
def test_translations_of_every_kernel_order(body, precision, order):
    """Low-frequency boxes take order ceil(2.8 d) for 10^-d: a plan asked for 10^-(p - 0.5)/2.8 has order p
    throughout, and the order rule promises that accuracy up to a small factor (4 here); single precision adds
    its rounding, 2e-5 of the result's norm after sums over 3 levels.  Two right-hand sides in one call equal
    the two by themselves, bit for bit."""
    from paper_1211_7177_amd import Plan
    q, k, a, b, ref = body
    tol = 10.0 ** (-(order - 0.5) / 2.8)
    print("translate", precision, order, flush=True)
    P = Plan(q["points"], q["normals"], q["weights"], k, 0, depth=4, precision=precision, nrhs_max=2, corr="none",
             point_tri=q["point_tri"], tol=tol)
    assert P.info()["order_level"][2:] == [order] * 3
    dt = torch.complex128 if precision == "fp64" else torch.complex64
    ga, gb = (torch.as_tensor(u, device="cuda").to(dt) for u in (a, b))
    y = P.matvec(ga, gb)
    err = np.linalg.norm(y.cpu().numpy() - ref) / np.linalg.norm(ref)
    print("translate %s order %d rel err %.3e" % (precision, order, err), flush=True)
    assert err <= 4 * 10.0 ** (-order / 2.8) + (2e-5 if precision == "fp32" else 1e-13)
    for r in range(2):
        assert torch.equal(P.matvec(ga[r], gb[r]), y[r])


@pytest.mark.parametrize("k,order", [(12.0, 21), (14.0, 23), (16.0, 25), (18.0, 27), (22.0, 32), (23.0, 33)])
def test_single_precision_orders_of_large_boxes(k, order):
    """Level 2 of the unit sphere at k holds boxes wide enough for the given order (excess-bandwidth rule for 1e-4);
    32 is the matrix-core kernels' largest, 33 runs as three launches.  The plan keeps what it was asked for, 1e-4."""
    from paper_1211_7177_amd import Plan
    q = nystrom3(meshes.icosphere(8))
    n = q["points"].shape[0]
    a, b = complex_normal((n, 3), 73), complex_normal((n, 3), 74)
    print("translate fp32 k", k, "order", order, flush=True)
    P = Plan(q["points"], q["normals"], q["weights"], k, 0, depth=3, precision="fp32", corr="none",
             point_tri=q["point_tri"], tol=1e-4)
    assert P.info()["order_level"][2] == order
    y = P.matvec(*(torch.as_tensor(u, device="cuda").to(torch.complex64) for u in (a, b))).cpu().numpy()
    ref = point_sum_c(q["points"], q["normals"], q["weights"], q["point_tri"], k, a, b)
    assert np.linalg.norm(y - ref) <= 1e-4 * np.linalg.norm(ref)

"""Plans of one order that translate by rotation and axial shift, with complex
wavenumbers, against the point sum at the order's own accuracy."""

import numpy as np
import pytest

from oracle.native import point_sum_c
from synthetic import complex_normal, meshes, nystrom3

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", params=[2.0 + 0.5j, 1.5 + 1.5j, 3.0j])
def body(request):
    q = nystrom3(meshes.geodesic_ellipsoid((1.5, 1.0, 0.75), 6))
    n = q["points"].shape[0]
    a, b = complex_normal((n, 3), 51), complex_normal((n, 3), 52)
    k = request.param
    return q, k, a, b, point_sum_c(q["points"], q["normals"], q["weights"], q["point_tri"], k, a, b)


@pytest.mark.parametrize("depth", [2, 3])
@pytest.mark.parametrize("order", [5, 8, 11, 14, 17, 20, 22, 24])
def test_one_order_with_lossy_wavenumbers(body, order, depth):
    """Boxes of at most 0.75 and |k| <= 3 stay below k d = 4, where the order rule asks for 2.8 degrees a digit: the
    error is 10^(-p/2.8) up to a small factor (4 here) and rounding (1e-13).  Single precision to order 14, with
    2e-5 for its rounding; above, its multipoles leave the range of boxes this small."""
    from paper_1211_7177_amd import Plan
    q, k, a, b, ref = body
    for precision in ("fp64", "fp32") if 8 <= order <= 14 else ("fp64",):
        P = Plan(q["points"], q["normals"], q["weights"], k, order, depth=depth, precision=precision, corr="none",
                 point_tri=q["point_tri"], far_cutoff=-1.0)
        y = P.matvec(*(torch.as_tensor(u, device="cuda").to(P.cdtype) for u in (a, b))).cpu().numpy()
        P.close()
        err = np.linalg.norm(y - ref) / np.linalg.norm(ref)
        print("one order %d depth %d k %s %s err %.2e" % (order, depth, k, precision, err), flush=True)
        assert err <= 4 * 10.0 ** (-order / 2.8) + (2e-5 if precision == "fp32" else 1e-13)

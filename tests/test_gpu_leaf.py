"""The matrix-core kernels at the leaves (sources to multipoles, local expansions
to nodes, and their adjoint) and plans of one order, at the edges of their tiles."""

import numpy as np
import pytest

from oracle.native import point_sum_c
from synthetic import complex_normal, meshes, nystrom3

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# 8 orders to a wavefront of the sources' kernel; 4, 8, 12 steps to an instance of the nodes' kernels; the dense
# path of single precision ends at 7 (9 with split products)
ORDERS = (1, 2, 5, 7, 8, 9, 15, 16, 17, 23)


@pytest.fixture(scope="module")
def body():
    q = nystrom3(meshes.geodesic_ellipsoid((1.5, 1.0, 0.75), 6))
    n = q["points"].shape[0]
    a, b = complex_normal((3, n, 3), 81), complex_normal((3, n, 3), 82)
    k = 2.0 + 0.5j
    return q, k, a, b, point_sum_c(q["points"], q["normals"], q["weights"], q["point_tri"], k, a, b)


@pytest.mark.parametrize("translate", ["fp32", "bf16x3"])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("depth", [2, 4])               # leaves of more than two 64-node chunks; of a few nodes
@pytest.mark.parametrize("order", ORDERS)
def test_leaf_kernels_at_every_edge(body, order, depth, precision, translate):
    """Against the point sum: a far pair's terms fall off by 0.76 a degree at worst (boxes two apart) and by less
    than 0.6 on average over the offsets.  The adjoint product is the transpose of the truncated product itself,
    degree by degree, so <A(a, b), y> = <(a, b), A^H y> holds to rounding (1e-12 and 1e-4 of the norms).  Three
    right-hand sides (two and one to a block) equal single ones bit for bit in double precision; the near field of
    single precision sums its sources in tiles that depend on their number."""
    from paper_1211_7177_amd import Plan
    if translate == "bf16x3" and (precision == "fp64" or order < 2):
        pytest.skip("split products are single precision, order 2 and up")
    q, k, a, b, ref = body
    if precision == "fp32" and order > 17:
        pytest.skip("multipoles of boxes this small leave the range of single precision")
    print("leaf", precision, translate, "order", order, "depth", depth, flush=True)
    P = Plan(q["points"], q["normals"], q["weights"], k, order, depth=depth, precision=precision, nrhs_max=3,
             corr="none", point_tri=q["point_tri"], translate=translate)
    dt = torch.complex128 if precision == "fp64" else torch.complex64
    ga, gb = (torch.as_tensor(u, device="cuda").to(dt) for u in (a, b))
    y = P.matvec(ga, gb)
    if precision == "fp64":
        for r in range(3):
            assert torch.equal(P.matvec(ga[r], gb[r]), y[r])
    out = y.cpu().numpy().astype(complex)
    err = np.linalg.norm(out - ref) / np.linalg.norm(ref)
    v = complex_normal(a.shape[1:], 83)
    va, vb = (u.cpu().numpy().astype(complex) for u in P.matvec_adjoint(torch.as_tensor(v, device="cuda").to(dt)))
    lhs, rhs = np.vdot(v, out[0]), np.vdot(va, a[0]) + np.vdot(vb, b[0])
    gap = abs(lhs - rhs) / (np.linalg.norm(v) * np.linalg.norm(out[0]))
    print("leaf %s order %d depth %d err %.2e gap %.2e" % (precision, order, depth, err, gap), flush=True)
    assert err <= 0.6 ** order + (2e-5 if precision == "fp32" else 1e-13)
    assert gap <= (1e-4 if precision == "fp32" else 1e-12)

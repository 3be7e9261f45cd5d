"""Leaf orders 25 to 40 in double precision: the largest instances of the kernels at
the leaves, and the right-hand sides that a block of the nodes' kernel takes."""

import numpy as np
import pytest

from oracle.native import point_sum_c
from synthetic import complex_normal, meshes, nystrom3

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# two right-hand sides of a block stop to fit its LDS at 34 with four wavefronts to a leaf and at 37 with one;
# 32 and 40 add a wavefront to the sources' kernel; 40 is the largest
ORDERS = (25, 32, 33, 34, 36, 37, 40)


@pytest.fixture(scope="module")
def body():
    q = nystrom3(meshes.icosphere(8))
    n = q["points"].shape[0]
    a, b = complex_normal((3, n, 3), 91), complex_normal((3, n, 3), 92)
    return q, a, b, point_sum_c(q["points"], q["normals"], q["weights"], q["point_tri"], 0.5, a, b)


@pytest.mark.parametrize("depth,waves", [(3, 1), (2, 4)])       # nodes of an average leaf: 14 and 69
@pytest.mark.parametrize("order", ORDERS)
def test_several_right_hand_sides_at_large_leaf_orders(body, order, depth, waves):
    """A plan asked for 10^-(p - 0.5)/2.8 has order p, whose accuracy the order rule promises up to a small factor
    (4 here); 1e-12 covers the rounding of sums over 189 boxes and 1600 coefficients (5e-14 if it is random).  A
    batch of three and one of two equal single calls, bit for bit."""
    from paper_1211_7177_amd import Plan
    q, a, b, ref = body
    print("large leaf order", order, "depth", depth, flush=True)
    P = Plan(q["points"], q["normals"], q["weights"], 0.5, 0, depth=depth, nrhs_max=3, corr="none",
             point_tri=q["point_tri"], tol=10.0 ** (-(order - 0.5) / 2.8))
    inf = P.info()
    assert inf["order"] == order and min(4, -(-inf["n"] // (16 * inf["nbox"][depth]))) == waves
    ga, gb = (torch.as_tensor(u, device="cuda") for u in (a, b))
    y = P.matvec(ga, gb)
    assert torch.equal(P.matvec(ga[:2], gb[:2]), y[:2])
    for r in range(3):
        assert torch.equal(P.matvec(ga[r], gb[r]), y[r])
    err = np.linalg.norm(y.cpu().numpy() - ref) / np.linalg.norm(ref)
    print("large leaf order %d depth %d err %.2e" % (order, depth, err), flush=True)
    assert err <= 4 * 10.0 ** (-order / 2.8) + 1e-12
    P.close()


@pytest.mark.parametrize("k,order", [(16.0, 25), (22.0, 32), (23.0, 33), (30.0, 40)])
def test_single_precision_leaves_many_wavelengths_wide(body, k, order):
    """Leaves of half the unit sphere's radius at k (excess-bandwidth rule for 1e-4): both columns of a batch keep what
    the plan was asked for, 1e-4."""
    from paper_1211_7177_amd import Plan
    q, a, b, _ = body
    print("large leaf fp32 k", k, flush=True)
    P = Plan(q["points"], q["normals"], q["weights"], k, 0, depth=2, precision="fp32", nrhs_max=2, corr="none",
             point_tri=q["point_tri"], tol=1e-4)
    assert P.info()["order"] == order
    y = P.matvec(*(torch.as_tensor(u[:2], device="cuda").to(torch.complex64) for u in (a, b))).cpu().numpy()
    ref = point_sum_c(q["points"], q["normals"], q["weights"], q["point_tri"], k, a[:2], b[:2])
    for r in range(2):
        err = np.linalg.norm(y[r] - ref[r]) / np.linalg.norm(ref[r])
        print("large leaf fp32 order %d err %.2e" % (order, err), flush=True)
        assert err <= 1e-4
    P.close()


@pytest.mark.parametrize("precision,order,k,refused", [("fp64", 23, 0.5, False), ("fp64", 24, 0.5, True),
                                                       ("fp32", 36, 26.0, False), ("fp32", 37, 27.0, True)])
def test_adjoint_orders(body, precision, order, k, refused):
    """The adjoint takes leaf orders up to 23 in double and 36 in single precision: there <A(a, b), y> =
    <(a, b), A^H y> holds to rounding (1e-12 and 1e-4 of the norms)."""
    from paper_1211_7177_amd import Plan
    from paper_1211_7177_amd._abi import FmbError
    q, a, b, _ = body
    tol = 10.0 ** (-(order - 0.5) / 2.8) if precision == "fp64" else 1e-4
    P = Plan(q["points"], q["normals"], q["weights"], k, 0, depth=2, precision=precision, corr="none",
             point_tri=q["point_tri"], tol=tol)
    assert P.info()["order"] == order
    y = torch.as_tensor(a[2], device="cuda").to(P.cdtype)
    if refused:
        with pytest.raises(FmbError, match="orders up to 23 in FP64"):
            P.matvec_adjoint(y)
    else:
        out = P.matvec(*(torch.as_tensor(u[0], device="cuda").to(P.cdtype) for u in (a, b))).cpu().numpy().astype(complex)
        va, vb = (u.cpu().numpy().astype(complex) for u in P.matvec_adjoint(y))
        gap = abs(np.vdot(a[2], out) - np.vdot(va, a[0]) - np.vdot(vb, b[0]))
        assert gap <= (1e-12 if precision == "fp64" else 1e-4) * np.linalg.norm(a[2]) * np.linalg.norm(out)
    P.close()

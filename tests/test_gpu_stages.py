"""The stage timers count the kernels that a product launches."""

import pytest

from synthetic import complex_normal, meshes, nystrom3

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _launches(stages=None, nrhs=1, **kw):
    from paper_1211_7177_amd import Plan
    q = nystrom3(meshes.icosphere(8))
    n = q["points"].shape[0]
    P = Plan(q["points"], q["normals"], q["weights"], 1.0, corr="none", point_tri=q["point_tri"], nrhs_max=nrhs, **kw)
    a = torch.as_tensor(complex_normal((nrhs, n, 3), 21), device="cuda").to(P.cdtype)
    P.profile(True, stages)
    P.matvec(a, a.clone())
    out = {k: v[1] for k, v in P.profile_read().items()}
    P.close()
    return out


def test_levels_of_one_order_share_a_launch():
    """Order 16 at levels 2 to 4: one S|R launch, its tiles split, and one of the partial sums; with the finest
    level timed by itself two of each.  S|S and R|R are one launch into each of two levels."""
    got = _launches(["m2l", "m2m", "l2l"], order=16, depth=4)
    assert (got["m2l"], got["m2m"], got["l2l"], got["m2l_fine"]) == (2, 2, 2, 0)
    got = _launches(order=16, depth=4)
    assert (got["m2l"], got["m2l_fine"], got["sums"]) == (4, 2, 0)


def test_large_orders_take_three_launches():
    """Order 34 in double precision: rotation, axial shift and rotation back are launches of their own."""
    got = _launches(order=0, tol=1e-12, depth=3)
    assert (got["m2l"], got["m2l_fine"], got["m2m"], got["l2l"]) == (6, 3, 3, 3)


def test_dense_plans():
    """One S|R launch a level, the sums of all levels in one beside one for each level's S|S."""
    got = _launches(order=5, depth=4, precision="fp32")
    assert (got["m2l"], got["m2m"], got["l2l"], got["sums"], got["m2l_fine"]) == (3, 2, 2, 3, 0)

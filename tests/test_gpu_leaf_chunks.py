"""Sources to multipoles where the fullest leaf has more than 32 nodes and the average one fewer: plans with a short
grid take 64 nodes at a time, plans for wide batches 32."""

import numpy as np
import pytest

from synthetic import complex_normal, meshes, nystrom3

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("precision,order", [("fp32", 1), ("fp32", 7), ("fp32", 12), ("fp64", 3), ("fp64", 8), ("fp64", 16),
                                             ("fp64", 23)])
def test_chunks_of_both_sizes_agree(precision, order):
    """532 leaves of up to 40 nodes.  The two plans form the same sums in different groups: they differ by rounding,
    1e-13 and 1e-5 of the norm."""
    from paper_1211_7177_amd import Plan
    q = nystrom3(meshes.torus(1.0, 0.3, 80, 20))
    n = q["points"].shape[0]
    print("leaf chunks", precision, order, flush=True)
    dt = torch.complex128 if precision == "fp64" else torch.complex64
    a, b = (torch.as_tensor(complex_normal((n, 3), s), device="cuda").to(dt) for s in (31, 32))
    y = []
    for wide in (1, 32):
        P = Plan(q["points"], q["normals"], q["weights"], 1.5, order, depth=4, precision=precision, nrhs_max=wide,
                 corr="none", point_tri=q["point_tri"])
        start = P.export_tree(4)["start"]
        assert np.diff(start).max() > 32 and n < 32 * P.info()["nbox"][4]
        y.append(P.matvec(a, b))
        P.close()
    assert torch.linalg.norm(y[0] - y[1]) <= (1e-13 if precision == "fp64" else 1e-5) * torch.linalg.norm(y[0])

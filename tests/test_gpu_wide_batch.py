"""The largest batch that a plan takes, 1,024 right-hand sides, on a body whose
translations then hold more threads than one launch may have (2^32)."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_largest_batch_equals_single_calls():
    """52,000 nodes in 46,379 leaves: the translations to the leaves from their parents are 5,798 groups of 256
    threads for each channel and right-hand side, 4.6e9 threads.  Every column equals that of a single call, bit
    for bit."""
    from paper_1211_7177_amd import Plan
    n, wide = 52000, 1024
    if torch.cuda.mem_get_info()[1] < 200 << 30:
        pytest.skip("needs 110 GB of device memory")
    rng = np.random.default_rng(5)
    p = rng.standard_normal((n, 3))
    p /= np.linalg.norm(p, axis=1)[:, None]
    print("wide batch", n, wide, flush=True)
    P = Plan(p, p, np.full(n, 4 * np.pi / n), 1.0, 0, depth=8, nrhs_max=wide, corr="none", tol=0.3)
    inf = P.info()
    assert inf["order"] == 3 and -(-inf["nbox"][8] // 8) * 3 * wide * 256 >= 1 << 32
    g = torch.Generator(device="cuda").manual_seed(7)
    a, b = (torch.randn((4, n, 3), dtype=torch.complex128, device="cuda", generator=g) for _ in range(2))
    y = P.matvec(a.repeat(wide // 4, 1, 1), b.repeat(wide // 4, 1, 1)).view(wide // 4, 4, n, 3)
    for r in range(4):
        one = P.matvec(a[r], b[r])
        assert bool((y[:, r] == one).all()) and bool(torch.isfinite(torch.view_as_real(one)).all())
    P.close()

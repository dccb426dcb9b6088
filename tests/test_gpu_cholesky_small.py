"""The factorisation of a matrix smaller than a diagonal block of 64: a chain as long as the
matrix, and not as the block."""
import time

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _spd(n):
    g = torch.randn(n, n, dtype=torch.float64, generator=torch.Generator().manual_seed(n))
    return (g @ g.T / n + torch.eye(n, dtype=torch.float64)).cuda()


@pytest.mark.parametrize("n", [1, 2, 7, 8, 9, 15, 16, 17, 55, 56, 57, 63])
def test_panels_up_to_the_matrix(n):
    """A = G G^T / n + I has a condition below 6 or so: residuals within some n roundings."""
    import paper_1707_03771_amd as dfx
    A = _spd(n)
    L, Li = dfx.cholesky(A)
    one = torch.eye(n, dtype=torch.float64, device="cuda")
    tol = 8 * (n + 8) * 2.0 ** -53
    assert torch.equal(L, torch.tril(L)) and torch.equal(Li, torch.tril(Li))
    assert float((L @ L.T - A).abs().max()) <= tol * float(A.abs().max())
    assert float((Li @ L - one).abs().max()) <= tol * 6.0


def test_one_row_takes_less_than_a_block():
    """1 x 1 and 64 x 64: launches, copies and the wait are the same, the chain is 64 times as
    long (0.87 of the time with a whole block's chain for either)."""
    import paper_1707_03771_amd as dfx
    best = {}
    for n in (1, 64):
        A = _spd(n)
        for _ in range(40):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            dfx.cholesky(A)
            torch.cuda.synchronize()
            best[n] = min(best.get(n, 1.0), time.perf_counter() - t0)
    print(f"{best[1] * 1e6:.1f} and {best[64] * 1e6:.1f} us")
    assert best[1] <= 0.75 * best[64]

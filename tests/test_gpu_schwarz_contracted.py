"""Schwarz factors of contracted shells, below and above the four primitives from which the
s and p pairs' Rys coefficients are staged in LDS, against the oracle.  All
contributions are positive squares of integrals to some 1e-14 each: 1e-12 of the largest."""
import time

import numpy as np
import pytest

import oracle as O
import systems

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _shells(ls, nprim, nat, seed=0):
    rng = np.random.default_rng(seed)
    ctr = rng.uniform(-9.0, 9.0, (nat, 3))
    return [systems.shell(c, l, [0.3 * 2.2 ** k for k in range(nprim)], [0.5 - 0.03 * k for k in range(nprim)])
            for c in ctr for l in ls]


@pytest.mark.parametrize("ls", [(0,), (0, 1), (0, 1, 2), (1, 3)])
@pytest.mark.parametrize("nprim", [1, 3, 4, 6])
def test_schwarz_factors(ls, nprim):
    import paper_1707_03771_amd as dfx
    sh = _shells(ls, nprim, 3 if 3 in ls else 5)
    sh[0] = systems.shell(sh[0]["center"], ls[0], [0.7])  # pairs of unequal lengths
    ax = [systems.shell([0.0, 0.0, 0.0], 0, [1.0])]
    Q = dfx.eri3(sh, ax).lists()[3]
    Qo = O.schwarz(O.Basis(sh), O.Basis(ax))[0]
    assert np.abs(Q - Qo).max() <= 1e-12 * Qo.max()


def test_long_contractions_of_s_are_cheap():
    """1830 pairs of ten-fold contracted s shells against as many of p shells, whose sums over
    components and recursions take four times as long (0.25; 0.31 with the power table and
    the coefficients of s pairs in memory)."""
    import paper_1707_03771_amd as dfx
    ax = [systems.shell([0.0, 0.0, 0.0], 0, [1.0])]
    best = {}
    for l in (0, 1):
        sh = _shells((l,), 10, 60)
        for _ in range(4):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            dfx.eri3(sh, ax).free()
            torch.cuda.synchronize()
            best[l] = min(best.get(l, 10.0), time.perf_counter() - t0)
    print(f"s {best[0] * 1e3:.1f} ms, p {best[1] * 1e3:.1f} ms")
    assert best[0] <= 0.28 * best[1]

"""The purification's step kernel at the edges of its 32 x 32 tiles and of its blocks
of k, odd sizes included: an SCF with it against one that takes every occupied space
from the full eigen-decomposition.  Both converge to |dE| < 1e-11 and a commutator
below 1e-7, which fixes the energy, second order in that error, to about 1e-12 of
its few tens of Hartree: 1e-9 absolute bounds it with the rounding of the sums."""
import numpy as np
import pytest

import systems

pytestmark = pytest.mark.gpu


def helium_line(nfun):
    """Helium atoms on a line with nfun s functions between them, six exponents at most each."""
    na = max(1, -(-nfun // 6))
    xyz = [[3.0 * a, 0.2 * (a % 2), 0.0] for a in range(na)]
    sh, ax = [], []
    for a in range(na):
        for j in range(len(range(a, nfun, na))):
            sh.append(systems.shell(xyz[a], 0, [40.0 * 0.3 ** j]))
        for j in range(7):
            ax.append(systems.shell(xyz[a], 0, [80.0 * 0.33 ** j]))
        ax.append(systems.shell(xyz[a], 1, [0.8]))
    return np.array(xyz), [2] * na, sh, ax


@pytest.mark.parametrize("nfun", [3, 8, 31, 32, 33, 64, 65, 97, 130])
def test_purified_and_diagonalised_scf_agree(nfun):
    import paper_1707_03771_amd as dfx
    xyz, Z, sh, ax = helium_line(nfun)
    opt = dict(schedule=dfx.SCHED_FP64, conv_dE=1e-11, conv_err=1e-7, max_iter=60)
    E, _, eps, info = dfx.scf(xyz, Z, sh, ax, purify=1, **opt)
    E0, _, eps0, info0 = dfx.scf(xyz, Z, sh, ax, purify=0, **opt)
    assert info["n_purified"] > 0 and info0["n_purified"] == 0
    assert info["purify_steps"] >= 4 * info["n_purified"]
    assert abs(E - E0) <= 1e-9
    # levels are first order in the Fock matrix, whose error is that of the density: the commutator's
    assert np.abs(eps - eps0).max() <= 1e-6

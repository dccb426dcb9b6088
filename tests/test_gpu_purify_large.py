"""The purification at and beyond the largest size of its step kernel (1792 functions).
Beyond, P is squared by the symmetric product for an even number of functions and by
the general one for an odd number, traces and decisions by way of the host.  Systems
and bounds as for the step kernel (test_gpu_purify_sizes.py); the energies are fourteen
times as large, and so are the step that counts as none and the bound on their
difference, rounded up."""
import numpy as np
import pytest

from test_gpu_purify_sizes import helium_line

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nfun", [1792, 1793, 1796])
def test_purified_and_diagonalised_scf_agree_at_the_line(nfun):
    import paper_1707_03771_amd as dfx
    xyz, Z, sh, ax = helium_line(nfun)
    opt = dict(schedule=dfx.SCHED_FP64, conv_dE=1e-9, conv_err=1e-7, max_iter=60)
    E, _, eps, info = dfx.scf(xyz, Z, sh, ax, purify=1, **opt)
    E0, _, eps0, info0 = dfx.scf(xyz, Z, sh, ax, purify=0, **opt)
    print(f"{nfun} functions: {info['niter']} iterations, {info['n_purified']} purified, "
          f"{info['purify_steps']} steps, |dE| {abs(E - E0):.1e}, levels {np.abs(eps - eps0).max():.1e}")
    assert info["ndropped"] == 0  # so every update is of this size
    assert info["n_purified"] > 0 and info0["n_purified"] == 0
    assert info["purify_steps"] >= 4 * info["n_purified"]
    assert abs(E - E0) <= 2e-8
    assert np.abs(eps - eps0).max() <= 1e-6

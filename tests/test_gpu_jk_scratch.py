"""Builds whose scratch is cut by the tiles of B that hold a kept pair, at numbers of kept
tiles where that cut asks for more parts than the one with every tile kept
(tests/test_jk_scratch.py sweeps the plans on the host).  Atoms a bohr apart on a
line, the shells of each together and the most diffuse of them such that pairs of
atoms are screened from a chosen distance on, so that a few tiles hold none."""
import numpy as np
import pytest

import systems

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def dfx():
    import paper_1707_03771_amd as m
    return m


def _tiles(rows):
    nt = (rows.shape[1] + 31) // 32
    return sum(bool((rows[:, 32 * i:32 * i + 32, 32 * j:32 * j + 32] != 0).any()) for i in range(nt)
               for j in range(i + 1)), nt * (nt + 1) // 2


def coulomb_line():
    """225 s functions, 32 on each of seven centres and one on an eighth; 1169 auxiliary s functions."""
    sh = [systems.shell([float(f // 32), 0.0, 0.0], 0, [1.85 + 0.2 * (f % 32)]) for f in range(225)]
    ax = [systems.shell([0.5 * q, 0.0, 0.0], 0, [4.0]) for q in range(1169)]
    return sh, ax


def gradient_line():
    """Nine atoms of 30 orbital and 90 auxiliary functions."""
    xyz = np.array([[float(a), 0.0, 0.0] for a in range(9)])
    sh, ax = [], []
    for r in xyz:
        for e in (1.2, 4.0, 12.0):
            sh += [systems.shell(r, l, [e]) for l in range(3)]
        sh.append(systems.shell(r, 1, [36.0]))
        for e in (4.0, 14.0, 50.0):
            ax += [systems.shell(r, l, [e]) for l in range(5)]
        ax += [systems.shell(r, l, [180.0]) for l in (0, 1, 2)]
        ax += [systems.shell(r, l, [650.0]) for l in (0, 2)]
    return xyz, sh, ax


def test_coulomb_alone_with_33_of_36_tiles(dfx):
    """J of a density and of orbitals without K, whose scratch would hide the Coulomb build's."""
    sh, ax = coulomb_line()
    B = dfx.eri3(sh, ax)
    assert (B.nbf, B.naux) == (225, 1169)
    rows = B.unpack()
    assert _tiles(rows) == (33, 36)
    g = torch.Generator().manual_seed(2)
    C = torch.randn((225, 24), generator=g, dtype=torch.float64).cuda()
    D = C @ C.T
    ref = torch.tensordot((rows * D).sum((1, 2)), rows, dims=1)
    for kw in (dict(), dict(kind=dfx.DENSITY)):
        J, K = dfx.jk(B, D if kw else C, want_k=False, **kw)
        assert K is None
        # sums of 225^2 and 1169 products in another order
        assert (J - ref).abs().max() <= 1e-11 * ref.abs().max()
    B.free()


def test_gradient_with_44_of_45_tiles(dfx):
    """The gradient does not depend on the order of the shells: all of them atom by atom, and
    dealt over the atoms in turn, where every tile holds a kept pair.  The same
    integrals and products are summed in another order through a metric of a
    condition below 1e6: 1e-16 1e6, with two digits for the cancellation of its parts."""
    xyz, sh, ax = gradient_line()
    B = dfx.eri3(sh, ax)
    assert (B.nbf, B.naux) == (270, 810)
    assert _tiles(B.unpack()) == (44, 45)
    assert B.info["kappa_lb"] < 1e6
    B.free()
    order = sorted(range(len(sh)), key=lambda s: (s % 10, s // 10))
    nf = [2 * s["l"] + 1 for s in sh]
    first = np.concatenate([[0], np.cumsum(nf)])
    rows = np.concatenate([np.arange(first[s], first[s] + nf[s]) for s in order])
    rng = np.random.default_rng(4)
    C = np.linalg.qr(rng.normal(size=(270, 27)))[0]
    eps = np.linspace(-3.0, -0.4, 27)
    Z = [6] * 9
    g0, _ = dfx.rhf_grad(xyz, Z, sh, ax, C, eps)
    g1, _ = dfx.rhf_grad(xyz, Z, [sh[s] for s in order], ax, C[rows], eps)
    assert np.abs(g0 - g1).max() <= 1e-8 * np.abs(g1).max()


@pytest.mark.parametrize("prec,nbf,naux,npos,nneg,tol", [
    (0, 100, 292, 47, 46, 1e-10), (0, 100, 292, 46, 47, 1e-10), (1, 65, 292, 29, 28, 1e-5),
    (2, 65, 292, 29, 28, 2e-2), (0, 600, 40, 600, 0, 1e-10), (0, 600, 40, 520, 80, 1e-10)])
def test_density_with_unequal_signs(dfx, prec, nbf, naux, npos, nneg, tol):
    """K of an indefinite density whose smaller count of one sign takes more scratch than the
    larger, and of densities of more than 512 columns.  FP64 as K of a density by its
    eigenvectors elsewhere (1e-10), the others at what they reach against the oracle,
    of the largest element of the positive part."""
    sh = [systems.shell([0.9 * f, 0.1 * (f % 2), 0.0], 0, [0.9 + 0.001 * f]) for f in range(nbf)]
    ax = [systems.shell([0.9 * nbf / naux * q, 0.0, 0.0], 0, [4.0 * (naux / nbf) ** 2]) for q in range(naux)]
    B = dfx.eri3(sh, ax)
    assert (B.nbf, B.naux) == (nbf, naux)
    rows = B.unpack()
    g = torch.Generator().manual_seed(11)
    Q = torch.linalg.qr(torch.randn((nbf, nbf), generator=g, dtype=torch.float64))[0].cuda()
    w = torch.zeros(nbf, dtype=torch.float64, device="cuda")
    w[:npos] = torch.linspace(0.5, 2.0, npos, dtype=torch.float64)
    w[npos:npos + nneg] = -torch.linspace(0.5, 1.5, nneg, dtype=torch.float64)
    k_of = lambda w: torch.matmul(torch.matmul(rows, ((Q * w) @ Q.T).expand(naux, nbf, nbf)), rows).sum(0)  # noqa: E731
    D = (Q * w) @ Q.T
    K = dfx.jk(B, (D + D.T) / 2, kind=dfx.DENSITY, precision=prec, want_j=False)[1]
    scale = max(1.0, k_of(w.clamp(min=0)).abs().max().item())
    assert (K - k_of(w)).abs().max() <= tol * scale
    B.free()

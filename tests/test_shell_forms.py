"""The forms in which a shell's numbers may come: what reaches the library is what
np.ascontiguousarray makes of exps and coefs and float() of the centre's first three items,
whatever mixture of lists, tuples, arrays and tensors a basis is made of (host only)."""
import ctypes

import numpy as np
import pytest

import paper_1707_03771_amd as dfx

torch = pytest.importorskip("torch")

COLUMNS = [
    [1.5, 0.25], (3.0,), [2, 1], np.array([0.5, 4.0, 8.0]), np.array([1.0, 2.0], np.float32), np.arange(6.0)[::2],
    torch.tensor([0.75, 0.5], dtype=torch.float64), [[1.0], [2.0], [3.0]], np.array([[1.0], [2.0]]), np.float64(7.0), 9.0,
    [np.float64(1.0), np.float32(0.5)], [np.array([2.0]), np.array([4.0])], ["1.25", "2.5"], range(1, 4),
    [torch.tensor(3.0), torch.tensor(5.0)],
]
CENTRES = [[0.0, 1.0, 2.0], (1, 2, 3), np.array([0.1, 0.2, 0.3]), np.arange(4.0), torch.tensor([1.0, 2.0, 3.0]),
           ["0.5", "1.5", "2.5"], {0: 1.0, 1: 2.0, 2: 4.0}]


def read(a, i):
    s = a.arr[i]
    get = lambda p: list((ctypes.c_double * s.nprim).from_address(p))  # noqa: E731
    return list(s.xyz), s.l, get(s.exps), get(s.coefs)


def plain(s):
    e, c = (np.ascontiguousarray(s[k], dtype=np.float64) for k in ("exps", "coefs"))
    return [float(s["center"][k]) for k in range(3)], int(s["l"]), list(e.ravel()[:len(e)]), list(c.ravel()[:len(e)])


@pytest.mark.parametrize("take", ["each", "all", "lists"])
def test_every_form_reaches_the_library(take):
    cols = [c for c in COLUMNS if take != "lists" or isinstance(c, (list, tuple))]
    shells = [{"center": CENTRES[i % len(CENTRES)], "l": np.int64(i % 4), "exps": c, "coefs": c}
              for i, c in enumerate(cols)]
    for group in ([[s] for s in shells] if take == "each" else [shells]):
        a = dfx._ShellArray(group)
        assert a.n == len(group)
        for i, s in enumerate(group):
            assert read(a, i) == plain(s)


@pytest.mark.parametrize("bad", [{"center": [1.0]}, {"center": [1.0, 2.0]}, {"center": 1.0}, {"center": [None] * 3},
                                 {"exps": [[1.0], [2.0, 3.0]]}, {"coefs": [1j]}, {"l": None}])
def test_what_has_no_such_numbers_is_refused(bad):
    good = {"center": [0.0, 0.0, 0.0], "l": 0, "exps": [1.0], "coefs": [1.0]}
    for shells in ([{**good, **bad}], [good, {**good, **bad}]):
        with pytest.raises((TypeError, ValueError, IndexError)):
            dfx._ShellArray(shells)


def test_no_shells():
    assert dfx._ShellArray([]).n == 0

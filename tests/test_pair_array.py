"""The epm_pair array of a batch as the binding marshals it: the fields as
plain ctypes assignments write them, whatever the specs hold -- matrices that
change after they were given, values that wrap, and what is refused."""

import copy
import ctypes
import pickle

import numpy as np
import pytest

import paper_2603_18401_amd as E


def _fields(specs):
    """Field by field; F as nine numbers."""
    arr = (E._Pair * len(specs))()
    q = k = 0
    for a, s in zip(arr, specs):
        a.F[:] = [float(v) for v in s.F]
        a.w2, a.h2 = s.w2, s.h2
        a.q_begin, a.m, a.k_begin, a.n = q, s.m, k, s.n
        q += s.m
        k += s.n
    return arr, q, k


def _same(specs):
    got, want = E._pair_array(specs), _fields(specs)
    assert got[1:] == want[1:]
    assert ctypes.sizeof(got[0]) == ctypes.sizeof(want[0])
    assert bytes(got[0]) == bytes(want[0])
    return got[0]


def _spec(F, w2=640, h2=480, m=3, n=5):
    return E.PairSpec(F, w2, h2, m, n)


BASE = np.arange(1.0, 10.0).reshape(3, 3)


@pytest.mark.parametrize("F", [BASE, BASE.T, BASE.astype(np.float32), BASE.tolist(),
                               np.asfortranarray(BASE), np.repeat(BASE, 2)[::2],
                               BASE.astype(">f8"), BASE.astype(int)],
                         ids=["c", "transposed", "f32", "list", "fortran", "strided",
                              "big-endian", "int"])
def test_matrices_given(F):
    a = _same([_spec(F), _spec(F, m=0, n=0), _spec(F, m=np.int64(7))])
    assert list(a[0].F) == np.asarray(F, float).reshape(9).tolist()


def test_no_pairs():
    _same([])


@pytest.mark.parametrize("make", [lambda: BASE.reshape(9).copy(),
                                  lambda: BASE.reshape(9).astype(np.float32),
                                  lambda: BASE.reshape(9).tolist(),
                                  lambda: np.repeat(BASE.reshape(9), 2)[::2]],
                         ids=["f64", "f32", "list", "strided"])
def test_matrices_assigned_and_changed(make):
    s = _spec(np.zeros((3, 3)))
    F = make()
    s.F = F
    _same([s])
    F[4] = -2.5  # the caller's own object, changed after it was assigned
    a = _same([s])
    assert a[0].F[4] == -2.5
    s.F[0] = 11.0
    a = _same([s, copy.copy(s), pickle.loads(pickle.dumps(s))])
    assert a[0].F[0] == a[2].F[0] == 11.0


def test_a_given_matrix_that_changes():
    F = BASE.copy()
    s = _spec(F)
    F[1, 1] = 0.25
    a = _same([s])
    assert a[0].F[4] == 0.25


def test_specs_of_other_kinds():
    class Own:
        F, w2, h2, m, n = tuple(range(9)), 10, 20, 1, 2

    class Sub(E.PairSpec):
        @property
        def F(self):
            return [1.0] * 9

        @F.setter
        def F(self, F):
            pass

    _same([Own(), Sub(BASE, 1, 2, 3, 4), _spec(BASE)])
    old = E.PairSpec.__new__(E.PairSpec)  # as saved before F was a property
    old.__dict__.update(F=BASE.reshape(9), w2=640, h2=480, m=3, n=5)
    _same([old])


@pytest.mark.parametrize("field", ["w2", "h2"])
@pytest.mark.parametrize("value", [2 ** 31, -2 ** 31 - 1, 2 ** 32 + 640])
def test_sizes_that_wrap(field, value):
    s = _spec(BASE)
    setattr(s, field, value)
    _same([s])


@pytest.mark.parametrize("what,value", [("F", BASE), ("F", [1.0] * 8), ("F", None),
                                        ("w2", 640.0), ("m", 3.0), ("n", None)])
def test_what_is_refused(what, value):
    s = _spec(BASE)
    with pytest.raises((TypeError, ValueError)):
        setattr(s, what, value)
        E._pair_array([s])

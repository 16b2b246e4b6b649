"""Small mechanisms and states at the edges of the rate expressions, with what
the oracle gives there; used by the host and the GPU tests of both kernel forms.
"""
import numpy as np

from workloads import tiny


def states(n, T, p=101325.0, y=(0.3, 0.2, 0.1, 0.4)):
    """n cells of the four-species mechanisms of workloads.tiny, over the given
    temperatures."""
    T = np.resize(np.asarray(T, dtype=np.float64), n)
    return T, np.full(n, float(p)), np.tile(np.asarray(y, dtype=np.float64), (n, 1))


# A Troe centre below zero: alpha is not bounded, and (1 - alpha) e^{-T/T3} +
# alpha e^{-T/T1} is negative above some temperature for alpha > 1 and T3 > T1.
# ln of it is NaN, so is the rate.  Here below zero from 200 K on at T1 = 50, and
# above it at T1 = 5000.
CENTRE = {"below": tiny.falloff(troe=(1.5, 1000.0, 50.0, None)),
          "above": tiny.falloff(troe=(1.5, 1000.0, 5000.0, None))}
CENTRE_T = [300.0, 900.0, 1500.0, 2900.0]


def oracle_source(om, T, p, Y):
    return np.array([om.rhs(p[i], np.concatenate([[T[i]], Y[i]])) for i in range(len(T))])


def check_source(f, fo):
    """The other parity tests' bar on source terms, and NaN exactly where the
    oracle has it."""
    assert np.array_equal(np.isnan(f), np.isnan(fo)), (f, fo)
    ok = ~np.isnan(fo).any(axis=1)
    assert np.all(np.abs(f - fo)[ok] <= 1e-11 * np.abs(fo[ok]).max(axis=1, keepdims=True) + 1e-300), (f, fo)

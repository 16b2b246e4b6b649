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


# Isomers A <=> B (dS = 1 R, same cp) whose enthalpies lie so far apart that
# 1/K_c is beyond the largest double in a cold cell, with an activation
# temperature that leaves the reverse rate an ordinary number.
RU = 8.314462618
DH, EA = 251000.0, 251371.0                    # (H_B - H_A)/R, Ea/R in K
FAR = {kind: tiny.text([("H", 1.008), ("O", 15.999), ("N", 14.007)],
                       [("A", "H=1,O=1"), ("B", "H=1,O=1"), ("C", "H=1,O=1"), ("N2", "N=2")],
                       [tiny._thermo("A", 3.5, -1000.0, 5.0), tiny._thermo("B", 3.5, DH - 1000.0, 6.0),
                        tiny._thermo("C", 3.5, -1000.0, 5.0), tiny._thermo("N2", 3.5, -1000.0, 4.0)],
                       [f"reaction {kind} A=1 B=1 {a!r} 0.0 {e * RU * 1e-3!r}{more}"])
       for kind, a, e, more in (("elementary", 1e13, EA, ""), ("thirdbody", 1e17, EA, ""),
                                ("plog", 1.0, 0.0, f" plog=1000.0:1e13:0.0:{EA * RU * 1e-3!r},"
                                 f"1e6:1e13:0.0:{EA * RU * 1e-3!r}"))}
FAR_T = [300.0, 330.0, 900.0]
FAR_Y = [(0.4, 0.3, 0.2, 0.1), (0.7, 0.0, 0.2, 0.1), (0.0, 0.7, 0.2, 0.1)]


def far_source(kind, T, p, Y):
    """dT/dt and dY/dt of FAR[kind] in numpy, the reverse rate constant as the
    exponential of the difference of logarithms."""
    W = np.array([17.007e-3, 17.007e-3, 17.007e-3, 28.014e-3])
    sig = (Y / W).sum(axis=1)
    rho = p / (RU * T * sig)
    C = rho[:, None] * Y / W
    lnk = np.log(1e13) - EA / T
    kf, kr = np.exp(lnk), np.exp(lnk - (1.0 - DH / T))
    q = kf * C[:, 0] - kr * C[:, 1]
    if kind == "thirdbody":
        q = 1e17 / 1e13 * 1e-6 * C.sum(axis=1) * q      # cm^3/mol -> m^3/mol
    f = np.zeros((len(T), 5))
    f[:, 1], f[:, 2] = -W[0] * q / rho, W[1] * q / rho
    f[:, 0] = -DH * q / (rho * sig * 3.5)               # -sum h wdot / (rho cp), cp/R = 3.5 throughout
    return f


# A logarithm of a subnormal number: the sum of an SRI factor, or a Troe centre,
# that is e^{-T/2} alone.  log10(P_r) is about 10, so F stays an ordinary number.
SMALL = {"sri": tiny.falloff(kind="sri", A0=1e28, sri=(0.0, 300.0, 2.0, 1.0, 0.0)),
         "troe": tiny.falloff(kind="troe", A0=1e28, troe=(1.0, 300.0, 2.0, None))}
SMALL_T = [1000.0, 1424.0, 1432.0, 1440.0]


def small_tolerance(T):
    """The bar of the parity tests, and what one unit in the last place of the
    subnormal e^{-T/2} (2^-1074) makes of it: its logarithm enters F with a factor
    of order one."""
    return 1e-11 + 4.0 * 2.0 ** -1074 / np.exp(-np.asarray(T) / 2.0)


def oracle_source(om, T, p, Y):
    return np.array([om.rhs(p[i], np.concatenate([[T[i]], Y[i]])) for i in range(len(T))])


def check_source(f, fo):
    """The other parity tests' bar on source terms, and NaN exactly where the
    oracle has it."""
    assert np.array_equal(np.isnan(f), np.isnan(fo)), (f, fo)
    ok = ~np.isnan(fo).any(axis=1)
    assert np.all(np.abs(f - fo)[ok] <= 1e-11 * np.abs(fo[ok]).max(axis=1, keepdims=True) + 1e-300), (f, fo)


def oracle_jacobian(om, T, p, Y):
    return np.array([om.jac(p[i], np.concatenate([[T[i]], Y[i]])) for i in range(len(T))])


def check_small(f, fj, J, fo, Jo, T):
    tol = small_tolerance(T)
    for g in (f, fj):
        assert np.all(np.abs(g - fo) <= tol[:, None] * np.abs(fo).max(axis=1, keepdims=True)), (g, fo)
    scale = np.abs(Jo).max(axis=2, keepdims=True)
    assert np.all(np.abs(J - Jo) <= 10.0 * tol[:, None, None] * scale), (J, Jo)

"""The wave-cooperative adjoint's rerun of the forward integration, which rounds
differently from the forward kernels: a step whose error estimate sits at the
acceptance limit may be accepted by one and rejected by the other.  The cells
here are put there by bisection in T0: the two neighbouring doubles between
which the forward kernels' first step, of the whole dt, stops being accepted."""
import os

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from workloads import mech_path, mech_text  # noqa: E402
from workloads.states import uniform_cells  # noqa: E402

RTOL, ATOL = 1e-8, 1e-12
# (the 32-species rates are slower: at 1e-9 s every cell takes one step)
MECHS = [("m9", "0", 1e-9), ("m16", None, 1e-9), ("m32", None, 1e-7)]


@pytest.fixture(scope="module")
def chem():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2508_16105_amd as chem
    return chem


def _g(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda:0")


@pytest.fixture(scope="module", params=MECHS, ids=[m for m, _, _ in MECHS])
def limit(request, chem):
    """(mechanism, dt, T accepted at once, T not, p, Y)"""
    name, lane_max, dt = request.param
    old = os.environ.pop("CHEM_LANE_MAX_SPECIES", None)
    try:
        if lane_max is not None:
            os.environ["CHEM_LANE_MAX_SPECIES"] = lane_max
        gm = chem.Mechanism(mech_path(name))
    finally:
        os.environ.pop("CHEM_LANE_MAX_SPECIES", None)
        if old is not None:
            os.environ["CHEM_LANE_MAX_SPECIES"] = old
    n = 256
    _, p, Y = uniform_cells(mech_text(name), n, 77)
    pg, Yg = _g(p), _g(Y)

    def at_once(T):
        r = chem.integrate(gm, _g(T), pg, Yg, dt, RTOL, ATOL, return_counts=True, allow_failed=True)
        return ((r[4] == 1) & (r[5] == 0)).cpu().numpy()
    lo, hi = np.full(n, 300.0), np.full(n, 3000.0)
    a, b = at_once(lo), at_once(hi)
    lo, hi = np.where(a, lo, hi), np.where(a, hi, lo)       # accepted at lo, not at hi (where they differ)
    use = a != b
    while True:
        mid = 0.5 * (lo + hi)
        inside = (mid != lo) & (mid != hi) & use
        if not inside.any():
            break
        ok = at_once(mid)
        lo, hi = np.where(inside & ok, mid, lo), np.where(inside & ~ok, mid, hi)
    assert use.sum() >= 32
    return gm, dt, lo[use], hi[use], p[use], Y[use]


def _adjoint(chem, gm, dt, T, p, Y, **kw):
    gT, gY = np.full(len(T), 1e-3), np.zeros(Y.shape)
    gY[:, 2] = 1.0
    out = chem.integrate_adjoint(gm, _g(T), _g(p), _g(Y), dt, RTOL, ATOL, _g(gT), _g(gY), allow_failed=True, **kw)
    return [v.cpu().numpy() if torch.is_tensor(v) else v for v in out]


def test_cells_the_forward_accepts_do_not_fail_in_the_rerun(chem, limit):
    """One attempt allowed, taken and accepted by the forward kernels: with and
    without their counts the call succeeds, also where the rerun rejects it."""
    gm, dt, T, _, p, Y = limit
    r = chem.integrate(gm, _g(T), _g(p), _g(Y), dt, RTOL, ATOL, return_counts=True, max_substeps=1)
    assert bool((r[3] == 0).all()) and bool((r[4] == 1).all())
    plain = _adjoint(chem, gm, dt, T, p, Y, max_substeps=1)
    told = _adjoint(chem, gm, dt, T, p, Y, max_substeps=1, forward_nacc=r[4])
    alone = _adjoint(chem, gm, dt, T, p, Y, max_substeps=1, forward_nacc=r[4], end_state=False)
    assert alone[5] is None and alone[6] is None
    for o in (plain, told, alone):
        assert o[7]["failed"] == 0
        assert all(np.isfinite(v).all() for v in o[:5])
        assert all(np.array_equal(x, y) for x, y in zip(o[:5], plain[:5]))
    for o in (plain, told):
        assert np.array_equal(o[5], r[0].cpu().numpy()) and np.array_equal(o[6], r[1].cpu().numpy())
    print("rerun took more steps in", plain[7]["accepted"] - len(T), "of", len(T), "cells")


def test_cells_the_forward_fails_fail(chem, limit):
    """The neighbouring doubles: one attempt is not enough for the forward kernels,
    so every cell fails, also where the rerun accepts it."""
    gm, dt, _, T, p, Y = limit
    r = chem.integrate(gm, _g(T), _g(p), _g(Y), dt, RTOL, ATOL, return_counts=True, max_substeps=1, allow_failed=True)
    assert bool((r[3] == 1).all())
    o = _adjoint(chem, gm, dt, T, p, Y, max_substeps=1)
    assert o[7]["failed"] == len(T)
    assert np.isnan(o[0]).all() and np.isnan(o[1]).all()
    assert all(np.all(g == 0.0) for g in o[2:5])
    assert np.array_equal(o[5], r[0].cpu().numpy()) and np.array_equal(o[6], r[1].cpu().numpy())


def test_an_entry_below_the_forward_count_fails_its_cell_alone(chem, limit):
    gm, dt, _, T, p, Y = limit
    r = chem.integrate(gm, _g(T), _g(p), _g(Y), dt, RTOL, ATOL, return_counts=True)
    assert bool((r[3] == 0).all()) and int(r[4].min()) >= 2
    base = _adjoint(chem, gm, dt, T, p, Y)
    short = r[4].clone()
    bad = np.arange(0, len(T), 5)
    short[torch.tensor(bad, device="cuda:0")] = 1
    keep = np.setdiff1d(np.arange(len(T)), bad)
    only = _adjoint(chem, gm, dt, T[keep], p[keep], Y[keep])
    for kw in ({}, {"end_state": False}):
        o = _adjoint(chem, gm, dt, T, p, Y, forward_nacc=short, **kw)
        # (a rerun that accepts the first step needs no more than the entry)
        failed = np.isnan(o[0])
        assert failed.sum() == o[7]["failed"] >= len(bad) // 4 and not failed[keep].any()
        assert np.array_equal(o[0][keep], base[0][keep]) and np.array_equal(o[1][keep], base[1][keep])
        if failed.sum() == len(bad):
            for k in (2, 3, 4):
                assert np.allclose(o[k], only[k], rtol=1e-11, atol=1e-11 * np.abs(only[k]).max())

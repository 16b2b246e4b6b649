"""Sizes at which the kernels' splits have their edges.

Wave-cooperative form (16 lanes a cell, 4 cells a wave, 4 waves a workgroup):
cell counts around each of these, mechanisms with one and two matrix rows a
lane, with and without every form of rate.  A cell's result does not depend on
the cells beside it, so prefixes are compared bitwise, the longest with the
oracle at the tolerances of the other parity tests (|dT| <= 1e-6 T, |dY| <= 1e-8
at rtol 1e-8).

Plain launches above the lanes the chip holds at once deal cells to idle lanes:
bitwise the launches that fit, and the persistent form."""
import os

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from workloads import mech_path, mech_text  # noqa: E402
from workloads.states import uniform_cells  # noqa: E402

RTOL, ATOL = 1e-8, 1e-12


@pytest.fixture(scope="module")
def chem():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2508_16105_amd as chem
    return chem


def _g(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda:0")


def _load(chem, name, lane_max=None):
    old = os.environ.pop("CHEM_LANE_MAX_SPECIES", None)
    try:
        if lane_max is not None:
            os.environ["CHEM_LANE_MAX_SPECIES"] = str(lane_max)
        return chem.Mechanism(mech_path(name))
    finally:
        os.environ.pop("CHEM_LANE_MAX_SPECIES", None)
        if old is not None:
            os.environ["CHEM_LANE_MAX_SPECIES"] = old


@pytest.mark.parametrize("name", ["m9", "m13x", "m16", "m32", "m32x"])
def test_wave_cooperative_cell_counts(chem, oracle_lib, name):
    gm, om = _load(chem, name, 0), oracle_lib.Mechanism(mech_path(name))
    n, dt = 65, 1e-8
    T, p, Y = uniform_cells(mech_text(name), n, 91)
    a = [_g(v) for v in (T, p, Y)]
    Tw, Yw, _ = chem.integrate(gm, *a, dt, RTOL, ATOL)
    f, J = chem.eval_source(gm, *a, jacobian=True)
    g = chem.eval_source(gm, *a, jacobian=False)[0]
    h = chem.step_fixed(gm, *a, 1e-10, RTOL, ATOL)
    To, Yo, _, _, _ = om.integrate(T, p, Y, dt, RTOL, ATOL)
    assert np.all(np.abs(Tw.cpu().numpy() - To) <= 1e-6 * To)
    assert np.all(np.abs(Yw.cpu().numpy() - Yo) <= 1e-8)
    for k in (1, 3, 4, 5, 15, 16, 17, 63, 64, 65):
        b = [v[:k].contiguous() for v in a]
        for form in (chem.FORM_PLAIN, chem.FORM_PERSISTENT):
            Tk, Yk, _ = chem.integrate(gm, *b, dt, RTOL, ATOL, form=form)
            assert torch.equal(Tk, Tw[:k]) and torch.equal(Yk, Yw[:k]), (k, form)
        fk, Jk = chem.eval_source(gm, *b, jacobian=True)
        assert torch.equal(fk, f[:k]) and torch.equal(Jk, J[:k]), k
        assert torch.equal(chem.eval_source(gm, *b, jacobian=False)[0], g[:k]), k
        # (a step of this size fails in some cells: NaN, in the same ones)
        for x, y in zip(chem.step_fixed(gm, *b, 1e-10, RTOL, ATOL), h):
            assert torch.allclose(x, y[:k], rtol=0, atol=0, equal_nan=True), k


@pytest.mark.parametrize("name,resident,first", [("m9", 65536, False), ("m9", 65536, True), ("m16", 8192, False)])
@pytest.mark.parametrize("extra", [1, 64, 777])
def test_dealt_plain_launch_is_bitwise_the_static_one(chem, name, resident, first, extra):
    gm = _load(chem, name)
    n = resident + extra
    T, p, Y = uniform_cells(mech_text(name), n, 17)
    a = [_g(v) for v in (T, p, Y)]
    h0 = _g(np.geomspace(1e-13, 1e-9, n)) if first else None
    run = lambda s, **kw: chem.integrate(gm, *(v[s].contiguous() for v in a), 2e-9, RTOL, ATOL, return_counts=True,
                                         **({} if h0 is None else {"h0": h0[s].contiguous()}), **kw)
    whole = run(slice(0, n))
    parts = [run(slice(s, min(n, s + resident // 2))) for s in range(0, n, resident // 2)]
    for k in (0, 1, 3, 4, 5):
        assert torch.equal(whole[k], torch.cat([q[k] for q in parts])), k
    if h0 is None:
        other = run(slice(0, n), form=chem.FORM_PERSISTENT)
        assert torch.equal(whole[0], other[0]) and torch.equal(whole[1], other[1])


@pytest.mark.parametrize("name,lane_max", [("m9", 0), ("m16", None), ("m32", None)])
def test_a_failed_single_step_has_no_finite_component(chem, name, lane_max):
    """Wave-cooperative form: also in the species no reaction changes, which are
    not part of the linear system; the cells beside it are untouched."""
    gm = _load(chem, name, lane_max)
    T, p, Y = uniform_cells(mech_text(name), 6, 5)
    good = [v.cpu() for v in chem.step_fixed(gm, _g(T), _g(p), _g(Y), 1e-13, RTOL, ATOL)]
    assert bool((good[2] == 1).all()) and bool(torch.isfinite(good[0]).all())
    T[3] = -1.0                                   # ln T is NaN
    yn, en, ok = (v.cpu() for v in chem.step_fixed(gm, _g(T), _g(p), _g(Y), 1e-13, RTOL, ATOL))
    assert ok.tolist() == [1, 1, 1, 0, 1, 1] and bool(torch.isnan(yn[3]).all()) and bool(torch.isnan(en[3]))
    rest = [0, 1, 2, 4, 5]
    assert torch.equal(yn[rest], good[0][rest]) and torch.equal(en[rest], good[1][rest])


@pytest.mark.parametrize("name,lane_max", [("m9", 0), ("m16", None), ("m32", None)])
@pytest.mark.parametrize("what", ["T", "p", "Y"])
def test_source_terms_of_a_state_that_is_not_finite(chem, name, lane_max, what):
    """Wave-cooperative form: NaN in every source term and Jacobian entry, also
    of the species no reaction changes; the cells beside it are untouched."""
    gm = _load(chem, name, lane_max)
    T, p, Y = uniform_cells(mech_text(name), 6, 5)
    f0, J0 = (v.cpu() for v in chem.eval_source(gm, _g(T), _g(p), _g(Y), jacobian=True))
    assert bool(torch.isfinite(f0).all()) and bool(torch.isfinite(J0).all())
    if what == "Y":
        Y[3, 0] = np.nan
    else:
        (T if what == "T" else p)[3] = np.nan
    f, J = (v.cpu() for v in chem.eval_source(gm, _g(T), _g(p), _g(Y), jacobian=True))
    g = chem.eval_source(gm, _g(T), _g(p), _g(Y), jacobian=False)[0].cpu()
    assert bool(torch.isnan(f[3]).all()) and bool(torch.isnan(J[3]).all()) and bool(torch.isnan(g[3]).all())
    rest = [0, 1, 2, 4, 5]
    assert torch.equal(f[rest], f0[rest]) and torch.equal(J[rest], J0[rest])


@pytest.mark.parametrize("name,lane_max", [("m9", None), ("m9", 0), ("m13", None), ("m13", 0), ("m16", None)])
@pytest.mark.parametrize("state", ["no mass", "too hot"])
def test_steps_that_fail_shrink_to_the_smallest(chem, name, lane_max, state):
    """Every trial step of such a cell holds NaN, so each takes 0.2 of the size
    before: 0.2^29 is the first below the default limit of 1e-20.  Its
    neighbours end as without it."""
    gm = _load(chem, name, lane_max)
    T, p, Y = uniform_cells(mech_text(name), 9, 5)
    out = []
    for k in (0, 1):
        Tw, Yw = _g(T), _g(Y)
        st, na, nr = (torch.zeros(9, dtype=torch.int32, device="cuda:0") for _ in range(3))
        chem.integrate_noalloc(gm, Tw, _g(p), Yw, 1e-9, RTOL, ATOL, status=st, nacc=na, nrej=nr)
        out.append([v.cpu() for v in (Tw, Yw, st, na, nr)])
        if state == "no mass":
            Y[4] = 0.0
        else:
            T[4] = 1e6
    assert out[1][2].tolist() == [0, 0, 0, 0, 2, 0, 0, 0, 0] and out[1][3][4] == 0 and out[1][4][4] == 29
    rest = [0, 1, 2, 3, 5, 6, 7, 8]
    assert all(torch.equal(x[rest], y[rest]) for x, y in zip(*out))


@pytest.mark.parametrize("name", ["m9", "m13"])
@pytest.mark.parametrize("state", ["no mass", "negative T"])
def test_a_failed_single_step_one_cell_per_lane(chem, oracle_lib, name, state):
    """NaN in T and in every species some reaction changes (the oracle's are), the
    cells beside it untouched."""
    gm, om = _load(chem, name), oracle_lib.Mechanism(mech_path(name))
    n = 70                                        # a whole wave and a part of one
    T, p, Y = uniform_cells(mech_text(name), n, 5)
    run = lambda: [v.cpu() for v in chem.step_fixed(gm, _g(T), _g(p), _g(Y), 1e-13, RTOL, ATOL)]
    good = run()
    assert bool((good[2] == 1).all()) and bool(torch.isfinite(good[0]).all())
    if state == "no mass":
        Y[3] = Y[66] = 0.0
    else:
        T[3] = T[66] = -1.0
    yn, en, ok = run()
    rest = [k for k in range(n) if k not in (3, 66)]
    assert ok[rest].tolist() == [1] * len(rest) and ok[[3, 66]].tolist() == [0, 0]
    assert torch.equal(yn[rest], good[0][rest]) and torch.equal(en[rest], good[1][rest])
    reacting = np.isnan(om.rhs(p[3], np.concatenate([[T[3]], Y[3]])))
    for c in (3, 66):
        assert bool(torch.isnan(en[c])) and np.all(np.isnan(yn[c].numpy())[reacting])


@pytest.mark.parametrize("name,lane_max", [("m13", None), ("m13", 0), ("m13x", None), ("m9", None), ("m16", None)])
def test_a_state_without_mass_never_passes(chem, name, lane_max):
    """Every form of launch leaves it as it was and reports it failed."""
    gm = _load(chem, name, lane_max)
    T, p, Y = uniform_cells(mech_text(name), 130, 5)
    cells = [0, 1, 4, 9, 64, 100, 129]
    Y[cells] = 0.0
    for form in (chem.FORM_PLAIN, chem.FORM_PERSISTENT):
        Tw, Yw, _, st, na, _ = chem.integrate(gm, _g(T), _g(p), _g(Y), 1e-9, RTOL, ATOL, form=form, return_counts=True,
                                              allow_failed=True)
        assert st[cells].tolist() == [2] * len(cells) and na[cells].tolist() == [0] * len(cells), form
        assert torch.equal(Tw[cells].cpu(), torch.tensor(T[cells])) and bool((Yw[cells] == 0.0).all())


@pytest.mark.parametrize("name,n", [("m9", 65536 + 777), ("m16", 8192 + 777)])
def test_a_captured_plain_launch_stands_alone(chem, name, n):
    """Replays of a plain launch above the resident lanes beside other calls on the
    same handle on another stream: each ends as it does alone."""
    gm = _load(chem, name)
    T, p, Y = uniform_cells(mech_text(name), n, 17)
    a, b = ([_g(v) for v in (T[s], p[s], Y[s])] for s in (slice(None), slice(None, None, -1)))
    run = lambda s: chem.integrate(gm, *s, 2e-10, RTOL, ATOL, form=chem.FORM_PLAIN, stats=False)[:2]
    alone = run(a), run(b)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = run(a)
    one, two = torch.cuda.Stream(), torch.cuda.Stream()
    for k in range(4):
        with torch.cuda.stream(one):
            for v in out:
                v.zero_()
            graph.replay()
        with torch.cuda.stream(two):
            other = [run(b) for _ in range(3)]
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip(out, alone[0])), k
        for o in other:
            assert all(torch.equal(x, y) for x, y in zip(o, alone[1])), k

"""Mechanisms at the sizes where the kernels change: 11 unknowns of the lane form
(the most whose factors stay in registers); wave-cooperatively three matrix rows
a lane (34 species: one unknown in the third row; 48: 47 unknowns), and the
row-per-lane form (48 reacting species; 1,782 reactions, whose tables do not fit
the LDS in the 16-lane form).  Bars as in the other parity tests."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from errnorm_ref import errnorm_bar, errnorm_with_spread  # noqa: E402
from workloads import resized  # noqa: E402
from workloads.states import uniform_cells  # noqa: E402

RTOL, ATOL = 1e-8, 1e-12


def _g(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda:0")


@pytest.fixture(scope="module")
def chem():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2508_16105_amd as chem
    return chem


@pytest.fixture(scope="module", params=sorted(resized.CASES))
def mech(request, chem, oracle_lib, tmp_path_factory):
    """(mechanism, the oracle's of the same rates, text, name)"""
    name = request.param
    wd = tmp_path_factory.mktemp("sizes")
    text = resized.CASES[name]()
    (wd / f"{name}.mech").write_text(text)
    plain = resized.resized(34) if name == "34by11" else text
    (wd / "plain.mech").write_text(plain)
    return chem.Mechanism(str(wd / f"{name}.mech")), oracle_lib.Mechanism(str(wd / "plain.mech")), plain, name


def test_source_terms_and_jacobian(chem, mech):
    gm, om, text, name = mech
    T, p, Y = uniform_cells(text, 37, 71)
    f, J = chem.eval_source(gm, _g(T), _g(p), _g(Y))
    g, _ = chem.eval_source(gm, _g(T), _g(p), _g(Y), jacobian=False)
    for k in (1, 5, 16):
        fk, Jk = chem.eval_source(gm, _g(T[:k]), _g(p[:k]), _g(Y[:k]))
        assert torch.equal(fk, f[:k]) and torch.equal(Jk, J[:k])
    f, J, g = f.cpu().numpy(), J.cpu().numpy(), g.cpu().numpy()
    for i in range(len(T)):
        y = np.concatenate([[T[i]], Y[i]])
        fo, Jo, Ja = om.rhs(p[i], y), om.jac_cs(p[i], y), om.jac(p[i], y)
        for v in (f[i], g[i]):
            assert np.all(np.abs(v - fo) <= 1e-11 * np.abs(fo).max() + 1e-300), i
        sc = np.abs(Jo).max(axis=1, keepdims=True) * np.maximum(np.abs(y), 1e-3)[None, :] \
            / np.maximum(np.abs(y), 1e-3).max()
        assert np.all(np.abs(J[i] - Jo) <= 1e-10 * (np.abs(Jo) + sc) + 4.0 * np.abs(Ja - Jo)), i


def test_integration(chem, mech):
    gm, om, text, name = mech
    n = 131
    T, p, Y = uniform_cells(text, n, 72)
    a = [_g(v) for v in (T, p, Y)]
    Tw, Yw, stats, st, na, nr = chem.integrate(gm, *a, 1e-8, RTOL, ATOL, form=chem.FORM_PLAIN, return_counts=True)
    To, Yo, nao, nro, sto = om.integrate(T, p, Y, 1e-8, RTOL, ATOL)
    assert stats["failed"] == 0 and np.all(sto == 0)
    assert np.all(np.abs(Tw.cpu().numpy() - To) <= 1e-6 * To) and np.all(np.abs(Yw.cpu().numpy() - Yo) <= 1e-8)
    assert np.sum((na.cpu().numpy() != nao) | (nr.cpu().numpy() != nro)) <= 2
    Tp, Yp, _ = chem.integrate(gm, *a, 1e-8, RTOL, ATOL, form=chem.FORM_PERSISTENT)
    assert torch.equal(Tp, Tw) and torch.equal(Yp, Yw)
    Tn, Yn = a[0].clone(), a[2].clone()
    chem.integrate_noalloc(gm, Tn, a[1], Yn, 1e-8, RTOL, ATOL)
    assert torch.equal(Tn, Tw) and torch.equal(Yn, Yw)
    for k in (1, 7, 64):
        Tk, Yk, _ = chem.integrate(gm, *(v[:k].contiguous() for v in a), 1e-8, RTOL, ATOL, form=chem.FORM_PLAIN)
        assert torch.equal(Tk, Tw[:k]) and torch.equal(Yk, Yw[:k])


def test_fixed_step(chem, mech):
    gm, om, text, name = mech
    T, p, Y = uniform_cells(text, 21, 75)
    # (hot cells of the 13-species reactions are stiffer: as in the other fixed-step
    # tests they take smaller steps, or the oracle's own spread hides the step)
    h = 1e-12 if name == "13" else 1e-11
    yn, en, ok = (v.cpu().numpy() for v in chem.step_fixed(gm, _g(T), _g(p), _g(Y), h, RTOL, ATOL))
    assert np.all(ok == 1)
    skipped = 0
    for i in range(len(T)):
        y0 = np.concatenate([[T[i]], Y[i]])
        eno, espread, yo, _ = errnorm_with_spread(om, p[i], y0, h, RTOL, ATOL)
        yspread = np.zeros(len(y0))
        for f in (1.0 + 2.0**-52, 1.0 - 2.0**-52):
            y1 = y0.copy()
            y1[0] *= f
            yspread = np.maximum(yspread, np.abs(om.step(p[i], y1, h)[0] - yo))
        if yspread[0] > 2.5e-11 * yo[0] or np.any(yspread[1:] > 2.5e-13):    # an ill-conditioned step
            skipped += 1
            continue
        assert abs(yn[i, 0] - yo[0]) <= 1e-10 * yo[0] and np.all(np.abs(yn[i, 1:] - yo[1:]) <= 1e-12), i
        assert abs(en[i] - eno) <= errnorm_bar(eno, espread), (i, en[i], eno)
    assert skipped <= len(T) // 5


def test_adjoint(chem, mech):
    """Gradients against the oracle's, to 1e-5 or four times what a change of T0 by
    one unit in the last place makes of them."""
    gm, om, text, name = mech
    if name == "34by11":
        pytest.skip("the adjoint's scratch of 1,782 reactions does not fit the LDS")
    T, p, Y = uniform_cells(text, 6, 67)
    gT, gY = np.full(len(T), 1e-3), np.zeros(Y.shape)
    gY[:, 2] = 1.0
    out = [v.cpu().numpy() if torch.is_tensor(v) else v
           for v in chem.integrate_adjoint(gm, _g(T), _g(p), _g(Y), 1e-8, RTOL, ATOL, _g(gT), _g(gY))]
    r = chem.integrate(gm, _g(T), _g(p), _g(Y), 1e-8, RTOL, ATOL, return_counts=True)
    assert np.array_equal(out[5], r[0].cpu().numpy()) and np.array_equal(out[6], r[1].cpu().numpy())
    told = chem.integrate_adjoint(gm, _g(T), _g(p), _g(Y), 1e-8, RTOL, ATOL, _g(gT), _g(gY), forward_nacc=r[4])
    assert all(np.array_equal(a, b.cpu().numpy()) for a, b in zip(out[:7], told[:7]))
    ref = om.adjoint(T, p, Y, 1e-8, RTOL, ATOL, gT, gY)
    alt = [om.adjoint(T * f, p, Y, 1e-8, RTOL, ATOL, gT, gY) for f in (1.0 + 2.0**-52, 1.0 - 2.0**-52)]
    for k in range(5):
        scale = np.abs(ref[k]).max(axis=-1, keepdims=True) if k == 1 else np.abs(ref[k]) if k == 0 else np.abs(ref[k]).max()
        spread = np.maximum(*(np.abs(a[k] - ref[k]) for a in alt))
        spread = spread.max(axis=-1, keepdims=True) if k == 1 else spread if k == 0 else spread.max()
        assert np.all(np.abs(out[k] - ref[k]) <= np.maximum(1e-5 * scale, 4 * spread)), k

"""The edges of the rate expressions on the GPU, one cell per lane and
wave-cooperatively, against the oracle."""
import os

import numpy as np
import pytest

import rate_cases as rc

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

FORMS = [("lane", None), ("wave", "0")]


@pytest.fixture(scope="module")
def evaluate(tmp_path_factory, oracle_lib):
    """(text, CHEM_LANE_MAX_SPECIES) -> source terms alone, with the Jacobian, the oracle's both"""
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2508_16105_amd as chem
    wd = tmp_path_factory.mktemp("rates")
    built = {}

    def run(text, lane_max, T, p, Y):
        key = (text, lane_max)
        if key not in built:
            path = wd / f"m{len(built)}.mech"
            path.write_text(text)
            old = os.environ.pop("CHEM_LANE_MAX_SPECIES", None)
            try:
                if lane_max is not None:
                    os.environ["CHEM_LANE_MAX_SPECIES"] = lane_max
                built[key] = chem.Mechanism(str(path)), oracle_lib.Mechanism(str(path))
            finally:
                os.environ.pop("CHEM_LANE_MAX_SPECIES", None)
                if old is not None:
                    os.environ["CHEM_LANE_MAX_SPECIES"] = old
        gm, om = built[key]
        a = [torch.tensor(v, dtype=torch.float64, device="cuda:0") for v in (T, p, Y)]
        f = chem.eval_source(gm, *a, jacobian=False)[0].cpu().numpy()
        fj, J = (v.cpu().numpy() for v in chem.eval_source(gm, *a, jacobian=True))
        return f, fj, J, rc.oracle_source(om, T, p, Y), rc.oracle_jacobian(om, T, p, Y)
    return run


@pytest.mark.parametrize("form,lane_max", FORMS)
@pytest.mark.parametrize("centre", sorted(rc.CENTRE))
def test_a_troe_centre_below_zero_is_not_a_number(evaluate, centre, form, lane_max):
    T, p, Y = rc.states(4, rc.CENTRE_T)
    f, fj, J, fo, _ = evaluate(rc.CENTRE[centre], lane_max, T, p, Y)
    rc.check_source(f, fo)
    rc.check_source(fj, fo)
    assert np.array_equal(np.isnan(J).any(axis=(1, 2)), np.isnan(fo).any(axis=1))


@pytest.mark.parametrize("form,lane_max", FORMS)
@pytest.mark.parametrize("kind", sorted(rc.FAR))
@pytest.mark.parametrize("y", rc.FAR_Y)
def test_a_reverse_rate_whose_equilibrium_constant_is_out_of_range(evaluate, kind, form, lane_max, y):
    """Tolerance: the exponential's argument is a difference of terms up to 837,
    each rounded (2^-53 of it), a few such errors: 1e-12; a forward rate constant
    below the smallest normal double keeps its rounding of 2^-1074, in source terms
    below 1e-290."""
    T, p, Y = rc.states(3, rc.FAR_T, y=y)
    f, fj, J, _, _ = evaluate(rc.FAR[kind], lane_max, T, p, Y)
    ref = rc.far_source(kind, T, p, Y)
    assert np.isfinite(J).all()
    for g in (f, fj):
        assert np.all(np.abs(g - ref) <= 1e-12 * np.abs(ref).max(axis=1, keepdims=True) + 1e-290), (g, ref)


@pytest.mark.parametrize("form,lane_max", FORMS)
@pytest.mark.parametrize("kind", sorted(rc.SMALL))
def test_logarithms_of_subnormal_numbers(evaluate, kind, form, lane_max):
    T, p, Y = rc.states(4, rc.SMALL_T)
    f, fj, J, fo, Jo = evaluate(rc.SMALL[kind], lane_max, T, p, Y)
    rc.check_small(f, fj, J, fo, Jo, T)

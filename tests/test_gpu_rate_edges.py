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
    """(text, CHEM_LANE_MAX_SPECIES) -> source terms alone, with the Jacobian, the oracle's"""
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
        return f, fj, J, rc.oracle_source(om, T, p, Y)
    return run


@pytest.mark.parametrize("form,lane_max", FORMS)
@pytest.mark.parametrize("centre", sorted(rc.CENTRE))
def test_a_troe_centre_below_zero_is_not_a_number(evaluate, centre, form, lane_max):
    T, p, Y = rc.states(4, rc.CENTRE_T)
    f, fj, J, fo = evaluate(rc.CENTRE[centre], lane_max, T, p, Y)
    rc.check_source(f, fo)
    rc.check_source(fj, fo)
    assert np.array_equal(np.isnan(J).any(axis=(1, 2)), np.isnan(fo).any(axis=1))

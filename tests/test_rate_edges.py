"""The edges of the rate expressions on the host: the per-lane device code,
compiled as C++ (see test_hostemu), against the oracle.  No GPU."""
import pathlib

import numpy as np
import pytest

import hostemu_build as hb
import rate_cases as rc

RU = 8.314462618


@pytest.fixture(scope="module")
def lane(tmp_path_factory, oracle_lib):
    """text -> (source terms alone, with the Jacobian, the oracle's both) over given states"""
    if not pathlib.Path(hb.CLANG).exists():
        pytest.skip("host clang++ not available")
    import paper_2508_16105_amd as chem
    wd = tmp_path_factory.mktemp("rates")
    built = {}

    def evaluate(text, T, p, Y):
        if text not in built:
            path = wd / f"m{len(built)}.mech"
            path.write_text(text)
            a, b, e = chem.Mechanism(str(path)).get_params()
            built[text] = (hb.build(str(path), wd, ["-O1"], path.stem), np.concatenate([a, b, e / RU]),
                           oracle_lib.Mechanism(str(path)))
        exe, par, om = built[text]
        f = hb.run(exe, wd, 4, par, T, p, Y, 0.0, 0.0, 0.0)["f"]
        both = hb.run(exe, wd, 2, par, T, p, Y, 0.0, 0.0, 0.0)
        return f, both["f"], both["J"], rc.oracle_source(om, T, p, Y), rc.oracle_jacobian(om, T, p, Y)
    return evaluate


@pytest.mark.parametrize("centre", sorted(rc.CENTRE))
def test_a_troe_centre_below_zero_is_not_a_number(lane, centre):
    T, p, Y = rc.states(4, rc.CENTRE_T)
    f, fj, J, fo, _ = lane(rc.CENTRE[centre], T, p, Y)
    assert np.isnan(fo).any() == (centre == "below")
    rc.check_source(f, fo)
    rc.check_source(fj, fo)
    assert np.array_equal(np.isnan(J).any(axis=(1, 2)), np.isnan(fo).any(axis=1))


@pytest.mark.parametrize("kind", sorted(rc.SMALL))
def test_logarithms_of_subnormal_numbers(lane, kind):
    T, p, Y = rc.states(4, rc.SMALL_T)
    f, fj, J, fo, Jo = lane(rc.SMALL[kind], T, p, Y)
    rc.check_small(f, fj, J, fo, Jo, T)

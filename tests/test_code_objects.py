"""The code objects of the committed mechanisms (compiled by build()): no vector
register is written between a divergent join and the restore of the execution
mask.  No GPU.

The compiler has done so: in an unrolled 13-species step the copies of two mass
fractions stood before the restore at the join of the branch around a falloff
reaction's logarithm, so a lane whose P_r was floored there went on with other
numbers in their place, and a cell that had failed was accepted with them."""
import concurrent.futures
import pathlib

import pytest

import code_objects as co

KCACHE = pathlib.Path(__file__).resolve().parents[1] / "paper_2508_16105_amd" / "kcache"


def test_no_vector_write_before_a_join_restores_the_mask():
    if not pathlib.Path(co.OBJDUMP).exists():
        pytest.skip("llvm-objdump not available")
    objects = sorted(KCACHE.glob("*.co"))
    if not objects:
        pytest.skip("no code objects: build() has not run")

    def scan(path):
        return [(path.name, name, bad) for name, ins in co.functions(path).items()
                if (bad := co.writes_before_rejoining(ins))]
    with concurrent.futures.ThreadPoolExecutor(4) as pool:
        assert not [b for found in pool.map(scan, objects) for b in found]


def test_the_scan_finds_such_a_write():
    """On the instructions of the faulty join, and of one in order."""
    def lines(join):
        code = ["s_and_saveexec_b64 s[4:5], s[0:1]", "s_cbranch_execz 1", "v_add_f64 v[0:1], v[2:3], v[4:5]"] + join
        return [(4 * k, t) for k, t in enumerate(code)]
    copy, back = "v_mov_b64_e32 v[114:115], v[128:129]", "s_or_b64 exec, exec, s[4:5]"
    assert co.writes_before_rejoining(lines([copy, back])) == [("0xc", [copy])]
    assert co.writes_before_rejoining(lines([back, copy])) == []

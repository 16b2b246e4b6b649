"""Build the chemistry library in-tree.

1. Embed csrc/device/*.hip into the host library as strings (the device
   code is compiled per mechanism, with the generated mechanism-specific
   code in front of it, by hipRTC for gfx950).
2. Compile the host library libchemmi.so with hipcc (HIP runtime + hipRTC).
3. Load each mechanism under workloads/mech so its gfx950 code object is
   compiled now and stored in the kernel cache beside the library.
"""
from __future__ import annotations

import os
import pathlib
import subprocess
import sys

PKG = pathlib.Path(__file__).resolve().parent
CSRC = PKG / "csrc"
LIB = PKG / "libchemmi.so"
ROOT = PKG.parent
# (mechanism, CHEM_LANE_MAX_SPECIES at load): the default builds and the
# wave-cooperative builds of the 9- and 13-species mechanisms
PREBUILT = [("m9", None), ("m13", None), ("m32", None), ("m9", "0"), ("m13", "0"),
            ("m13x", None), ("m13x", "0"), ("m32x", None), ("m16", None)]
# CHEMKIN renderings the tests load (written into the build folder first)
PREBUILT_CHEMKIN = ["m9", "m32x"]
# OpenFOAM renderings the tests load
PREBUILT_OPENFOAM = ["m9", "m32s"]
HOST_SOURCES = ["capi.cpp", "runtime.cpp", "module.cpp", "mechanism.cpp", "chemkin.cpp", "foam.cpp", "codegen.cpp",
                "noalloc.hip"]


def embed_device_source():
    delim = "CHEMDEV"
    out = "// generated from device/*.hip by build.py; do not edit\n"
    for var, name in (("kMathSource", "math.hip"), ("kCommonSource", "common.hip"),
                      ("kIntegratorSource", "integrator.hip"), ("kWideSource", "wide.hip"),
                      ("kWideAdjointSource", "wide_adjoint.hip"),
                      ("kWideRowsSource", "wide_rows.hip"),
                      ("kEulerSource", "euler.hip")):
        src = (CSRC / "device" / name).read_text()
        assert f"){delim}\"" not in src
        out += f"static const char {var}[] = R\"{delim}(\n{src}){delim}\";\n"
    target = CSRC / "_device_source.inc"
    if not target.exists() or target.read_text() != out:
        target.write_text(out)


def compile_host(verbose=False):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = LIB.with_suffix(".so.tmp")
    cmd = [hipcc, "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wno-unused-result",
           "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           *[str(CSRC / s) for s in HOST_SOURCES], "-o", str(tmp), "-lhiprtc", "-ldl"]
    if verbose:
        print(" ".join(cmd))
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)


def _prebuild(kind, nm, lane_max=None):
    """Compile the device code of one mechanism into the cache."""
    # torch brings its own hipRTC; loaded first it is the compiler a program
    # that imports torch gets, and the cache key names the compiler
    import torch  # noqa: F401
    import tempfile
    sys.path.insert(0, str(ROOT))
    from paper_2508_16105_amd import _lib
    from workloads import gen_mech, resized
    os.environ.pop("CHEM_LANE_MAX_SPECIES", None)
    if lane_max is not None:
        os.environ["CHEM_LANE_MAX_SPECIES"] = lane_max
    golden = ROOT / "tests" / "golden"
    with tempfile.TemporaryDirectory() as td:
        td = pathlib.Path(td)
        if kind == "mech":
            _lib.load_mechanism_handle(str(ROOT / "workloads" / "mech" / f"{nm}.mech"))
        elif kind == "resized":
            p = td / f"{nm}.mech"
            p.write_text(resized.CASES[nm]())
            _lib.load_mechanism_handle(str(p))
        elif kind == "chemkin":
            p = td / f"{nm}.inp"
            p.write_text(gen_mech.to_chemkin(gen_mech.build_mechanism(nm)))
            _lib.load_mechanism_handle(str(p))
        elif kind == "openfoam":
            r, t = gen_mech.to_openfoam(gen_mech.build_mechanism(nm))
            rp, tp = td / f"{nm}.foam", td / "thermo"
            rp.write_text(r)
            tp.write_text(t)
            _lib.load_mechanism_handle(str(rp), str(tp), "openfoam")
        elif kind == "golden":
            if nm == "foam_small":
                _lib.load_mechanism_handle(str(golden / nm / "reactions"), str(golden / nm / "thermo"), "openfoam")
            else:
                _lib.load_mechanism_handle(str(golden / f"{nm}.inp"))


def prebuild_mechanisms(builds=None):
    """Compile the device code of the committed mechanisms into the cache, a few
    at a time in processes of their own."""
    import concurrent.futures
    sys.path.insert(0, str(ROOT))
    from workloads import resized
    jobs = [("mech", *b) for b in builds or PREBUILT]
    if builds is None:
        # (the ones that take longest first)
        jobs = [("resized", nm) for nm in resized.CASES] + jobs
        jobs += [("chemkin", nm) for nm in PREBUILT_CHEMKIN]
        jobs += [("openfoam", nm) for nm in PREBUILT_OPENFOAM]
        jobs += [("golden", nm) for nm in ("ck_small", "foam_small")]

    def run(job):
        subprocess.run([sys.executable, str(pathlib.Path(__file__).resolve()), *(a for a in job if a is not None)],
                       check=True)
    with concurrent.futures.ThreadPoolExecutor(min(4, len(os.sched_getaffinity(0)))) as pool:
        list(pool.map(run, jobs))


def prune_cache(since):
    """Drop cached code objects neither produced nor used since `since`."""
    for f in (PKG / "kcache").glob("*.co"):
        if f.stat().st_mtime < since:
            f.unlink()


def build(verbose=False, mechanisms=True):
    import time
    t0 = time.time() - 1.0
    embed_device_source()
    compile_host(verbose)
    if mechanisms:
        prebuild_mechanisms()
        prune_cache(t0)


if __name__ == "__main__":
    if sys.argv[1:]:
        _prebuild(*sys.argv[1:])
    else:
        build(verbose=True)

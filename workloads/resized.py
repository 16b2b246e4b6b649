"""Mechanisms of other sizes made from the 32-species one (or another): fewer
species (the first of the list, and the reactions among them), or more (copies of
reacting species, with some of the reactions of the species each is a copy of)."""
import re

from workloads import mech_text


def split(text, k):
    """The mechanism with every reaction k times over at a k-th of its rate (both
    limits of a falloff reaction): the same production rates from k times the
    reactions."""
    out = []
    for ln in text.splitlines():
        if ln.startswith("name "):
            ln += f"by{k}"
        if not ln.startswith("reaction "):
            out.append(ln)
            continue
        w = ln.split()
        if w[1] == "plog":
            raise ValueError("pressure-tabulated reactions are not split")
        w[4] = repr(float(w[4]) / k)
        if w[1] in ("troe", "lindemann", "sri"):
            w[7] = repr(float(w[7]) / k)
        out += [" ".join(w)] * k
    return "\n".join(out) + "\n"


def _sides(line):
    w = line.split()
    side = lambda s: [tuple(t.split("=")) for t in s.split(",")]
    return w, side(w[2]), side(w[3])


def resized(ns, per_copy=6, inert=True, base="m32", first=None):
    """The text of an ns-species mechanism, named after its size; without `inert`
    every species reacts.  first: species kept of the base's (default ns)."""
    lines = [ln for ln in mech_text(base).splitlines() if ln.strip() and not ln.startswith("#")]
    species = [ln.split()[1] for ln in lines if ln.startswith("species ")]
    comp = {ln.split()[1]: ln for ln in lines if ln.startswith("species ")}
    thermo = {ln.split()[1]: ln for ln in lines if ln.startswith("thermo ")}
    reactions = [ln for ln in lines if ln.startswith("reaction ")]
    if not inert:
        used = {s for ln in reactions for side in _sides(ln)[1:] for s, _ in side}
        species = [s for s in species if s in used]
    keep = species[:first or ns]
    rx = []
    for ln in reactions:
        _, a, b = _sides(ln)
        if all(s in keep for s, _ in a + b):
            m = re.search(r" eff=(\S+)", ln)
            if m:
                eff = [e for e in m.group(1).split(",") if e.split(":")[0] in keep]
                ln = ln.replace(m.group(0), " eff=" + ",".join(eff) if eff else "")
            rx.append(ln)
    reacting = [s for s in keep if any(s in dict(_sides(ln)[1] + _sides(ln)[2]) for ln in rx)]
    out_comp, out_thermo, k = [comp[s] for s in keep], [thermo[s] for s in keep], 0
    while len(out_comp) < ns:
        s = reacting[k % len(reacting)]
        copy = f"{s}_{k // len(reacting) + 1}"
        out_comp.append(comp[s].replace(f"species {s} ", f"species {copy} ", 1))
        out_thermo.append(thermo[s].replace(f"thermo {s} ", f"thermo {copy} ", 1))
        mine = [ln for ln in rx if (s, "1") in _sides(ln)[1] + _sides(ln)[2]][:per_copy]
        for ln in mine:
            w, a, b = _sides(ln)
            side = lambda q: ",".join(f"{copy if (n, c) == (s, '1') else n}={c}" for n, c in q)
            w[2], w[3] = side(a), side(b)
            rx.append(" ".join(w))
        k += 1
    head = [ln for ln in lines if ln.startswith(("chemmi-mech", "element"))]
    return "\n".join([head[0], f"name {base}to{ns}" + ("" if inert else "r")] + head[1:] + out_comp + out_thermo + rx + ["end"]) + "\n"


# The sizes at which the kernels change: the most unknowns of the lane form whose
# factors stay in registers (11); the fewest and the most unknowns at three matrix
# rows a lane of the wave-cooperative form; above them, and where the tables of a
# mechanism do not fit the LDS in that form, its row-per-lane form.
CASES = {"13": lambda: resized(13, 4, base="m13", first=11),
         "34": lambda: resized(34), "48": lambda: resized(48), "48r": lambda: resized(48, 5, inert=False),
         "34by11": lambda: split(resized(34), 11)}

"""Reading the code objects the library built: what a divergent join does first.

A lane that skips a block re-joins the others where the execution mask is
restored.  Vector instructions between the label the skipping branch jumps to
and that restore are executed for the lanes of the block alone, so a register
copy the compiler puts there is missing in the lanes that skipped it."""
import re
import subprocess

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
_INS = re.compile(r"^\s+(\S.*?)\s*// ([0-9A-F]+): ([0-9A-F ]+)")
_WRITES = ("v_", "scratch_load", "global_load", "flat_load", "buffer_load", "ds_read", "ds_load", "ds_bpermute")
_SCALAR = ("v_readlane", "v_writelane", "v_readfirstlane", "v_cmp")


def functions(path):
    """name -> [(address, text)] of the object's functions"""
    out, ins = {}, None
    txt = subprocess.run([OBJDUMP, "-d", str(path)], check=True, capture_output=True, text=True).stdout
    for line in txt.splitlines():
        m = re.match(r"^[0-9a-f]+ <(.+)>:", line)
        if m:
            ins = out.setdefault(m.group(1), [])
            continue
        m = _INS.match(line)
        if m and ins is not None:
            ins.append((int(m.group(2), 16), m.group(1)))
    return out


def _joins(ins):
    """label -> the mask registers saved by the branches that jump to it when no
    lane is left (directly, or around it over a long jump)"""
    out = {}
    for i, (a, t) in enumerate(ins):
        m = re.match(r"s_cbranch_exec(z|nz) (\d+)", t)
        if not m:
            continue
        saved = None
        for _, u in reversed(ins[max(0, i - 40):i]):
            mm = re.match(r"s_and_saveexec_b64 (s\[\d+:\d+\])", u) or re.match(r"s_mov_b64 (s\[\d+:\d+\]), exec", u)
            if mm:
                saved = mm.group(1)
                break
            if u.startswith(("s_cbranch", "s_branch")):
                break
        if m.group(1) == "z":
            k = int(m.group(2))
            out.setdefault(a + 4 + 4 * (k - 65536 if k >= 32768 else k), set()).add(saved)
            continue
        for j in range(i + 1, min(i + 8, len(ins) - 2)):
            if ins[j][1].startswith("s_getpc_b64"):
                lo = re.match(r"s_add_u32 s\d+, s\d+, (\S+)", ins[j + 1][1])
                hi = re.match(r"s_addc_u32 s\d+, s\d+, (\S+)", ins[j + 2][1])
                if lo and hi:
                    d = int(lo.group(1), 0) & 0xffffffff | (int(hi.group(1), 0) & 0xffffffff) << 32
                    out.setdefault((ins[j + 1][0] + d) & (1 << 64) - 1, set()).add(saved)
                break
    return out


def writes_before_rejoining(ins):
    """The joins of a function at which vector registers are written before the
    mask is restored: [(address, [instructions])]."""
    at = {a: i for i, (a, _) in enumerate(ins)}
    bad = []
    for label, saved in sorted(_joins(ins).items()):
        if label not in at:
            continue
        found, reloaded = [], set()
        for _, t in ins[at[label]:]:
            op = t.split()[0]
            if op.startswith(("s_branch", "s_cbranch", "s_setpc", "s_endpgm")) or "saveexec" in op:
                break
            m = re.match(r"s_or_b64 exec, exec, (s\[(\d+):\d+\])", t)
            if m:
                # (the join of this very branch: its own mask, or one from a spill lane)
                if found and (m.group(1) in saved or m.group(2) in reloaded):
                    bad.append((hex(label), found))
                break
            if re.match(r"s_\w+ exec", t):
                break
            m = re.match(r"v_readlane_b32 s(\d+)", t)
            if m:
                reloaded.add(m.group(1))
            if op.startswith(_WRITES) and not op.startswith(_SCALAR):
                found.append(t)
    return bad

"""Distances between instructions that the hardware asks for and the compiler keeps for its own instructions only,
checked in the assembly of this library's kernels where they hold loads written by hand."""
import os
import re
import subprocess

import pytest

import paper_2604_07874_amd.build as B   # not a `from` import, which would load the library (before torch has loaded its HIP runtime)

VMEM = re.compile(r"(global|buffer|flat|scratch)_\w+$")
INSTR = re.compile(r"^\s+([a-z][a-z0-9_]+)(?:\s+(.*?))?\s*(?:;.*)?$")
SGPRS = re.compile(r"\bs(?:(\d+)\b|\[(\d+):(\d+)\])")
NEEDED = 5   # wait states between a vector instruction's write of a scalar register and a memory instruction's read of it


def sgprs(text):
    out = set()
    for one, lo, hi in SGPRS.findall(text):
        out.update([int(one)] if one else range(int(lo), int(hi) + 1))
    if re.search(r"\bvcc\b", text):
        out.add("vcc")
    return out


def parse(asm):
    """Instructions of every function in order, as (line, name, operands), and where each label stands."""
    code, labels = [], {}
    for n, line in enumerate(asm.splitlines(), 1):
        text = line.split(";")[0].rstrip()
        m = re.match(r"^([.\w$]+):$", text)
        if m:
            labels[m.group(1)] = len(code)
            continue
        m = INSTR.match(text)
        if m and not m.group(1).startswith("."):
            code.append((n, m.group(1), m.group(2) or ""))
    return code, labels


def too_close(asm):
    """Every memory instruction that reads a scalar register fewer than NEEDED wait states behind a vector instruction
    that wrote it, over all ways that lead there, and every global->LDS load right behind a write of m0."""
    code, labels = parse(asm)
    into = {}
    for i, (_, name, ops) in enumerate(code):
        if name.startswith(("s_branch", "s_cbranch")) and ops in labels:
            into.setdefault(labels[ops], []).append(i)

    def before(i):
        if i > 0 and code[i - 1][1] not in ("s_branch", "s_endpgm", "s_setpc_b64"):
            yield i - 1
        yield from into.get(i, [])

    found = []
    for i, (line, name, ops) in enumerate(code):
        if not VMEM.match(name):
            continue
        lds = "_lds_" in name
        reads = sgprs(ops)
        work = [(j, 0, frozenset(reads), lds) for j in before(i)]
        seen = set()
        while work:
            j, states, wanted, m0 = work.pop()
            if (j, states, wanted, m0) in seen:
                continue
            seen.add((j, states, wanted, m0))
            jline, jname, jops = code[j]
            dest, _, rest = jops.partition(",")
            two = sgprs(rest.partition(",")[0]) if jname.startswith(("v_add_co", "v_sub_co", "v_addc_co", "v_subb_co", "v_div_scale", "v_mad_u64", "v_mad_i64")) else set()
            writes = sgprs(dest) | two if jname.startswith("v_") else set()
            if m0 and states < 1 and jname.startswith("s_") and dest.strip() == "m0":
                found.append((line, name, jline, jname, states))
            if writes & wanted:
                found.append((line, name, jline, jname, states))
                continue
            if jname.startswith("s_"):
                wanted = wanted - sgprs(dest)     # a scalar write stands between
            states += int(jops.split()[0], 0) + 1 if jname == "s_nop" else 1
            if states < NEEDED and (wanted or m0):
                work.extend((k, states, wanted, m0) for k in before(j))
    return found


@pytest.mark.parametrize("gap,bad", [("s_nop 4", False), ("s_nop 3", True), ("s_mov_b32 m0, s5\n\ts_nop 0", True), ("", True),
                                     ("s_mov_b64 s[10:11], s[2:3]", False), ("s_cbranch_scc1 .LB0\n\ts_nop 4\n.LB0:", True)])
def test_the_check_itself(gap, bad):
    asm = f"f:\n\tv_readlane_b32 s11, v2, 0\n\t{gap}\n\tglobal_load_lds_dwordx4 v1, s[10:11]\n\ts_endpgm\n"
    assert bool(too_close(asm)) == bad
    assert too_close("f:\n\ts_mov_b32 m0, s3\n\tglobal_load_lds_dwordx4 v1, s[10:11]\n")


@pytest.mark.parametrize("source", ["prefill.hip", "attn.hip", "reclaim.hip", "pool.hip"])
def test_scalar_bases_of_memory_instructions_are_settled(source, tmp_path):
    """A memory instruction needs five wait states behind a vector instruction that wrote its scalar base (v_readlane of
    a block address ahead of a global->LDS load, for one); fewer leave its address undefined."""
    out = str(tmp_path / "code.s")
    cmd = [B.hipcc_path(), "--offload-arch=gfx950", "--offload-device-only", "-S", "-O3", "-std=c++17",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-I", os.path.join(B.ROOT, "include"), "-I", B.CSRC,
           os.path.join(B.CSRC, source), "-o", out]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    asm = open(out).read()
    loads = [n for _, n, _ in parse(asm)[0] if VMEM.match(n)]
    assert loads
    if source == "prefill.hip":
        assert sum("load_lds_dwordx4" in n for n in loads) >= 16
    bad = too_close(asm)
    assert not bad, "\n".join(f"line {l}: {n} {s} wait states behind line {jl}: {jn}" for l, n, jl, jn, s in bad)

"""count_i8_stream_kernel brings R's values by loads that only its own wait counts cover: the compiler takes their registers as
written when the load is issued, three stages before the data is there.  A copy or a spill of one that it put in between would read what
the register held before.  So the assembly of this file's own build is walked from every such load: on every way from it the first
instruction that names its register is the addition to the accumulators, behind a wait that covers the load (CPU only)."""
import os
import re
import subprocess

from paper_2305_08872_amd import build as hip_build

VMEM = re.compile(r"(global|buffer|flat|scratch)_(load|store|atomic)")
R_LOAD = re.compile(r"global_load_dword (v\d+),")


def instructions(kernel):
    """(text, targets) of a kernel's instructions, where control may go from each; numeric labels are the asm's own."""
    out, named, numeric = [], {}, {}
    for line in kernel.splitlines():
        line = line.split(";")[0].strip()
        while True:
            m = re.match(r"(\.?\w+):\s*", line)
            if not m:
                break
            (numeric if m.group(1).isdigit() else named).setdefault(m.group(1), []).append(len(out))
            line = line[m.end():]
        if line and not line.startswith("."):
            out.append(line)
    def where(at, label):
        m = re.fullmatch(r"(\d+)([fb])", label)
        if not m:
            return named[label][0]
        places = numeric[m.group(1)]
        return min(p for p in places if p > at) if m.group(2) == "f" else max(p for p in places if p <= at)
    for at, text in enumerate(out):
        op = text.split()[0]
        if op == "s_endpgm":
            yield text, []
        elif op == "s_branch":
            yield text, [where(at, text.split()[1])]
        elif op.startswith("s_cbranch"):
            yield text, [at + 1, where(at, text.split()[1])]
        else:
            assert not op.startswith(("s_setpc", "s_swappc", "s_call")), text
            yield text, [at + 1]


def constants(code):
    """Scalar registers that hold one number throughout: every instruction that may write one moves that number there."""
    value, other = {}, set()
    for text, _ in code:
        op, _, rest = text.partition(" ")
        if op.startswith(("s_cmp", "s_cbranch", "s_branch", "s_waitcnt", "s_nop", "s_barrier", "s_endpgm", "s_bitcmp", "s_sleep", "s_setprio")):
            continue
        dest = rest.split(",")[0].strip()
        m = re.fullmatch(r"s_mov_b32 s(\d+), (\d+)", text)
        if m:
            value.setdefault(int(m.group(1)), set()).add(int(m.group(2)))
            continue
        m = re.fullmatch(r"s\[(\d+):(\d+)\]", dest) or re.fullmatch(r"s(\d+)", dest)
        if m:
            other.update(range(int(m.group(1)), int(m.group(m.lastindex)) + 1))
    return {r: v.copy().pop() for r, v in value.items() if len(v) == 1 and r not in other}


def names(text, register):
    n = int(register[1:])
    return any(int(a) <= n <= int(b or a) for a, b in re.findall(r"\bv(?:\[)?(\d+)(?::(\d+)\])?", text))


def faults(kernel):
    """What is wrong with the R loads of a kernel's assembly, and how many there are."""
    code = list(instructions(kernel))
    fixed = constants(code)
    found, loads = [], 0
    for at, (text, _) in enumerate(code):
        m = R_LOAD.match(text)
        if not m:
            continue
        loads += 1
        register = m.group(1)
        todo, seen = [(at + 1, 0, False)], set()     # (place, memory operations behind the load, it has been waited for)
        while todo:
            state = todo.pop()
            if state in seen:
                continue
            seen.add(state)
            place, behind, there = state
            text, after = code[place]
            if names(text, register):
                dest, *sources = text.partition(" ")[2].split(",")
                if not there or not text.startswith("v_add_u32") or not any(names(s, register) for s in sources) or names(dest, register):
                    found.append("%s of %r: %s%s" % (register, code[at][0], text, "" if there else " (not waited for)"))
                continue
            if not after:
                found.append("%s of %r: not read" % (register, code[at][0]))
                continue
            if VMEM.match(text):
                behind = min(behind + 1, 64)
            waited = re.match(r"s_waitcnt\b.*vmcnt\((\d+)\)", text)
            there = there or bool(waited and int(waited.group(1)) <= behind)
            m = re.fullmatch(r"s_cmp_eq_u32 s(\d+), 0", text)
            if m and fixed.get(int(m.group(1)), 0) != 0 and code[place + 1][0].startswith("s_cbranch_scc"):
                # (never equal: scc0)
                text, after = code[place + 1]
                after = after[1:] if "scc0" in text else after[:1]
            todo += [(p, behind, there) for p in after]
    return found, loads


def test_the_walk_sees_a_register_touched_too_early():
    good = """
        s_mov_b32 s9, 1
        global_load_dword v5, v1, s[2:3] nt
        s_cmp_eq_u32 s9, 0
        s_cbranch_scc1 1f
        global_load_lds_dwordx4 v7, s[4:5]
        global_load_lds_dwordx4 v7, s[4:5]
    1:
        s_cbranch_vccz .LBB0_2
        v_mov_b32 v[10:11], 0
    .LBB0_2:
        s_waitcnt vmcnt(2)
        v_add_u32_e32 v6, v6, v5
        s_endpgm"""
    assert faults(good) == ([], 1)
    for old, new in [("v_mov_b32 v[10:11], 0", "v_mov_b32 v10, v5"), ("v_mov_b32 v[10:11], 0", "scratch_store_dword off, v5, s1"), ("v_mov_b32 v[10:11], 0", "v_mov_b32 v[4:5], 0"),
                     ("vmcnt(2)", "vmcnt(3)"), ("s_mov_b32 s9, 1", "s_mov_b32 s9, s8"), ("v6, v6, v5", "v5, v6, v5"), ("v_add_u32_e32 v6, v6, v5", "s_nop 0")]:
        assert old in good and faults(good.replace(old, new))[0], new


def test_r_values_are_read_first_by_the_addition_that_waits_for_them(tmp_path):
    asm = os.path.join(str(tmp_path), "stream.s")
    subprocess.run([hip_build._hipcc()] + hip_build.HIPCC_FLAGS + ["--offload-device-only", "-S", os.path.join(hip_build.CSRC, "count_i8_stream.hip"), "-o", asm],
                   check=True, stderr=subprocess.DEVNULL)
    with open(asm) as f:
        text = f.read()
    kernels = re.findall(r"^(_ZN6amulet22count_i8_stream_kernel\w+):(.*?)^\.Lfunc_end", text, re.S | re.M)
    assert len(kernels) == 4
    for name, body in kernels:
        assert faults(body) == ([], 64), name        # (each lane's 64 counts)

"""Host analysis (no GPU) of the compiled rotary statistics kernels: registers that inline-assembly loads are still
filling are left alone until a wait has covered them.

The compiler takes the output of an inline load as written at once. It may copy such a register, or use it for
something else once its value is no longer read, while the data are on their way. The check follows every path through
the assembly with, for each register of a load in flight, the least number of vector memory instructions issued since;
`s_waitcnt vmcnt(n)` completes those with at least n."""
import os
import re
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
VECTOR_MEMORY = re.compile(r"^(global_|buffer_|flat_|scratch_)")


def _regs(text):
    out = set()
    for a, b, c in re.findall(r"\bv\[(\d+):(\d+)\]|\bv(\d+)\b", text):
        out |= {int(c)} if c else set(range(int(a), int(b) + 1))
    return out


def touched_in_flight(body):
    """(number of inline loads, instructions that touch a register in flight) of one kernel's assembly."""
    ins, labels, inline = [], {}, False
    for line in body.split("\n"):
        if "#ASMSTART" in line or "#ASMEND" in line:
            inline = "#ASMSTART" in line
            continue
        s = line.split(";")[0].strip()
        label = re.match(r"^(\.LBB\S+):", s)
        if label:
            labels[label.group(1)] = len(ins)
        elif s and not s.startswith(".") and not s.endswith(":"):
            ins.append((s, inline))
    loads, state, work, bad = 0, {0: {}}, [0], set()
    parsed = []
    for s, inline in ins:
        ops = s.split(None, 1)[1] if " " in s else ""
        wait = re.search(r"vmcnt\((\d+)\)", s) if s.startswith("s_waitcnt") else None
        load = inline and s.startswith("global_load_dwordx4")
        loads += load
        parsed.append((s, load, ops, int(wait.group(1)) if wait else None))
    while work:
        i = work.pop()
        if i >= len(parsed):
            continue
        s, load, ops, wait = parsed[i]
        flight = state[i]
        out = flight
        if wait is not None:
            out = {r: k for r, k in flight.items() if k < wait}
        elif load:
            dst, src = ops.split(",", 1)
            if _regs(src) & flight.keys():
                bad.add((i, s))
            out = {r: k + 1 for r, k in flight.items()}
            out.update({r: 0 for r in _regs(dst)})
        elif not s.startswith("s_"):
            if flight and _regs(ops) & flight.keys():
                bad.add((i, s))
            if VECTOR_MEMORY.match(s):
                out = {r: k + 1 for r, k in flight.items()}
        branch = re.match(r"^s_(c?branch\S*)\s+(\.LBB\S+)", s)
        if branch:
            nxt = [labels[branch.group(2)]] + ([i + 1] if branch.group(1).startswith("cbranch") else [])
        else:
            nxt = [] if s.startswith("s_endpgm") else [i + 1]
        for t in nxt:
            old = state.get(t)
            if old is None:
                state[t] = dict(out)
                work.append(t)
            else:
                less = {r: k for r, k in out.items() if r not in old or k < old[r]}
                if less:
                    old.update(less)
                    work.append(t)
    return loads, sorted(bad)


def test_analysis_sees_copies_and_reuse():
    asm = "\n".join(["\t;;#ASMSTART", "\tglobal_load_dwordx4 v[2:5], v[8:9], off", "\t;;#ASMEND", "\t%s",
                     "\tglobal_store_dword v[10:11], v12, off", "\ts_waitcnt vmcnt(%d)", "\tv_mul_f32_e32 v2, v3, v4",
                     "\ts_endpgm"])
    assert touched_in_flight(asm % ("v_mov_b32_e32 v20, v21", 1)) == (1, [])
    for other, wait in (("v_mov_b64_e32 v[20:21], v[4:5]", 1), ("v_lshlrev_b32_e32 v2, 2, v20", 1),
                        ("v_mov_b32_e32 v20, v21", 2)):
        assert len(touched_in_flight(asm % (other, wait))[1]) == 1


def test_rotary_statistics_leave_registers_in_flight_alone(tmp_path):
    sys.path.insert(0, os.path.join(ROOT, "paper_2609_00891_amd"))
    try:
        import build as lib_build
    finally:
        sys.path.pop(0)
    out = str(tmp_path / "rope.s")
    subprocess.run([lib_build._hipcc()] + lib_build.COMMON + ["-x", "hip", "-S", "--cuda-device-only",
                   os.path.join(lib_build.CSRC, "cb_stats_rope.hip"), "-o", out], check=True, capture_output=True)
    kernels = re.findall(r"(?ms)^(_ZN\S*stats_kernel\S*):.*?\n(.*?)^\.Lfunc_end", open(out).read())
    assert len(kernels) == 8
    for name, body in kernels:
        loads, bad = touched_in_flight(body)
        assert loads > 0 and not bad, (name, bad[:5])

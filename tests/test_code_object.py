"""Wait states that the hardware does not enforce, and registers that occupancy rests on, checked on the library's own
gfx950 code.

A VALU write of a scalar register needs 5 wait states before a vector-memory instruction reads that register. The
compiler inserts them between instructions it knows; it does not look into inline assembly, so the copies written
there have to hold the rule by themselves, whatever stands in front of them (a readfirstlane, a restored spill).
"""
import os
import re
import shutil
import subprocess

import pytest

WAIT = 5
OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")
_INSN = re.compile(r"^\s+(\S+)\s*(.*?)\s*//\s*([0-9A-F]+):")
_FUNC = re.compile(r"^([0-9a-f]+) <(.+)>:")
_TARGET = re.compile(r"<.+\+0x([0-9a-f]+)>\s*$")
_SREG = re.compile(r"\bs(?:(\d+)\b|\[(\d+):(\d+)\])|\b(vcc)\b")


def _sregs(text):
    out = set()
    for one, lo, hi, vcc in _SREG.findall(text):
        out |= {int(one)} if one else {106, 107} if vcc else set(range(int(lo), int(hi) + 1))
    return out


def _valu_sgpr_writes(op, args):
    """Scalar registers that a VALU instruction writes."""
    parts = re.split(r",\s*(?![^\[]*\])", args)
    if op.startswith(("v_readfirstlane", "v_readlane", "v_cmp")):
        return _sregs(parts[0])
    if "_co_" in op or op.startswith(("v_div_scale", "v_mad_u64", "v_mad_i64")):
        return _sregs(parts[1]) if len(parts) > 1 else set()
    return set()


def hazards(listing):
    """(function, address, registers) of every vector-memory read of a scalar register that a VALU instruction wrote
    less than WAIT wait states before, along any path of a function's branches."""
    found, funcs = [], []
    for line in listing.splitlines():
        m = _FUNC.match(line)
        if m:
            funcs.append((m[2], int(m[1], 16), []))
            continue
        m = _INSN.match(line)
        if m and funcs:
            t = _TARGET.search(line) if m[1].startswith(("s_cbranch", "s_branch")) else None
            target = funcs[-1][1] + int(t[1], 16) if t else funcs[-1][1] if m[1].startswith("s_cbranch") else None
            funcs[-1][2].append((int(m[3], 16), m[1], m[2], target))
    for name, _, code in funcs:
        at = {a: i for i, (a, *_) in enumerate(code)}
        pred = [[i - 1] if i and code[i - 1][1] not in ("s_branch", "s_endpgm", "s_setpc_b64") else []
                for i in range(len(code))]
        for i, (_, op, _, target) in enumerate(code):
            if target in at:
                pred[at[target]].append(i)
        for i, (addr, op, args, _) in enumerate(code):
            if not op.startswith(("global_", "buffer_", "flat_", "scratch_")):
                continue
            regs = _sregs(args)
            todo, seen = [(p, 0, frozenset(regs)) for p in pred[i]] if regs else [], set()
            while todo:
                j, dist, live = todo.pop()
                if dist >= WAIT or not live or (j, dist, live) in seen:
                    continue
                seen.add((j, dist, live))
                _, o, a, _ = code[j]
                if o.startswith("v_") and _valu_sgpr_writes(o, a) & live:
                    found.append((name, addr, sorted(_valu_sgpr_writes(o, a) & live)))
                    break
                if o.startswith("s_") and not o.startswith(("s_cmp", "s_bitcmp", "s_waitcnt", "s_nop", "s_barrier",
                                                            "s_cbranch", "s_branch")):
                    live = live - _sregs(a.split(",")[0] if "[" not in a.split(",")[0] else a[:a.index("]") + 1])
                step = int(a.split()[0], 0) + 1 if o == "s_nop" else 1
                todo += [(p, dist + step, live) for p in pred[j]]
    return found


def _listing(tmp_path, lib, tool=OBJDUMP, option="-d"):
    if not os.path.exists(OBJDUMP):
        pytest.skip("llvm-objdump is not installed")
    copy = shutil.copy(lib, tmp_path / "lib.so")              # the code objects are extracted beside it
    subprocess.run([OBJDUMP, "--offloading", copy], check=True, capture_output=True)
    objs = sorted(p for p in os.listdir(tmp_path) if p.endswith("gfx950"))
    assert objs, "no gfx950 code object in the library"
    return [subprocess.run([tool, option, str(tmp_path / o)], check=True, capture_output=True, text=True).stdout
            for o in objs]


def test_the_scan_finds_short_waits():
    head = "0000000000000100 <f>:\n"
    load = "\tglobal_load_lds_dwordx4 v1, s[4:5] // 000000000130: 0\n"
    write = "\tv_readfirstlane_b32 s5, v3 // 000000000100: 0\n"
    assert hazards(head + write + "\ts_mov_b32 m0, s9 // 000000000104: 0\n\ts_nop 0 // 000000000108: 0\n" + load)
    assert not hazards(head + write + "\ts_mov_b32 m0, s9 // 000000000104: 0\n\ts_nop 3 // 000000000108: 0\n" + load)
    # a scalar write in between, and a base that comes round a loop
    assert not hazards(head + write + "\ts_mov_b64 s[4:5], s[8:9] // 000000000104: 0\n" + load)
    assert hazards(head + load.replace("130", "100") + write.replace("100:", "104:") +
                   "\ts_cbranch_scc1 65533 // 000000000108: 0 <f+0x0>\n")


def test_vector_memory_waits_for_scalar_registers_written_by_valu(tmp_path):
    import paper_2607_20467_amd as dcl
    loads, bad = 0, []
    for text in _listing(tmp_path, dcl.library_path()):
        loads += text.count("global_load_lds_dwordx4")
        bad += hazards(text)
    assert loads > 1000, "the library's direct-to-LDS copies were not found"
    assert not bad, f"{len(bad)} reads with fewer than {WAIT} wait states, first: {bad[:3]}"


def test_tail_gemms_leave_room_for_two_workgroups(tmp_path):
    """Two workgroups of eight waves on a CU take at most 128 vector registers per wave. The LM head's tail kernel needs
    more and runs one."""
    import paper_2607_20467_amd as dcl
    regs = {}
    for text in _listing(tmp_path, dcl.library_path(), os.path.join(os.path.dirname(OBJDUMP), "llvm-readobj"), "--notes"):
        for name, n in re.findall(r"\.name: +(_Z\S+)(?:(?!\.name:).)*?\.vgpr_count: +(\d+)", text, re.S):
            regs[name] = int(n)
    tail = {k: v for k, v in regs.items() if re.search(r"gemm_kernel.*Lb1E", k) and "EpiLm" not in k}
    assert len(tail) >= 5 and max(tail.values()) <= 128, tail

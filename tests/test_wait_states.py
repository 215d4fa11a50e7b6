"""gfx950 leaves some register hazards to software: an instruction that reads what one just in front of it wrote needs wait states
between them.  The compiler puts them in for its own instructions and cannot look inside assembly statements, so the built library is read
back here, whole, and every such pair counted."""
import collections
import concurrent.futures
import functools
import os
import re
import shutil
import subprocess

import pytest

from paper_1708_04801_amd import build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
REG = re.compile(r"\b([sv])(\d+)\b|\b([sv])\[(\d+):(\d+)\]|\b(vcc|m0)")
CARRY_OUT = re.compile(r"v_(add|sub|subrev)_co_u32|v_addc_co|v_subb(rev)?_co|v_mad_[ui]64|v_div_scale")
TRANS = re.compile(r"v_(rcp|rsq|exp|log|sqrt|sin|cos)_")
Instruction = collections.namedtuple("Instruction", "text kind writes reads dpp lane_read lane_select to_lds stored trans states ends")


def _regs(operands):
    out = set()
    for m in REG.finditer(" ".join(operands)):
        if m.group(1):
            out.add(m.group(1) + m.group(2))
        elif m.group(3):
            out.update(m.group(3) + str(i) for i in range(int(m.group(4)), int(m.group(5)) + 1))
        else:
            out.add(m.group(6))
    return frozenset(out)


@functools.lru_cache(maxsize=None)
def _parse(text):
    op, _, rest = text.partition(" ")
    ops = [o.strip() for o in rest.split(",")] if rest else []
    kind, writes, reads = "other", frozenset(), _regs(ops)
    if op.startswith("v_"):
        kind, n = "valu", 2 if CARRY_OUT.match(op) else 1
        writes, reads = _regs(ops[:n]), _regs(ops[n:])
        if "swap" in op:
            writes = reads = _regs(ops)
        elif op.startswith(("v_fmac", "v_mac")):
            reads |= _regs(ops[:1])
        if op.startswith("v_div_fmas"):      # (the others name their carry)
            reads |= {"vcc"}
    elif op.startswith(("buffer_", "global_", "flat_", "scratch_")):
        kind = "vmem"
    elif op.startswith("s_") and not op.startswith(("s_cmp", "s_bitcmp", "s_waitcnt", "s_nop", "s_barrier", "s_cbranch", "s_branch")):
        kind, writes, reads = "salu", _regs(ops[:1]), _regs(ops[1:])
    states = int(ops[0], 0) + 1 if op == "s_nop" else 1
    # (stores of more than eight bytes: the address of a global store comes first, the data of a buffer store)
    stored = _regs(ops[1:2] if op.startswith("global") else ops[:1]) if re.search(r"_store_dwordx[34]", op) else frozenset()
    lane_select = _regs(ops[2:3]) if op.startswith(("v_readlane", "v_writelane")) else frozenset()
    return Instruction(text, kind, writes, reads, _regs(ops[1:2]) if "_dpp" in op else frozenset(), op.startswith(("v_readlane", "v_readfirstlane")),
                       lane_select, kind == "vmem" and ("_lds_" in op or rest.endswith(" lds")), stored, bool(TRANS.match(op)), states,
                       op in ("s_branch", "s_endpgm", "s_setpc_b64"))


def _needed(w, r):
    """wait states between the two, and what for"""
    if w.stored:
        return (1, "data of a store") if r.kind == "valu" and w.stored & r.writes else (0, "")
    if w.kind == "salu":
        return (1, "M0, then a load to LDS") if "m0" in w.writes and r.to_lds else (0, "")
    scalars = [x for x in w.writes if x[0] == "s" or x == "vcc"]
    if r.kind == "vmem":
        return (5, "scalar register, then memory") if any(x in r.reads for x in scalars) else (0, "")
    if r.kind != "valu":
        return 0, ""
    if any(x in r.lane_select for x in scalars):
        return 4, "lane select"
    if any(x in r.reads for x in scalars):
        return (4, "v_div_fmas") if r.text.startswith("v_div_fmas") else (2, "scalar register, then vector instruction")
    if r.dpp and w.writes & r.dpp:
        return 2, "DPP operand"
    if r.lane_read and w.writes & r.reads:
        return 1, "lane read"
    if w.trans and not r.trans and w.writes & r.reads:
        return 1, "transcendental result"
    return 0, ""


def _functions(lines):
    """(name, instructions, which one a branch goes to) of a disassembly"""
    name, base, code, places, targets = "?", 0, [], {}, {}

    def done():
        return name, code, {i: places[at] for i, at in targets.items() if at in places}

    for line in lines:
        if line.endswith(">:\n"):
            yield done()
            name, base, code, places, targets = line[line.index("<") + 1:-3], int(line.split()[0], 16), [], {}, {}
            continue
        text, _, comment = line.partition("//")
        text = text.strip()
        if not text or text[0] not in "vsdbgf" or "_" not in text:
            continue
        if comment:
            places[int(comment.split(":")[0], 16)] = len(code)
        if "branch" in text and "+0x" in comment:
            targets[len(code)] = base + int(comment[comment.rindex("+0x") + 1:comment.rindex(">")], 16)
        code.append(_parse(" ".join(text.split())))
    yield done()


def short_of_waits(lines):
    """[(function, what for, needed, there, writer, reader)] of a disassembly, on every way from the one to the other"""
    found = []
    for function, code, targets in _functions(lines):
        for i, before in enumerate(code):
            if not before.writes and not before.stored:
                continue
            ways = [(i + 1, 0)]
            while ways:
                j, states = ways.pop()
                while j < len(code) and states < 5:
                    now = code[j]
                    if now.kind in ("valu", "vmem"):
                        need, why = _needed(before, now)
                        if need > states:
                            found.append((function, why, need, states, before.text, now.text))
                    states += now.states
                    if j in targets:
                        ways.append((targets[j], states))
                    if now.ends:
                        break
                    j += 1
    return found


@pytest.mark.parametrize("listing,count", [
    ("v_readlane_b32 s3, v20, s61\nv_cmp_eq_u32_e32 vcc, s3, v15\n", 1),
    ("v_cmp_eq_u32_e32 vcc, s3, v15\nv_addc_co_u32_e32 v26, vcc, v26, v26, vcc\n", 1),
    ("v_cmp_eq_u32_e32 vcc, s3, v15\ns_nop 1\nv_addc_co_u32_e32 v26, vcc, v26, v26, vcc\n", 0),
    ("v_readlane_b32 s51, v126, 51\ns_mov_b32 m0, s7\ns_nop 0\nbuffer_load_dword v118, s[48:51], 0 offen sc1 lds\n", 1),
    ("v_readlane_b32 s51, v126, 51\ns_mov_b32 m0, s7\ns_nop 3\nbuffer_load_dword v118, s[48:51], 0 offen sc1 lds\n", 0),
    ("s_mov_b32 m0, s88\nbuffer_load_dword v1, s[40:43], 0 offen lds\n", 1),
    ("s_mov_b32 m0, s88\nglobal_load_lds_dword v[0:1], off\n", 1),
    ("v_add_f32_e32 v1, v2, v3\nv_add_f32_dpp v1, v1, v1 row_mirror row_mask:0xf bank_mask:0xf\n", 1),
    ("v_add_f32_dpp v1, v1, v1 row_mirror row_mask:0xf bank_mask:0xf\nv_readlane_b32 s0, v1, 63\n", 1),
    ("v_exp_f32_e32 v1, v1\nv_add_f32_e32 v1, 1.0, v1\n", 1),
    ("global_store_dwordx4 v[0:1], v[4:7], off\nv_mov_b32_e32 v5, 0\n", 1),
    ("global_store_dwordx4 v[0:1], v[4:7], off\ns_nop 0\nv_mov_b32_e32 v5, 0\n", 0),
    ("v_cmp_eq_u32_e32 vcc, s3, v15\ns_branch 7\nv_addc_co_u32_e32 v26, vcc, v26, v26, vcc\n", 0),
    ("0000000000000100 <f>:\nv_addc_co_u32_e32 v26, s[0:1], v26, v26, vcc // 000000000100: 00\nv_cmp_eq_u32_e32 vcc, s3, v15 // 000000000104: 00\n"
     "s_cbranch_scc1 65533 // 000000000108: 00 <f+0x0>\ns_endpgm // 00000000010C: 00\n", 1),
    ("0000000000000100 <f>:\ns_nop 0 // 000000000100: 00\nv_addc_co_u32_e32 v26, s[0:1], v26, v26, vcc // 000000000104: 00\n"
     "v_cmp_eq_u32_e32 vcc, s3, v15 // 000000000108: 00\ns_cbranch_scc1 65533 // 00000000010C: 00 <f+0x0>\ns_endpgm // 000000000110: 00\n", 0),
])
def test_the_rules(listing, count):
    assert len(short_of_waits(listing.splitlines(keepends=True))) == count


@pytest.fixture(scope="module")
def found(tmp_path_factory):
    where = tmp_path_factory.mktemp("listing")
    lib = shutil.copy(build.LIB if os.path.exists(build.LIB) else build.build_library(), where)
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=where, check=True, capture_output=True)
    objects = sorted(str(p) for p in where.glob("*gfx950*"))

    def look(path):
        return subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", path], check=True, capture_output=True, text=True).stdout

    out, instructions = [], 0
    with concurrent.futures.ThreadPoolExecutor(8) as pool:
        for text in pool.map(look, objects):
            lines = text.splitlines(keepends=True)
            instructions += len(lines)
            out += short_of_waits(lines)
    assert instructions > 100000               # (all kernels were there to be read)
    return out


@pytest.mark.parametrize("why", ["scalar register, then vector instruction", "lane select", "v_div_fmas", "DPP operand", "lane read", "transcendental result",
                                 "M0, then a load to LDS", "scalar register, then memory", "data of a store"])
def test_no_kernel_is_short_of_wait_states(found, why):
    short = [f for f in found if f[1] == why]
    assert not short, f"{len(short)}, such as:\n" + "\n".join(map(str, short[:20]))

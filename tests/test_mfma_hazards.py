"""The strip kernels' MFMAs are inline assembly, so the compiler does not know that what they write may not be read or written by
anything but another MFMA for some wait states.  It must not spill or copy an accumulator right behind one: this looks through the
machine code of the built library for it."""
import glob
import os
import re
import shutil
import subprocess

import pytest

from paper_2604_02715_amd import binding as B
from paper_2604_02715_amd import build

WAIT_STATES = 8                  # what the compiler leaves behind the builtin of the same instruction (s_nop 7)
MFMA = "v_mfma_f32_16x16x32_bf16"
OBJDUMP = os.path.join(os.path.dirname(os.path.dirname(build.HIPCC)), "llvm", "bin", "llvm-objdump")


def registers(text):
    out = set()
    for a, b, c in re.findall(r"\ba(?:\[(\d+):(\d+)\]|(\d+)\b)", text):
        out.update([int(c)] if c else range(int(a), int(b) + 1))
    return out


def scalars(text):
    m = re.fullmatch(r"s(?:\[(\d+):(\d+)\]|(\d+))", text)
    return set() if not m else {int(m[3])} if m[3] else set(range(int(m[1]), int(m[2]) + 1))


def parse(listing):
    """{function: ([(mnemonic, operands)], {label: index})}"""
    functions, name = {}, None
    for line in listing.splitlines():
        m = re.match(r"[0-9a-f]+ <(\w+)>:", line)
        if m and not re.fullmatch(r"L\d+", m[1]):
            name = m[1]
            functions[name] = ([], {})
        elif m:
            functions[name][1][m[1]] = len(functions[name][0])
        elif name and line.startswith("\t"):
            op, _, args = line.split("//")[0].strip().partition(" ")
            functions[name][0].append((op, args.strip()))
    return functions


def hazards(code, labels):
    """Instructions other than MFMAs that touch an MFMA's accumulators within WAIT_STATES of it, along every path.  The compiler routes
    some paths by a flag (s_mov_b64 s, 0 or -1; s_and_b64 vcc, exec, s; s_cbranch_vccz): those go where the flag sends them."""
    touched = [registers(args) if not op.startswith("v_mfma") else set() for op, args in code]
    found = []
    for i, (op, args) in enumerate(code):
        if op != MFMA:
            continue
        acc = registers(args.split(",")[0])
        todo, seen = [(i + 1, 0, ())], set()
        while todo:
            at, waited, flags = todo.pop()
            if at >= len(code) or waited >= WAIT_STATES or (at, waited, flags) in seen:
                continue
            seen.add((at, waited, flags))
            op2, args2 = code[at]
            if touched[at] & acc:
                found.append((i, at, waited, op2 + " " + args2))
                continue
            waited += int(args2, 0) + 1 if op2 == "s_nop" else 1
            if op2 == "s_endpgm":
                continue
            known, parts = dict(flags), [x.strip() for x in args2.split(",")]
            if op2.startswith("s_") and not op2.startswith(("s_cmp", "s_branch", "s_cbranch", "s_nop", "s_waitcnt", "s_barrier")):
                value = None
                if op2 == "s_mov_b64" and parts[1] in ("0", "-1"):
                    value = parts[1] != "0"
                elif op2 in ("s_and_b64", "s_andn2_b64") and parts[:2] == ["vcc", "exec"] and parts[2] in known:
                    value = known[parts[2]] != (op2 == "s_andn2_b64")
                for k in [k for k in known if k == parts[0] or scalars(k) & scalars(parts[0])]:
                    del known[k]
                if value is not None:
                    known[parts[0]] = value
            elif re.match(r"v_cmp|v_div_scale|v_add_co|v_sub", op2):
                known.pop("vcc", None)
            flags = tuple(sorted(known.items()))
            taken = known.get("vcc") == (op2 == "s_cbranch_vccnz") if op2.startswith("s_cbranch_vcc") and "vcc" in known else None
            if op2.startswith(("s_branch", "s_cbranch")) and taken is not False:
                todo.append((labels[args2], waited, flags))
            if op2 != "s_branch" and taken is not True:
                todo.append((at + 1, waited, flags))
    return found


def test_the_check_sees_a_spill_behind_an_mfma():
    listing = """0000 <f>:
\tv_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]// 00:
\ts_cbranch_scc1 L1 // 00:
%s
\ts_endpgm // 00:
0010 <L1>:
%s
\ts_endpgm // 00:
"""
    spill, clean = "\tscratch_store_dwordx4 off, a[0:3], off // 00:", "\tv_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]// 00:"
    found = lambda a, b: len(hazards(*parse(listing % (a, b))["f"]))
    assert found(clean, clean) == 0
    assert found(spill, clean) == 1 and found(clean, spill) == 1
    assert found("\ts_nop 15 // 00:\n\ts_nop 15 // 00:\n" + spill, "\tv_accvgpr_read_b32 v0, a4 // 00:") == 0
    assert found("\ts_nop 3 // 00:\n\tv_accvgpr_read_b32 v0, a3 // 00:", clean) == 1
    by_flag = "\ts_mov_b64 s[0:1], %s // 00:\n\ts_and_b64 vcc, exec, s[0:1] // 00:\n\ts_cbranch_vccz L2 // 00:\n" + spill + "\n0020 <L2>:"
    assert found(by_flag % "0", clean) == 0 and found(by_flag % "-1", clean) == 1 and found(by_flag % "s[2:3]", clean) == 1


def test_no_accumulator_is_touched_right_behind_its_mfma(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no disassembler for the library that was built here")
    B.lib()                                                  # built, or built now
    so = str(tmp_path / "lib.so")
    shutil.copy(build.OUT, so)
    subprocess.run([OBJDUMP, "--offloading", so], check=True, capture_output=True, cwd=tmp_path)
    kernels = mfmas = 0
    for f in glob.glob(so + ".*gfx950"):
        listing = subprocess.run([OBJDUMP, "-d", "--symbolize-operands", "--no-show-raw-insn", f], check=True, capture_output=True, text=True).stdout
        for name, (code, labels) in parse(listing).items():
            n = sum(op == MFMA for op, _ in code)
            if n:
                assert hazards(code, labels) == [], name
                kernels, mfmas = kernels + 1, mfmas + n
    assert kernels >= 10 and mfmas > 1000

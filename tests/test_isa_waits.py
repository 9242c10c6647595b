"""Wait states in the compiled kernels.  The matrix instruction and inline assembly meet where the compiler's hazard pass cannot see:
it neither counts the cycles behind a register that assembly wrote, nor those ahead of one that assembly reads.  The library's own
code objects are disassembled and the distances that gfx950 wants are counted, along branches too:
  - a vector instruction's result is an operand of a matrix instruction 2 wait states later at the earliest,
  - a matrix instruction's result is read by the conversion to bf16 after its passes and 4 more (32x32x2 f32: 16 passes, 32x32x16 bf16:
    8, 16x16x32 bf16: 4),
  - a scalar register that a vector instruction wrote is the base of a copy to LDS 5 wait states later at the earliest, and M0 is
    written 1 ahead of it."""
import os
import re
import struct
import subprocess

import pytest

from paper_1711_04325_amd import build

OBJDUMP = os.path.join(os.path.dirname(os.path.realpath(build.HIPCC)), "..", "llvm", "bin", "llvm-objdump")
PASSES = {"v_mfma_f32_32x32x2_f32": 16, "v_mfma_f32_32x32x16_bf16": 8, "v_mfma_f32_16x16x32_bf16": 4}
LINE = re.compile(r"\t(\S+) ?(.*?)\s*// 0*([0-9A-F]+):(?:.*<(\S+)\+0x([0-9a-f]+)>)?")
REG = re.compile(r"\b([vsa])(?:(\d+)|\[(\d+):(\d+)\])|\b(m0)\b")


def code_objects(lib):
    """The gfx950 code objects of a shared library built by hipcc."""
    data, at = open(lib, "rb").read(), 0
    while (at := data.find(b"__CLANG_OFFLOAD_BUNDLE__", at)) >= 0:
        count, p = struct.unpack_from("<Q", data, at + 24)[0], at + 32
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + n]:
                yield data[at + off:at + off + size]
            p += 24 + n
        at += 24


def functions(text):
    """(name, [(mnemonic, operands, target)]) of every function of a listing; target: index of a branch's target in the list."""
    for part in re.split(r"^(?=[0-9a-f]{16} <)", text, flags=re.M)[1:]:
        head, body = part.split("\n", 1)
        base, code, at = int(head[:16], 16), [], {}
        for m in LINE.finditer(body):
            at[int(m.group(3), 16)] = len(code)
            code.append((m.group(1), m.group(2), int(m.group(5), 16) + base if m.group(5) and m.group(1).startswith(("s_cbranch", "s_branch")) else None))
        yield head[18:].rstrip(">:"), [(op, args, at.get(t)) for op, args, t in code]


def regs(text):
    """Registers an operand text names."""
    out = set()
    for kind, one, lo, hi, m0 in REG.findall(text):
        out.update([m0] if m0 else [kind + str(i) for i in range(int(one or lo), int(one or hi) + 1)])
    return out


def violations(code):
    jumps = {}
    for i, (_, _, t) in enumerate(code):
        if t is not None:
            jumps.setdefault(t, []).append(i)

    def before(i, budget, hit):
        """Whether an instruction for which `hit` is true ends less than `budget` wait states ahead of instruction i."""
        todo, seen = [(i, budget)], {}
        while todo:
            i, left = todo.pop()
            preds = jumps.get(i, []) + ([i - 1] if i and code[i - 1][0] not in ("s_branch", "s_endpgm", "s_setpc_b64") else [])
            for p in preds:
                if hit(*code[p][:2], left):
                    return True
                rest = left - (int(code[p][1], 0) + 1 if code[p][0] == "s_nop" else 1)
                if rest > 0 and seen.get(p, 0) < rest:
                    seen[p] = rest
                    todo.append((p, rest))
        return False

    for i, (op, args, _) in enumerate(code):
        if op.startswith("v_mfma"):
            want = regs(args.split(",", 1)[1])
            if before(i, 2, lambda o, a, _: o.startswith("v_") and not o.startswith("v_mfma") and regs(a.split(",", 1)[0]) & want):
                yield op, args
        elif op.startswith("v_cvt_pk_bf16"):
            want = regs(args.split(",", 1)[1])
            if before(i, 20, lambda o, a, left: o in PASSES and PASSES[o] + 4 > 20 - left and regs(a.split(",", 1)[0]) & want):
                yield op, args
        elif op.startswith("global_load_lds"):
            want = {r for r in regs(args) if r[0] == "s"}
            if before(i, 5, lambda o, a, _: o.startswith("v_") and regs(a.split(",", 1)[0]) & want) or before(i, 1, lambda o, a, _: a.startswith("m0")):
                yield op, args


def listing(lib, tmp_path):
    for i, obj in enumerate(code_objects(lib)):
        path = tmp_path / ("%d.co" % i)
        path.write_bytes(obj)
        yield subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", str(path)], capture_output=True, text=True, check=True).stdout


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler here")
def test_wait_states(tmp_path):
    seen, bad = set(), []
    for text in listing(build.LIB, tmp_path):
        for name, code in functions(text):
            seen.update(op for op, _, _ in code)
            bad += ["%s: %s %s" % (name, op, args) for op, args in violations(code)]
    assert seen.issuperset(PASSES) and "v_cvt_pk_bf16_f32" in seen and "global_load_lds_dwordx4" in seen
    assert not bad, "%d places:\n%s" % (len(bad), "\n".join(bad[:20]))


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler here")
def test_half_kernels_use_no_scratch(tmp_path):
    """Three sets of sums leave igemm_half_kernel few registers: where some spill, a launch takes a third longer."""
    seen = []
    for i, co in enumerate(code_objects(build.LIB)):
        path = tmp_path / str(i)
        path.write_bytes(co)
        notes = subprocess.run([OBJDUMP.replace("objdump", "readelf"), "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        seen += [(name, int(scratch)) for name, scratch in re.findall(r"\.name: +(_Z\S*igemm_half_kernel\S*)\n\s+\.private_segment_fixed_size: (\d+)", notes)]
    assert len(seen) == 6 and all(scratch == 0 for _, scratch in seen), seen

"""Wait states around the matrix instructions that are written as assembly statements, which the compiler knows nothing of: read off the
built library, along every path of every kernel that has such statements.

v_mfma_f32_16x16x32_bf16 may read a register that a vector instruction wrote once two other wait states have passed, and what it writes
may be read by anything but a product that accumulates on it after seven (four passes and three).  A wait state is an instruction of the
same wavefront, or one of the s_nop's.  The kernels whose products are builtins are the compiler's.

Likewise M0, which the global -> LDS loads take their LDS address from: statements write it, and a load (some windows later, in the
attention kernel and the wide products) uses it.  One other wait state stands between them, and nothing else writes it there: every write
is used before the next one.
"""
import os
import re
import struct
import subprocess

import pytest

from paper_2512_07350_amd import build

OBJDUMP = os.path.join(os.path.dirname(os.path.realpath(build._hipcc())), "..", "llvm", "bin", "llvm-objdump")
KERNELS = ("attention_kernel", "gemm_kernel")


def code_objects(path):
    """The gfx950 code objects of a library: bundles of (offset, size, target) entries."""
    data, magic = open(path, "rb").read(), b"__CLANG_OFFLOAD_BUNDLE__"
    for m in re.finditer(magic, data):
        at = m.start() + len(magic)
        n, at = struct.unpack_from("<Q", data, at)[0], at + 8
        for _ in range(n if n < 16 else 0):
            offset, size, length = struct.unpack_from("<3Q", data, at)
            at += 24 + length
            if b"gfx950" in data[at - length:at]:
                yield data[m.start() + offset:m.start() + offset + size]


def registers(operand):
    out = set()
    for file, lo, hi, one in re.findall(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+))(?!\w)", operand):
        out |= {(file, i) for i in (range(int(lo), int(hi) + 1) if lo else (int(one),))}
    return out


class Instruction:
    def __init__(self, text):
        self.op, _, rest = text.partition(" ")
        ops = [o.strip() for o in re.split(r",(?![^\[]*\])", rest)]
        self.product, self.vector = self.op.startswith("v_mfma"), self.op.startswith("v_")
        self.states = int(ops[0], 0) + 1 if self.op == "s_nop" else 1
        both = "swap" in self.op
        reads_first = both or not self.vector and ("store" in self.op or "write" in self.op or " lds" in rest) or self.op.startswith(("v_cmp", "v_readfirst"))
        self.reads = set().union(*(registers(o) for o in ops[0 if reads_first else 1:]))
        self.writes = registers(ops[0]) if not reads_first or both else set()
        if both:
            self.writes |= registers(ops[1])
        self.sum_on = registers(ops[3]) if self.product else set()
        self.writes_m0, self.uses_m0 = ops[0] == "m0", self.op.startswith("buffer_load") and rest.endswith(" lds")


def kernels(path, tmp):
    """(name, instructions, predecessors of each) of the kernels in KERNELS."""
    for i, obj in enumerate(code_objects(path)):
        name = str(tmp / ("%d.co" % i))
        open(name, "wb").write(obj)
        kernel, code, at, jumps = None, [], {}, []
        for line in subprocess.run([OBJDUMP, "-d", name], check=True, capture_output=True, text=True).stdout.splitlines() + ["0 <end>:"]:
            head = re.match(r"[0-9a-f]+ <(\S+)>:", line)
            if head:
                if kernel and any(k in kernel for k in KERNELS):
                    before = [[j] if j >= 0 and code[j].op not in ("s_branch", "s_endpgm", "s_setpc_b64") else [] for j in range(-1, len(code) - 1)]
                    for j, target in jumps:
                        before[at[target]].append(j)
                    yield kernel, code, before
                kernel, code, at, jumps = head.group(1), [], {}, []
                continue
            m = re.match(r"\s+(\S.*?)\s*// ([0-9A-F]+):.*?(?:<[^>+]*\+0x([0-9a-f]+)>|<([^>+]*)>)?$", line)
            if m and kernel:
                address = int(m.group(2), 16)
                if not at:
                    base = address
                at[address - base] = len(code)
                if m.group(1).startswith(("s_branch", "s_cbranch")):
                    jumps.append((len(code), int(m.group(3) or "0", 16)))
                code.append(Instruction(m.group(1)))


def too_close(code, before):
    """(reader, writer, states between them) of every pair that stands too close on some path."""
    bad = []
    for i, x in enumerate(code):
        if not x.reads or x.op.startswith("s_"):
            continue
        paths, seen = [(j, 0) for j in before[i]], set()
        while paths:
            j, passed = paths.pop()
            if passed >= 7 or (j, passed) in seen:
                continue
            seen.add((j, passed))
            y = code[j]
            if x.product and y.vector and not y.product and y.writes & x.reads and passed < 2:
                bad.append((i, j, passed))
            if y.product and y.writes & (x.reads - x.sum_on if x.product else x.reads):
                bad.append((i, j, passed))
            paths += [(k, passed + y.states) for k in before[j]]
    return bad


def m0_lost(code, before):
    """Loads whose M0 was written right in front of them, and writes of M0 that meet another write before a load."""
    bad = [i for i, x in enumerate(code) if x.uses_m0 and any(code[j].writes_m0 for j in before[i])]
    for i in (i for i, x in enumerate(code) if x.writes_m0):
        paths, seen = list(before[i]), set()
        while paths:
            j = paths.pop()
            if j in seen or code[j].uses_m0:
                continue
            seen.add(j)
            if code[j].writes_m0:
                bad.append(i)
            else:
                paths += before[j]
    return bad


def test_wait_states_around_products(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump beside hipcc")
    count = 0
    for name, code, before in kernels(build.LIB, tmp_path):
        count += sum(x.product for x in code) > 0
        bad = too_close(code, before)
        assert not bad, (name, [(code[j].op, code[i].op, passed) for i, j, passed in bad[:4]])
        assert not m0_lost(code, before), name
    assert count >= 8 + 30             # attention_kernel in four forms at either head_dim; the tilings of the products


def test_the_check_sees_what_stands_too_close():
    def found(*lines):
        code = [Instruction(l) for l in lines]
        return too_close(code, [[j] if j >= 0 else [] for j in range(-1, len(code) - 1)])
    product = "v_mfma_f32_16x16x32_bf16 v[4:7], v[8:11], a[12:15], v[4:7]"
    assert found("v_mov_b32_e32 v7, v0", "s_waitcnt lgkmcnt(0)", product) == [(2, 0, 1)]
    assert not found("v_mov_b32_e32 v7, v0", "s_nop 1", product)
    assert found("v_accvgpr_write_b32 a13, v0", "s_nop 0", product) == [(2, 0, 1)]
    assert not found(product, product)
    assert found(product, "s_nop 5", "v_exp_f32_e32 v0, v5") == [(2, 0, 6)]
    assert not found(product, "s_nop 6", "v_exp_f32_e32 v0, v5")
    assert found(product, "v_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[20:23], a[0:3]") == [(1, 0, 0)]
    assert found(product, "ds_write_b128 v0, v[4:7]") == [(1, 0, 0)]
    load = "buffer_load_dwordx4 v0, s[4:7], s8 offen lds"
    lost = lambda *lines: m0_lost([Instruction(l) for l in lines], [[j] if j >= 0 else [] for j in range(-1, len(lines) - 1)])
    assert not lost("s_add_u32 m0, s0, 16", product, load, "s_mov_b32 m0, s1", "s_nop 0", load)
    assert lost("s_mov_b32 m0, s1", load) == [1]
    assert lost("s_mov_b32 m0, s1", product, "s_mov_b32 m0, -1", product, load) == [2]

"""The latent-KV kernels as compiled: what their assembly statements rely on and the compiler does not check.

The MFMAs of mla_tile_kernel are assembly statements, so no wait states are inserted between an MFMA and the instructions
that touch its registers, and its loads into LDS take their LDS address from m0.  Both are read here from the device code of
the built library (its own disassembly), over every path through a kernel."""
import glob
import os
import re
import subprocess

import pytest

from paper_2510_14686_amd import build as xbuild

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
# Wait states (issue slots of a wave) between an MFMA and a vector or memory instruction that touches its result: 19 is what
# the longest MFMAs (16 passes) need, those used here (8 passes) need 12.  Between a vector instruction and an MFMA or a
# lane swap that reads its result: 2; between one that writes a scalar register and a memory instruction that reads it: 5.
# An MFMA occupies the pipe for its passes, so one that follows another counts 8.
RESULT_WAIT, OPERAND_WAIT, SCALAR_WAIT, PASSES = 19, 2, 5, 8
REG = re.compile(r"\b([vas])(?:(\d+)\b|\[(\d+):(\d+)\])")


def _registers(text):
    out = set()
    for kind, one, first, last in REG.findall(text):
        out |= {(kind, i) for i in (range(int(first), int(last) + 1) if first else (int(one),))}
    return out


def _parse(text):
    """{kernel: [(address, operation, operands, branch target or None)]}"""
    kernels, code = {}, None
    for line in text.splitlines():
        m = re.match(r"([0-9a-f]+) <(\S+)>:", line)
        if m:
            base, name = int(m[1], 16), m[2]
            code = kernels[name] = []
            continue
        m = re.match(r"\t(\S+)\s*(.*?)\s*// ([0-9A-F]+):[^<]*(?:<(\S+?)(?:\+0x([0-9a-f]+))?>)?", line)
        if m and code is not None:
            target = base + int(m[5] or "0", 16) if m[4] and "branch" in m[1] else None
            code.append((int(m[3], 16), m[1], m[2], target))
    return kernels


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    work = tmp_path_factory.mktemp("code")
    lib = os.path.join(str(work), "lib.so")
    os.symlink(xbuild.build(), lib)
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=str(work), check=True, capture_output=True)
    out = {}
    for part in glob.glob(os.path.join(str(work), "*gfx950")):
        out.update(_parse(subprocess.run([OBJDUMP, "-d", part], check=True, capture_output=True, text=True).stdout))
    return out


def _blocks(code):
    """Basic blocks as (first, end) index pairs, and each block's successors."""
    at = {ins[0]: i for i, ins in enumerate(code)}
    starts = {0} | {at[ins[3]] for ins in code if ins[3] is not None}
    starts |= {i + 1 for i, ins in enumerate(code) if "branch" in ins[1] or ins[1] == "s_endpgm"}
    starts = sorted(s for s in starts if s < len(code))
    number = {s: k for k, s in enumerate(starts)}
    spans = list(zip(starts, starts[1:] + [len(code)]))
    follow = []
    for k, (first, end) in enumerate(spans):
        op, target = code[end - 1][1], code[end - 1][3]
        to = [number[at[target]]] if target is not None else []
        if op not in ("s_branch", "s_endpgm") and k + 1 < len(spans):
            to.append(k + 1)
        follow.append(to)
    return spans, follow


def _of(registers, kinds):
    return {r for r in registers if r[0] in kinds}


def _hazards(code):
    """Instructions that come too soon behind an MFMA or a vector instruction.  The state at a block's start holds, per
    register, the fewest wait states that any way to it leaves behind."""
    spans, follow = _blocks(code)
    decoded = []
    for _, op, operands, _ in code:
        ops = [_registers(o) for o in operands.split(", ")]
        everything = _registers(operands)
        vector, swap, mfma = op.startswith("v_"), "permlane" in op and "swap" in op, op.startswith("v_mfma")
        memory = op.startswith(("buffer_", "global_", "flat_", "scratch_"))
        writes = ops[0] | (ops[1] if swap else set()) if vector else set()
        scalar_dest = ops[0] if op.startswith("s_") and not op.startswith(("s_cmp", "s_bitcmp")) else set()
        late = set()                                    # must not have been written by a vector instruction just before
        if mfma:
            late = set().union(*ops[1:])
        elif swap:
            late = ops[0] | ops[1]
        elif memory:
            late = _of(everything, "s")
        touches = _of(everything, "va") if vector or memory or op.startswith("ds_") else set()
        decoded.append((mfma, writes, late, touches, ops[3] if mfma else scalar_dest, int(operands, 0) + 1 if op == "s_nop" else 1))
    entry = [None] * len(spans)
    entry[0] = ({}, {}, {})
    bad, todo = set(), [0]
    while todo:
        k = todo.pop()
        # register -> wait states since an MFMA / a vector instruction / a vector instruction (scalar registers) wrote it
        state = tuple(dict(s) for s in entry[k])
        results, values, scalars = state

        def pass_time(n):
            for ages, most in zip(state, (RESULT_WAIT, OPERAND_WAIT, SCALAR_WAIT)):
                for r in [r for r, age in ages.items() if age + n >= most]:
                    del ages[r]
                for r in ages:
                    ages[r] += n

        for i in range(*spans[k]):
            mfma, writes, late, touches, other, slots = decoded[i]
            if any(r in values or r in scalars for r in late):
                bad.add(i)
            if mfma:                                    # an accumulator that is added to and written again needs no wait
                again = writes if other == writes else set()
                if any(r in results for r in touches - again):
                    bad.add(i)
                pass_time(PASSES)
                for r in writes:
                    results[r] = 0
                    values.pop(r, None)
                continue
            if any(r in results for r in touches):
                bad.add(i)
            pass_time(slots)
            for r in writes:
                (scalars if r[0] == "s" else values)[r] = 0
            for r in other:                             # written anew by a scalar instruction, which needs no wait
                scalars.pop(r, None)
        for t in follow[k]:
            old = entry[t]
            new = state if old is None else tuple({r: min(a.get(r, 99), b.get(r, 99)) for r in set(a) | set(b)} for a, b in zip(old, state))
            if new != old:
                entry[t] = tuple(dict(s) for s in new)
                todo.append(t)
    assert sum(e is not None for e in entry) > 0.9 * len(entry)          # nearly all of the kernel was reached
    return [code[i] for i in sorted(bad)]


@pytest.mark.parametrize("mode", [0, 1, 2])
def test_mfma_statements_have_their_wait_states(kernels, mode):
    code = [c for name, c in kernels.items() if "mla_tile_kernelILi%dE" % mode in name]
    assert len(code) == 1
    n = sum(ins[1] == "v_mfma_f32_32x32x16_bf16" for ins in code[0])
    assert n > 300
    assert _hazards(code[0]) == []


def test_the_hazard_check_sees_hazards():
    """Planted in text: a result read too soon, an operand written too late, a result carried over a branch."""
    mfma = "v_mfma_f32_32x32x16_bf16", "v[0:15], v[16:19], v[20:23], v[0:15]", None
    end = "s_endpgm", "", None

    def code(*ins):
        return [(4 * i,) + x for i, x in enumerate(ins)]

    nops = lambda n: ("s_nop", str(n - 1), None)      # noqa: E731
    assert len(_hazards(code(mfma, nops(16), ("v_add_f32_e32", "v30, v31, v3", None), end))) == 1
    assert _hazards(code(mfma, nops(16), nops(3), ("v_add_f32_e32", "v30, v31, v3", None), end)) == []
    assert len(_hazards(code(("v_mov_b32_e32", "v21, v40", None), nops(1), mfma, end))) == 1
    assert _hazards(code(("v_mov_b32_e32", "v21, v40", None), nops(2), mfma, end)) == []
    assert _hazards(code(mfma, mfma, end)) == []
    load = "buffer_load_dwordx4", "v2, s[4:7], s9 offen nt lds", None
    assert len(_hazards(code(("v_readfirstlane_b32", "s9, v3", None), nops(4), load, end))) == 1
    assert _hazards(code(("v_readfirstlane_b32", "s9, v3", None), nops(5), load, end)) == []
    assert len(_hazards(code(("v_max3_f32", "v3, v4, v5, v6", None), ("v_permlane32_swap_b32_e32", "v2, v3", None), end))) == 1
    around = code(mfma, ("s_cbranch_vccz", "1", 12), nops(24), ("v_mov_b32_e32", "v50, v0", None), end)
    assert [ins[1] for ins in _hazards(around)] == ["v_mov_b32_e32"]
    loop = code(("v_add_f32_e32", "v30, v31, v3", None), mfma, ("s_cbranch_scc1", "0", 0), end)
    assert [ins[1] for ins in _hazards(loop)] == ["v_add_f32_e32"]


def test_loads_into_lds_take_their_address_from_an_m0_the_compiler_knows_of(kernels):
    """m0 is an operand of the load's statement: a statement that wrote m0 behind the compiler's back would break any use
    that the compiler makes of it.  In the code every such load has its own write of m0 ahead, a wait state between."""
    for path in glob.glob(os.path.join(xbuild.CSRC, "*.hip")) + glob.glob(os.path.join(xbuild.CSRC, "*.h")):
        with open(path) as f:
            assert not re.search(r'"[^"\n]*\bm0\s*,', f.read()), path
    loads = 0
    for name, code in kernels.items():
        write = None
        starts = {s for s, _ in _blocks(code)[0]}
        for i, (_, op, operands, _) in enumerate(code):
            if i in starts:
                write = None
            if re.match(r"m0\b", operands):
                write = i
            elif operands.endswith(" lds"):
                loads += 1
                assert write is not None and i - write >= 2, (name, i)
                write = None
    assert loads > 500


def test_loads_into_lds_wait_for_their_scalar_operands(kernels):
    """Their statements read scalar registers (descriptor, offset), which the compiler may have just written from a lane."""
    names = [name for name, code in kernels.items() if any(ins[2].endswith(" lds") for ins in code)]
    assert len(names) >= 16
    for name in names:
        assert [ins for ins in _hazards(kernels[name]) if ins[2].endswith(" lds")] == [], name

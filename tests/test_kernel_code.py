"""Properties of the kernels that their results do not show, from the assembly of the sources as the library is built."""
import functools
import os
import re
import subprocess

import pytest

from paper_2510_24606_amd import build


@functools.lru_cache(maxsize=None)
def assembly_text(source):
    cmd = [build.hipcc()] + build.FLAGS + ["--cuda-device-only", "-S", "-o", "-", os.path.join(build.HERE, "csrc", source)]
    return subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, check=True).stdout


def assembly(source):
    """{kernel symbol: its lines}"""
    text = assembly_text(source)
    found = re.findall(r"^(_Z\S+):[^\n]*\n(.*?)^\.Lfunc_end", text, flags=re.S | re.M)
    return {name: [line.strip() for line in body.splitlines()] for name, body in found}


def test_a_kept_boundary_is_marked_before_it_stops_being_undecided():
    """Other waves read `undecided`, then `kept`: one that sees a position as decided has to see that it is kept."""
    (code,) = [c for name, c in assembly("boundaries.hip").items() if "k_nms_windows" in name]
    ops = [op for op in (line.split(";")[0].strip() for line in code) if op]
    at = [i for i, op in enumerate(ops) if op.startswith("ds_and_b32")]
    assert at
    for i in at:
        back = ops[max(0, i - 8):i]
        mark = max(j for j, op in enumerate(back) if op.startswith("ds_or_b32"))
        assert any("lgkmcnt(0)" in op for op in back[mark:]), back


def scratch(source):
    """{kernel symbol: bytes of scratch memory per lane}"""
    return {name: int(n) for name, n in re.findall(r"\.amdhsa_kernel (\S+)\n.*?\.amdhsa_private_segment_fixed_size (\d+)",
                                                   assembly_text(source), flags=re.S)}


@pytest.mark.parametrize("source", ["recall.hip"])
def test_kernels_keep_their_registers(source):
    """Spilled registers go through memory in the inner loop."""
    found = scratch(source)
    assert found and not any(found.values()), found


def test_f32_attention_of_small_heads_keeps_three_waves():
    """32-row workgroups of D = 64: 512 registers per SIMD lane hold three waves of at most 168."""
    (n,) = [int(n) for name, n in re.findall(r"\.amdhsa_kernel (\S+)\n.*?\.amdhsa_next_free_vgpr (\d+)",
                                             assembly_text("attn.hip"), flags=re.S) if "ILi64ELi2E" in name]
    assert n <= 168 and [b for name, b in scratch("attn.hip").items() if "ILi64ELi2E" in name] == [0]


def test_wave_accumulators_and_m0_are_left_alone():
    """O lives in fixed accumulation registers between the assembly statements that name them, and the loads into LDS
    count on M0: the compiler puts nothing there."""
    kernels = {name: code for name, code in assembly("attn_wave.hip").items() if "k_attn_wave" in name}
    assert len(kernels) == 3 and not any(scratch("attn_wave.hip").values())
    for name, body in kernels.items():
        # row blocks of 32 x 32 columns, twice (once per half of the keys) where a wave has a tile of at most 64 rows
        mine = set(range(16 * 4 * {"1ILi3E": 3, "1ILi2E": 4, "2ENS": 2}[re.search(r"k_attn_wave(1ILi.E|2ENS)", name)[1]]))
        inside, seen = False, set()
        for line in body:
            if "ASMSTART" in line or "ASMEND" in line:
                inside = "ASMSTART" in line
                continue
            regs = {int(x) for x in re.findall(r"\ba(\d+)\b", line)}
            for lo, hi in re.findall(r"\ba\[(\d+):(\d+)\]", line):
                regs |= set(range(int(lo), int(hi) + 1))
            if inside:
                seen |= regs & mine
            else:
                assert not regs & mine and not re.search(r"\bm0\b", line), (name, line)
        assert seen == mine


def wave_kernels():
    """{(row blocks of a wave, waves of a tile): lines of the kernel}"""
    kernels = {name: code for name, code in assembly("attn_wave.hip").items() if "k_attn_wave" in name}
    return {{"1ILi3E": (3, 1), "1ILi2E": (2, 1), "2ENS": (2, 2)}[re.search(r"k_attn_wave(1ILi.E|2ENS)", name)[1]]: code
            for name, code in kernels.items()}


@pytest.mark.parametrize("shape", [(2, 1), (3, 1), (2, 2)])
def test_wave_loops_make_no_products_for_their_rare_branches(shape):
    """The vector unit has no issue cycles to spare beside the matrix products.  A unit (32 keys of a row block) needs one
    product, its scaled reference; the compiler has made those of the branch that moves references, 16 a unit, before it."""
    blocks = re.split(r"^(?:\.LBB\S+:.*|; %bb.*)$", "\n".join(wave_kernels()[shape]), flags=re.M)
    hot = [b for b in blocks if b.count("v_mfma") > 2]
    assert sum(b.count("v_mfma") for b in hot) >= 2 * shape[0] * 16
    assert sum(len(re.findall(r"^v_mul_f32", b, flags=re.M)) for b in hot) <= 2 * shape[0]


def registers(op, after=0):
    """Names of the vector and accumulation registers among the operands of an instruction, from operand `after` on."""
    found = set()
    for text in op.split(None, 1)[1].split(",")[after:] if " " in op else []:
        for kind, lo, hi in re.findall(r"\b([va])(?:(\d+)\b|\[)(?=(?:\d+:(\d+)\])?)", text):
            if lo:
                found.add(kind + lo)
            elif hi:
                first = int(re.search(rf"\b{kind}\[(\d+):{hi}\]", text)[1])
                found |= {f"{kind}{n}" for n in range(first, int(hi) + 1)}
    return found


def within(ops, labels, i, states, visit):
    """Calls visit(instruction) for all that can follow ops[i] within so many wait states, over both ways of a branch."""
    seen, todo = {}, [(i + 1, 0)]
    while todo:
        at, waited = todo.pop()
        if at >= len(ops) or waited >= states or seen.get(at, states) <= waited:
            continue
        seen[at] = waited
        op = ops[at]
        visit(op)
        if op.startswith(("s_branch", "s_cbranch")):
            todo.append((labels[op.split()[1]], waited + 1))
        if not op.startswith(("s_branch", "s_endpgm")):
            todo.append((at + 1, waited + (int(op.split()[1]) + 1 if op.startswith("s_nop") else 1)))


@pytest.mark.parametrize("shape", [(2, 1), (3, 1), (2, 2)])
def test_distances_that_the_hardware_does_not_keep_for_products_in_assembly(shape):
    """The compiler keeps them for its own instructions only.  A product of 8 passes: 12 wait states until anything but a
    product touches its result (and none may have it as a factor sooner); 2 from a vector instruction's result to the product
    that reads it."""
    ops, labels = [], {}
    for line in wave_kernels()[shape]:
        line = line.split(";")[0].strip()
        if line.endswith(":"):
            labels[line[:-1]] = len(ops)
        elif line and not line.startswith("."):
            ops.append(line)
    products = 0
    for i, op in enumerate(ops):
        result = registers(op.split(",")[0])
        if op.startswith("v_mfma"):
            products += 1

            def late(other, result=result, op=op):
                mine = registers(other, 1) if other.startswith("v_mfma") else registers(other)
                if other.startswith("v_mfma") and registers(other.split(",")[0]) == result:
                    mine -= result                                   # the next product of the sum
                assert not mine & result, (op, other)
            within(ops, labels, i, 12, late)
        elif op.startswith("v_") and result:
            def soon(other, result=result, op=op):
                assert not other.startswith("v_mfma") or not registers(other, 1) & result, (op, other)
            within(ops, labels, i, 2, soon)
    assert products >= 2 * shape[0] * 16

"""The accumulators of the 64-row backward kernels in the code that is built.

hexi_bf16_quad.hip issues the products that it sums over the whole sequence through inline assembly, which the compiler does not know to be
MFMAs: it counts no wait states before an instruction of its own that touches such an accumulator.  The source has none between the products,
but a register copy placed by the compiler would read a value that is still being written.  This compiles the file to assembly and follows
every path through each kernel.
"""
import os
import re
import subprocess

import pytest

from paper_2605_07569_amd import build

SRC = "hexi_bf16_quad.hip"
# wait states between an MFMA of 16 passes (these have 8) and a vector instruction that reads or writes its result
WAIT_STATES = 18


def kernels(text):
    """{name: (instructions, {label: index})}; an instruction is (text, whether it stands in inline assembly)"""
    out, cur, asm = {}, None, False
    for line in text.split("\n"):
        start = re.match(r"^(_Z\w+):\s*; @", line)
        if start:
            cur, asm = out.setdefault(start.group(1), ([], {})), False
        elif line.startswith(".Lfunc_end"):
            cur = None
        elif cur is None:
            continue
        elif "#ASMSTART" in line or "#ASMEND" in line:
            asm = "#ASMSTART" in line
        elif re.match(r"^\.LBB\w+:", line):
            cur[1][line.split(":")[0]] = len(cur[0])
        else:
            code = line.split(";")[0].strip()
            if code and not code.startswith("."):
                cur[0].append((code, asm))
    return out


def accumulation_registers(text):
    regs = set()
    for a, lo, hi in re.findall(r"\ba(?:(\d+)|\[(\d+):(\d+)\])", text):
        regs |= {int(a)} if a else set(range(int(lo), int(hi) + 1))
    return regs


def violations(ins, labels):
    """Instructions that touch a register of an inline-assembly MFMA's result fewer than WAIT_STATES after it, on some path.  Further such
    products may: the hardware forwards an accumulator to the next product on it."""
    state, bad, work = {0: {}}, set(), [0]         # per instruction: {register: wait states since its MFMA}
    while work:
        i = work.pop()
        text, asm = ins[i]
        op, now = text.split()[0], dict(state[i])
        if asm and op.startswith("v_mfma"):
            step = 1
            for r in accumulation_registers(text.split(",")[0]):
                now[r] = -step                     # (counted from the instruction after it)
        else:
            if any(r in now for r in accumulation_registers(text)):
                bad.add(text)
            step = int(text.split()[1]) + 1 if op == "s_nop" else 1
        now = {r: n + step for r, n in now.items() if n + step < WAIT_STATES}
        if op == "s_endpgm":
            nxt = []
        elif op == "s_branch":
            nxt = [labels[text.split()[1]]]
        else:
            nxt = [i + 1] + ([labels[text.split()[1]]] if op.startswith("s_cbranch") else [])
        for j in nxt:
            old = state.get(j)
            new = now if old is None else {r: min(now.get(r, WAIT_STATES), old.get(r, WAIT_STATES)) for r in now.keys() | old.keys()}
            if new != old:
                state[j] = new
                work.append(j)
    return bad


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    if not os.path.exists(build._hipcc()):
        pytest.skip("hipcc not available")
    out = str(tmp_path_factory.mktemp("quad") / "quad.s")
    r = subprocess.run([build._hipcc()] + build.FLAGS + build.FILE_FLAGS.get(SRC, []) + ["--offload-device-only", "-S", os.path.join(build.CSRC, SRC), "-o", out],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    with open(out) as f:
        return f.read()


def test_nothing_touches_an_accumulator_before_it_has_settled(assembly):
    found = kernels(assembly)
    backward = {n: k for n, k in found.items() if "bwd_quad" in n}
    assert len(backward) == 4 and len(found) == 6
    for name, (ins, labels) in backward.items():
        assert sum(asm and code.startswith("v_mfma") for code, asm in ins) >= 32, name
        assert violations(ins, labels) == set(), name


def test_no_kernel_keeps_registers_in_memory(assembly):
    spills = re.findall(r"\.vgpr_spill_count:\s*(\d+)", assembly)
    assert len(spills) == 6 and set(spills) == {"0"}


def test_a_copy_between_two_products_is_noticed(assembly):
    # planted in the text: a copy out of an accumulator one and six instructions behind a product, and behind the wait that ends them all (allowed)
    name, (ins, labels) = next((n, k) for n, k in kernels(assembly).items() if "bwd_quad" in n)
    at = [i for i, (code, asm) in enumerate(ins) if asm and code.startswith("v_mfma")]
    reg = min(accumulation_registers(ins[at[len(at) // 2]][0].split(",")[0]))
    jump = next(i for i in range(at[-1], len(ins)) if ins[i][0].startswith("s_nop 15"))
    for where, seen in ((at[len(at) // 2] + 1, True), (at[len(at) // 2] + 6, True), (jump + 2, False)):
        planted = ins[:where] + [(f"v_accvgpr_read_b32 v0, a{reg}", False)] + ins[where:]
        moved = {n: i + (i >= where) for n, i in labels.items()}
        assert bool(violations(planted, moved)) == seen

"""The projections' matrix products are inline assembly, so the compiler does not know how long their results take. What the
source promises instead is read from the assembly that it compiles to: nothing but a product touches a product's result
before the wait behind the last one, no vector instruction writes an operand right in front of its product, nothing spills."""
import os
import re
import subprocess

import pytest

from paper_2505_16175_amd import build

RESULT_WAIT = 12   # wait states from a 16x16x32 product (8 passes) to a vector read or write of its result
OPERAND_WAIT = 2   # ... from a vector write of a register to a product that reads it
PRODUCT = "v_mfma_f32_16x16x32_bf16"


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("asm") / "gemm_bf16.s")
    cmd = [a for a in build.hipcc_command(out) if a not in ("-shared", "-fPIC") and not a.endswith(".hip")]
    subprocess.run(cmd + ["-S", "--offload-device-only", os.path.join(build.CSRC, "gemm_bf16.hip")], check=True, capture_output=True)
    with open(out) as f:
        return f.read()


def _registers(text):
    regs = set()
    for a, b in re.findall(r"\bv\[(\d+):(\d+)\]", text):
        regs.update(range(int(a), int(b) + 1))
    regs.update(int(r) for r in re.findall(r"\bv(\d+)\b", text))
    return regs


def violations(text):
    """(products, what breaks the promise) of a listing, in program order; a wait state per instruction, n + 1 for s_nop n."""
    pending, written, now, products, bad = {}, {}, 0, 0, []
    for line in text.splitlines():
        line = line.split(";")[0].strip()
        if re.match(r"_Z\w+:", line):
            pending, written = {}, {}
        if not line or line.startswith(".") or line.endswith(":"):
            continue
        name, _, rest = line.partition(" ")
        ops = [o.strip() for o in rest.split(",")]
        if name == PRODUCT:
            products += 1
            dst, a, b, c = ops
            if dst != c:
                bad.append(f"not in place: {line}")
            bad += [f"operand written {now - written[r]} before: {line}" for r in _registers(a) | _registers(b) | _registers(c)
                    if now - written.get(r, -99) <= OPERAND_WAIT]
            bad += [f"operand is a result under way: {line}" for r in _registers(a) | _registers(b) if now - pending.get(r, -99) <= RESULT_WAIT]
            for r in _registers(dst):
                pending[r] = now
        else:
            touched = _registers(rest)
            bad += [f"result touched {now - pending[r]} after its product: {line}" for r in touched if now - pending.get(r, -99) <= RESULT_WAIT]
            if name.startswith("v_"):
                for r in _registers(ops[0]):
                    written[r] = now
        now += 1 + (int(ops[0]) if name == "s_nop" else 0)
    return products, bad


def test_results_are_left_alone_until_the_wait(assembly):
    products, bad = violations(assembly)
    assert products > 1000 and not bad, bad[:5]


def test_a_touched_result_is_found(assembly):
    """The reading itself: a copy of an accumulator behind its product, and an operand written in front of it."""
    first = re.search(PRODUCT + r" v\[(\d+):\d+\], v\[(\d+):.*\n", assembly)
    for at, line in ((first.end(), f"\tv_mov_b32_e32 v0, v{first.group(1)}\n"), (first.start(), f"v_mov_b32_e32 v{first.group(2)}, 0\n\t")):
        assert violations(assembly[:at] + line + assembly[at:])[1]


def test_no_kernel_spills(assembly):
    for key in (".vgpr_spill_count", ".sgpr_spill_count", ".private_segment_fixed_size"):
        counts = re.findall(re.escape(key) + r":\s+(\d+)", assembly)
        assert counts and set(counts) == {"0"}, key

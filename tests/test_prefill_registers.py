"""CPU: what the prefill kernels' assembly text relies on, read from the built library's own code.  Their accumulators live in fixed accumulation
registers that the compiler does not know to be live, so nothing else may ever be kept in one; and the wide kernel's matrix instructions
bring no wait states of their own, so an operand's last vector instruction has to lie far enough ahead."""
import re
import subprocess
from pathlib import Path

import pytest

from paper_2506_12038_amd.build import LIB
from test_kernel_resources import _code_objects

OBJDUMP = Path("/opt/rocm/llvm/bin/llvm-objdump")
MFMA = re.compile(r"v_mfma_f32_32x32x16_f16 a\[(\d+):(\d+)\], v\[(\d+):(\d+)\], v\[(\d+):(\d+)\], a\[(\d+):(\d+)\]$")
WAIT_STATES = 2      # between a vector instruction that writes a register and a matrix instruction that reads it as an operand


def _accumulators(name):
    """16-register accumulators of every body (output tile) that a kernel holds, None: no prefill kernel."""
    kernel, args = re.match(r"_ZN3lcd\d+(\w+?)I((?:Li\d+E)+)E", name).groups() if re.match(r"_ZN3lcd\d+\w+?I(?:Li\d+E)+E", name) else (name, "")
    args = [int(a) for a in re.findall(r"Li(\d+)E", args)]
    if kernel == "gemm_split_kernel":
        _, pairs, blocks = args
        return [pairs * blocks]
    if kernel == "gemm_wide_kernel":
        _, blocks, _, pairs = args
        return [pairs * b for b in (blocks, blocks - 1) if b > 0]
    if kernel == "gemm_mixed_kernel":
        _, split, blocks, pairs = args
        return [2 * split, pairs * blocks, pairs * (blocks - 1)]
    return None


def _written(text):
    """Vector registers that an instruction of the vector pipe writes."""
    m = re.match(r"v_(?!mfma|cmp|readlane|readfirstlane|nop)\w+ (?:v(\d+)|v\[(\d+):(\d+)\])", text)
    if not m:
        return ()
    return (int(m[1]),) if m[1] else range(int(m[2]), int(m[3]) + 1)


def _slots(text):
    m = re.match(r"s_nop (\d+)", text)
    return int(m[1]) + 1 if m else 1


def _too_near(lines):
    """Matrix instructions of a kernel that read a register within the wait states behind the vector instruction that wrote it, over every way
    the control flow takes there.  lines: instructions, and labels as 'L7:'."""
    at = {t[:-1]: i for i, t in enumerate(lines) if t.endswith(":")}
    into = {}
    for i, t in enumerate(lines):
        m = re.match(r"s_c?branch\w* (L\d+)", t)
        if m:
            into.setdefault(at[m[1]], []).append(i)
    found = []

    def back(i, slots, needed, mfma):
        """from instruction i - 1 backwards"""
        while slots < WAIT_STATES and i > 0:
            if lines[i].endswith(":"):
                for source in into.get(i, ()):
                    back_over(source, slots, needed, mfma)
            i -= 1
            if re.match(r"s_branch |s_endpgm", lines[i]):
                return
            if lines[i].endswith(":"):
                continue
            if needed & set(_written(lines[i])):
                found.append((mfma, lines[i]))
                return
            slots += _slots(lines[i])

    def back_over(branch, slots, needed, mfma):
        if slots + 1 < WAIT_STATES:
            back(branch, slots + 1, needed, mfma)

    for i, t in enumerate(lines):
        m = MFMA.match(t)
        if m:
            needed = set(range(int(m[3]), int(m[4]) + 1)) | set(range(int(m[5]), int(m[6]) + 1))
            back(i, 0, needed, t)
    return found


def test_the_search_finds_a_near_write():
    mfma = "v_mfma_f32_32x32x16_f16 a[0:15], v[4:7], v[8:11], a[0:15]"
    assert _too_near(["s_nop 0", "v_perm_b32 v5, v1, v2, v3", mfma])
    assert _too_near(["s_nop 0", "v_pk_lshlrev_b16 v[8:9], 1, v[2:3]", "s_waitcnt lgkmcnt(0)", mfma])
    assert not _too_near(["s_nop 0", "v_perm_b32 v5, v1, v2, v3", "s_nop 1", mfma])
    assert not _too_near(["s_nop 0", "v_perm_b32 v12, v5, v2, v3", mfma])
    assert _too_near(["s_nop 0", "L0:", mfma, "s_nop 7", "v_perm_b32 v5, v1, v2, v3", "s_cbranch_scc1 L0"])
    assert not _too_near(["s_nop 0", "L0:", mfma, "s_nop 7", "v_perm_b32 v5, v1, v2, v3", "s_nop 0", "s_cbranch_scc1 L0"])


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{name: instructions and labels} of the prefill kernels in the library."""
    if not OBJDUMP.exists():
        pytest.skip("no llvm-objdump")
    folder, found = tmp_path_factory.mktemp("code"), {}
    for i, code in enumerate(_code_objects(LIB.read_bytes())):
        if not re.search(rb"gemm_(split|wide|mixed)_kernel", code):
            continue
        f = folder / f"{i}.co"
        f.write_bytes(code)
        text = subprocess.run([str(OBJDUMP), "-d", "--symbolize-operands", str(f)], capture_output=True, text=True, check=True).stdout
        for part in re.split(r"^[0-9a-f]+ <(?=_Z)", text, flags=re.M)[1:]:
            name, body = part.split(">:\n", 1)
            if _accumulators(name) is None:
                continue
            lines = []
            for line in body.splitlines():
                label = re.match(r"[0-9a-f]+ <(L\d+)>:", line)
                if label:
                    lines.append(label[1] + ":")
                elif line.startswith("\t"):
                    lines.append(line.split("//")[0].strip())
            found[name] = lines
    return found


def test_accumulation_registers_hold_accumulators_only(kernels):
    assert len(kernels) == 18 + 36 + 24
    wrong = {}
    for name, lines in kernels.items():
        bodies, zeroed = _accumulators(name), 0
        for t in lines:
            if not re.search(r"\ba(\d+|\[\d+:\d+\])", t):
                continue
            m = MFMA.match(t)
            if m:
                good = (m[1], m[2]) == (m[7], m[8]) and int(m[1]) % 16 == 0 and int(m[2]) == int(m[1]) + 15 and int(m[2]) < 16 * max(bodies)
            elif re.match(r"v_accvgpr_write_b32 a\d+, 0$", t):
                zeroed += 1
                good = int(re.match(r"\S+ a(\d+)", t)[1]) < 16 * max(bodies)
            else:
                good = re.match(r"v_accvgpr_read_b32 v\d+, a\d+$", t)
            if not good:
                wrong.setdefault(name, []).append(t)
        if zeroed != 16 * sum(bodies):           # (a body sets each of its registers to zero once)
            wrong.setdefault(name, []).append(f"{zeroed} registers set to zero")
    assert not wrong, {n: w[:4] for n, w in wrong.items()}


def test_operands_are_ready_for_their_matrix_instructions(kernels):
    near = {name: found for name, lines in kernels.items() if (found := _too_near(lines))}
    assert not near, {n: f[:2] for n, f in near.items()}

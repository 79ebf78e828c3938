"""The tall tiles of the small-tile GEMM name some MFMAs by hand, and the compiler puts no wait states around those: the
distances have to be in the program that it makes of them.  Reads the assembly of this library's own source."""
import os
import re
import subprocess

import pytest

from paper_2507_18181_amd import build

WAIT = 19   # wait states from a 16-pass matrix result to any other access to it, the longest on this family
AHEAD = 2   # from a vector write to a matrix read


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """name -> lines (instruction, by hand or not) of the kernels with hand-written MFMAs."""
    out = str(tmp_path_factory.mktemp("mid") / "mid.s")
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-Wall")]
    subprocess.check_call([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + flags + ["--offload-device-only", "-S", "-o", out,
                          os.path.join(build.CSRC, "kernels_mid.hip")], stderr=subprocess.DEVNULL)
    found, name, hand = {}, None, False
    for line in open(out):
        line = line.split(";;#ASM")[0].strip() + (line[line.find(";;#ASM"):].strip() if ";;#ASM" in line else "")
        label = re.match(r"(_ZN7specasr15gemm_mid_kernel\w+):", line)
        if label:
            name = label.group(1)
            found[name] = []
        elif line.startswith(".Lfunc_end"):
            name = None
        elif line.startswith(";;#ASM"):
            hand = "START" in line
        elif name and re.match(r"[a-z]\w+( |$)|\.LBB", line):
            found[name].append((line.split(";")[0].strip(), hand))
    found = {n: ls for n, ls in found.items() if any(h and l.startswith("v_mfma") for l, h in ls)}
    assert len(found) == 4   # six and seven bands, partial sums and SwiGLU
    return found


def _regs(op):
    m = re.match(r"-?\|?([va])\[(\d+):(\d+)\]", op)
    if m:
        return {(m.group(1), i) for i in range(int(m.group(2)), int(m.group(3)) + 1)}
    m = re.match(r"-?\|?([va])(\d+)", op)
    return {(m.group(1), int(m.group(2)))} if m else set()


def _operands(line):
    return [_regs(o.strip()) for o in line.split(None, 1)[1].split(",")] if " " in line else []


def _states(line):
    """Wait states that an instruction takes at least."""
    m = re.match(r"s_nop (\d+)", line)
    return 1 + int(m.group(1)) if m else 1


def test_products_by_hand_stand_before_sixteen_others(kernels):
    """Per plane the hand-written products come first and the 16 others behind them, in straight code: whatever follows a
    step has these between itself and the hand-written results."""
    for name, lines in kernels.items():
        kind = "".join("h" if h else "c" if l.startswith("v_mfma") else "|" for l, h in lines
                       if l.startswith(("v_mfma", "s_cbranch", "s_branch", ".LBB")))
        tiles = int(re.search(r"ILi(\d)ELi3E", name).group(1)) * 3
        blocks = [b for b in re.split(r"\|+", kind) if b]
        assert blocks
        for b in blocks:
            assert re.fullmatch("(h{%d}c{16})+" % (tiles - 16), b), (name, b)


def test_nothing_touches_a_result_by_hand_too_early(kernels):
    """Along every straight run (branches take wait states too, and fall through is the nearest): no instruction but another
    MFMA on exactly the same accumulator comes within WAIT states of a hand-written product, and nothing writes an operand
    of one right in front of it."""
    for name, lines in kernels.items():
        for i, (line, hand) in enumerate(lines):
            if not (hand and line.startswith("v_mfma")):
                continue
            dst, a, b, c = _operands(line)
            assert dst == c
            states = 0
            for later, _ in lines[i + 1:]:
                if states >= WAIT or later.startswith(".LBB"):
                    break
                ops = _operands(later) if later.startswith(("v_", "ds_", "global_", "buffer_", "scratch_", "flat_")) else []
                if later.startswith("v_mfma"):
                    assert all(not (dst & o) or (k in (0, 3) and o == dst) for k, o in enumerate(ops)), (name, line, later)
                    states += 8   # an MFMA of 8 passes is behind the one before it in the one matrix pipe
                else:
                    assert not any(dst & o for o in ops), (name, line, later)
                    states += _states(later)
            states = 0
            for earlier, _ in reversed(lines[:i]):
                if states >= AHEAD or earlier.startswith(".LBB"):
                    break
                if earlier.startswith("v_") and not earlier.startswith("v_mfma"):
                    assert not (_operands(earlier)[0] & (a | b | c)), (name, earlier, line)
                states += _states(earlier)


def test_sums_wait_for_the_results(kernels):
    """In front of the LDS sums stands a wait that the accumulators depend on."""
    for name, lines in kernels.items():
        first_store = next(i for i, (l, _) in enumerate(lines) if l.startswith("ds_write_b128") and _operands(l)[1])
        nops = [i for i, (l, h) in enumerate(lines[:first_store]) if h and l.startswith("s_nop")]
        assert nops and sum(_states(lines[i][0]) for i in nops) >= WAIT, name
        assert not any(l.startswith("v_mfma") for l, _ in lines[nops[0]:first_store]), name

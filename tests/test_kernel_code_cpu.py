"""What the compiler made of the kernels, from the instructions of the built library, for what neither a result nor the
metadata shows: which loads are in flight together."""
import os
import re
import subprocess
import tempfile

import pytest

import paper_2410_18248_amd as P
from paper_2410_18248_amd import build
from test_kernel_resources_cpu import _code_objects, _metadata

OBJDUMP = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(build.HIPCC))), "llvm", "bin", "llvm-objdump")


def _code(part):
    """name -> (address, instruction) of the kernels whose code object has one with `part` in its name"""
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump beside hipcc")
    out = {}
    for co in _code_objects(open(P.lib_path(), "rb").read()):
        if not any(part in k[".name"] for k in _metadata(co)):
            continue
        with tempfile.NamedTemporaryFile(suffix=".o") as f:
            f.write(co)
            f.flush()
            text = subprocess.check_output([OBJDUMP, "-d", "--no-show-raw-insn", f.name], text=True)
        name = None
        for line in text.split("\n"):
            m = re.match(r"([0-9a-f]+) <(\S+)>:", line)
            if m:
                name, start = m.group(2), int(m.group(1), 16)
                out[name] = []
                continue
            m = re.match(r"\s+(.*\S)\s*// *([0-9A-F]+):(.*)", line)
            if name and m:
                out[name].append((int(m.group(2), 16) - start, m.group(1) + m.group(3)))
    return {n: x for n, x in out.items() if part in n}


@pytest.fixture(scope="module")
def balanced():
    """name -> instructions of the kernels of balanced decode launches"""
    out = {n: [i for _, i in x] for n, x in _code("decode_balanced").items() if "merge" not in n}
    assert len(out) == 30
    return out


def test_requests_of_a_lane_are_asked_for_together(balanced):
    """Batches of 65 to 256 are planned by waves that hold four requests per lane: eight loads, masks (bytes) and
    lengths, and one wait."""
    for name, code in balanced.items():
        runs, n = [], 0
        for x in code:
            if x.startswith("global_load_ubyte"):
                n += 1
            elif x.startswith("s_waitcnt") and "vmcnt" in x:
                runs.append(n)
                n = 0
        assert max(runs) >= 4, (name, sorted(runs)[-3:])


def test_the_plan_divides_by_32_bits(balanced):
    """General 64-bit divisions (2^64 as a float is a constant of each) are 120 instructions in front of the first byte:
    only the four for sequences of 2^31 chunks and more (two ends of a share, its range, and a range's last share)."""
    for name, code in balanced.items():
        assert sum("0x5f7ffffc" in x for x in code) <= 4, name


def test_where_loops_begin_in_a_fetch():
    """The loops of narrow tiles of heads of 64, whose time goes by that: the last backward branch over more than 600 bytes."""
    seen = 0
    for name, code in _code("prefill_mfma").items():
        m = re.search(r"prefill_mfmaILi64ELb(\d)ELi16ELi1ELb0E", name)
        if not m:
            continue
        begin = None
        for at, x in code:
            t = re.match(r"s_c?branch.*<\S+\+0x([0-9a-f]+)>", x)
            if t and int(t.group(1), 16) < at - 600:
                begin = int(t.group(1), 16)
        assert begin % 32 == 4, (name, begin % 32)
        seen += 1
    assert seen == 2


def test_teams_move_a_reference_without_lds():
    """All eight waves wait for the one whose reference point moves, which peaked scores make it do in most stages: lanes compare by register
    swaps, and inside the loop (from the first s_setprio 1 on) no product waits for the loads of operands behind its own."""
    seen = 0
    for name, code in _code("prefill_teams").items():
        text = [x for _, x in code]
        assert not any(x.startswith("ds_bpermute") for x in text), name
        at = next(k for k, x in enumerate(text) if x.startswith("s_setprio 1"))
        loop = text[at:at + next(k for k, x in enumerate(text[at:]) if x.startswith("s_setprio 0"))]
        assert sum(x.startswith("v_mfma") for x in loop) >= 32, name
        waits = [x for x in loop if "lgkmcnt" in x]
        assert waits and not any("lgkmcnt(0)" in x for x in waits[:len(waits) // 2]), (name, waits)
        seen += 1
    assert seen == 4

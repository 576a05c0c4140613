"""Wait states of the LDS-DMA loads, in the AMD assembly of this build.

The loads (buffer_load ... lds) are issued from inline assembly, which the
compiler's hazard pass does not look into, so the blocks carry the wait states
themselves. On GFX9 a VALU write of a scalar register (v_readfirstlane,
v_readlane: where the compiler takes a descriptor word out of a vector register
right before the block) needs 5 wait states before a vector-memory instruction
reads that register, and a scalar write of m0 needs 1 before an LDS-DMA load,
which takes its LDS address from m0. An instruction is one wait state, s_nop N
is N + 1. CPU only: compiles the sources that issue such loads for gfx950 and
walks back from every load."""
import os
import re
import shutil
import subprocess

import pytest

HAVE_HIPCC = shutil.which("hipcc") is not None or os.path.exists("/opt/rocm/bin/hipcc")
pytestmark = pytest.mark.skipif(not HAVE_HIPCC, reason="needs hipcc")

LOAD = re.compile(r"buffer_load_dwordx4 v\d+, s\[(\d+):(\d+)\], (\S+) offen.* lds$")


def instructions(asm):
    """The instructions of an assembly listing; None at each label."""
    out = []
    for line in asm.splitlines():
        line = line.split(";")[0].strip()
        if re.match(r"^[\w.$]+:", line):
            out.append(None)
        elif line and not line.startswith("."):
            out.append(line)
    return out


def wait_states(ins):
    m = re.match(r"s_nop (\d+)", ins)
    return int(m.group(1)) + 1 if m else 1


def scalar_dest(ins):
    """Scalar registers that a VALU instruction writes (its first operand; carry
    and compare results are the scalar pairs among the first two)."""
    if not ins.startswith("v_"):
        return set()
    regs = set()
    for op in ins.split(None, 1)[1].split(",")[:2]:
        m = re.fullmatch(r"s\[(\d+):(\d+)\]", op.strip())
        if m:
            regs |= set(range(int(m.group(1)), int(m.group(2)) + 1))
    m = re.match(r"v_\w+ s(\d+),", ins)
    return regs | ({int(m.group(1))} if m else set())


def valu_hazards(ins):
    """(index, load) of the loads that may read a scalar register fewer than 5 wait
    states after a VALU instruction wrote it (a label counts as such a write of
    every register: what jumps there is not looked at)."""
    bad, loads = [], 0
    for i, x in enumerate(ins):
        m = LOAD.match(x) if x else None
        if not m:
            continue
        loads += 1
        read = set(range(int(m.group(1)), int(m.group(2)) + 1))
        if re.fullmatch(r"s\d+", m.group(3)):
            read.add(int(m.group(3)[1:]))
        states = 0
        for y in reversed(ins[:i]):
            if states >= 5:
                break
            if y is None or scalar_dest(y) & read:
                bad.append((i, x))
                break
            states += wait_states(y)
    return bad, loads


def m0_hazards(ins):
    """The loads right after an instruction that writes m0 (or a label)."""
    loads = [i for i, x in enumerate(ins) if x and LOAD.match(x)]
    return [(i, ins[i - 1]) for i in loads
            if ins[i - 1] is None or re.match(r"s_\w+ m0,", ins[i - 1])]


@pytest.fixture(scope="module")
def listing(tmp_path_factory):
    """The gfx950 assembly of a source, compiled with the build's own flags."""
    from paper_2510_00207_amd import build
    out = tmp_path_factory.mktemp("asm")
    cache = {}

    def get(name):
        if name not in cache:
            s = out / (name + ".s")
            subprocess.run([build.hipcc(), *build.HIPCC_FLAGS, "--cuda-device-only", "-S",
                            os.path.join(build.CSRC, name + ".hip"), "-o", str(s)],
                           check=True, capture_output=True, timeout=600)
            cache[name] = instructions(s.read_text())
        return cache[name]

    return get


def test_checker_sees_the_hazard():
    load = "buffer_load_dwordx4 v1, s[4:7], 0 offen lds"
    near = ["v_readfirstlane_b32 s6, v9", "s_mov_b32 s12, m0", "s_mov_b32 m0, s81", load]
    assert valu_hazards(near) == ([(3, load)], 1)
    far = near[:3] + ["s_nop 2", load]
    assert valu_hazards(far) == ([], 1)
    assert valu_hazards([None, "s_nop 3", load]) == ([(2, load)], 1)
    assert valu_hazards([None, "s_nop 4", load]) == ([], 1)
    assert m0_hazards(near + [load]) == [(3, near[2])]
    assert m0_hazards(far) == []
    assert scalar_dest("v_cmp_gt_i32_e64 s[4:5], v1, v2") == {4, 5}
    assert scalar_dest("v_add_co_u32_e64 v1, s[8:9], v2, v3") == {8, 9}


@pytest.mark.parametrize("name", ["gemm", "attn"])
def test_descriptor_wait_states(listing, name):
    bad, loads = valu_hazards(listing(name))
    assert loads > 100, loads
    assert not bad, f"{len(bad)} of {loads} loads, the first: {bad[:3]}"


@pytest.mark.parametrize("name", ["gemm", "attn"])
def test_m0_wait_states(listing, name):
    bad = m0_hazards(listing(name))
    assert not bad, f"{len(bad)} loads, the first: {bad[:3]}"

"""CPU checks of waits in the built device code that no compiler pass adds for
instructions written as inline assembly.

A vector memory instruction may read a scalar register only five wait states
after a vector instruction (v_readfirstlane and the like) wrote it, and a load
into LDS reads m0 only one wait state after s_mov wrote it (AMD Instinct CDNA3
ISA, manually inserted wait states).  Each instruction counts as one wait
state, s_nop N as N + 1.  The compiler inserts what is missing around its own
instructions, not around inline assembly: the code objects inside libhqr.so
are disassembled and every vector memory instruction is checked.

Relaxed atomics of one lane to different words are not ordered either: in the
triangular solves spread over workgroups the published block count has to have
arrived before the workgroup counts itself done, because the last one to do so
zeroes the counts for the next solve.
"""
import os
import re
import struct
import subprocess

import pytest

OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
SGPR = re.compile(r"^s(\d+)$|^s\[(\d+):(\d+)\]$")


def code_objects(lib):
    """The gfx950 code objects bundled in a library."""
    data = open(lib, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, p)
            ident = data[p + 24:p + 24 + idlen].decode()
            p += 24 + idlen
            if "gfx950" in ident and size:
                yield data[at + off:at + off + size]
        at = data.find(MAGIC, at + 1)


def sgprs(operand):
    """Scalar registers named by an operand."""
    m = SGPR.match(operand)
    if operand == "vcc":
        return {"vcc"}
    if not m:
        return set()
    lo = int(m.group(1) or m.group(2))
    return set(range(lo, int(m.group(1) or m.group(3)) + 1))


def operands(ins):
    return [re.split(r"\s", o.strip())[0] for o in ins.partition(" ")[2].split(",")]


def vector_written(ins):
    """Scalar registers that a vector instruction writes: compares and lane
    reads in the first operand, carries and v_div_scale in the second."""
    op = operands(ins)
    out = sgprs(op[0])
    if len(op) > 1 and ("_co_" in ins or "div_scale" in ins):
        out |= sgprs(op[1])
    return out


def wait_states(ins):
    return int(ins.split()[1], 0) + 1 if ins.startswith("s_nop") else 1


def missing_waits(lines):
    """(instruction, writer, wait states between) of each vector memory
    instruction that comes too early, in a listing in program order."""
    bad = []
    for i, ins in enumerate(lines):
        name = ins.split(" ", 1)[0]
        if not name.startswith(("buffer_", "global_", "flat_", "scratch_")):
            continue
        to_lds = bool(re.search(r"\blds\b", ins))
        read = set().union(*[sgprs(o) for o in operands(ins)])
        between = 0
        for prev in reversed(lines[max(0, i - 5):i]):
            if between >= 5 or is_label(prev):
                break
            if prev.startswith("v_") and vector_written(prev) & read:
                bad.append((ins, prev, between))
                break
            if to_lds and between < 1 and prev.startswith("s_") and operands(prev)[0] == "m0":
                bad.append((ins, prev, between))
                break
            between += wait_states(prev)
    return bad


def listing(path):
    text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", path], check=True,
                          capture_output=True, text=True).stdout
    out = []
    for line in text.splitlines():
        line = line.split("//")[0].strip()
        if not line:
            continue
        out.append(line)
    return out


def is_label(line):
    return line.startswith("<") and line.endswith(">:")


def functions(lines):
    """(name, instructions) of each function of a listing."""
    at = [i for i, s in enumerate(lines) if is_label(s)] + [len(lines)]
    return [(lines[a], lines[a + 1:b]) for a, b in zip(at, at[1:])]


def test_the_check_sees_a_missing_wait():
    load = "buffer_load_dwordx4 v1, s[4:7], 0 offen sc1 lds"
    for n, ok in ((0, False), (2, False), (3, True)):
        assert bool(missing_waits(["v_readfirstlane_b32 s4, v28", "s_mov_b32 m0, s0", "s_nop %d" % n, load])) != ok
    assert missing_waits(["s_mov_b32 m0, s0", load])
    assert not missing_waits(["v_readfirstlane_b32 s8, v28", "s_mov_b32 m0, s0", "s_nop 0", load])
    assert missing_waits(["v_cmp_eq_u32_e64 s[6:7], v0, v1", "s_nop 1", load])
    assert not missing_waits(["v_mfma_f64_16x16x4_f64 a[4:7], v[0:1], v[2:3], a[4:7]", load.replace("s[4:7]", "s[8:11]")])


@pytest.fixture(scope="module")
def listings(hqr_lib, tmp_path_factory):
    from paper_1110_1553_amd import _lib

    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    out = []
    for k, obj in enumerate(code_objects(_lib.LIB_PATH)):
        path = str(tmp_path_factory.mktemp("isa") / ("%d.o" % k))
        with open(path, "wb") as f:
            f.write(obj)
        out.append(listing(path))
    return out


def test_vector_memory_after_vector_written_scalars(listings):
    loads = 0
    for lines in listings:
        loads += sum(1 for s in lines if s.startswith("buffer_load") and re.search(r"\blds\b", s))
        bad = missing_waits(lines)
        assert not bad, "%d of %d instructions, first: %s" % (len(bad), len(lines), bad[:3])
    assert loads > 0  # the loads into LDS were found


def test_block_count_arrives_before_done(listings):
    # the ticket and the done count are the only counted atomics of these kernels; the done count comes last
    seen = 0
    for lines in listings:
        for name, body in functions(lines):
            if "trsv_chain_kernel" not in name and "ir_trsv_kernel" not in name:
                continue
            seen += 1
            adds = [i for i, s in enumerate(body) if s.startswith("global_atomic_add")]
            assert len(adds) == 2, (name, [body[i] for i in adds])
            before = [s for s in body[:adds[1]] if s.startswith(("global_store", "s_waitcnt")) and
                      (s.startswith("global_store") or "vmcnt(0)" in s)]
            assert before[-1].startswith("s_waitcnt"), (name, before[-1])
    assert seen >= 9  # three tile sizes of the solve, R and R^T of the refinement


def test_staged_panels_are_waited_for(listings):
    # a barrier hands over what the loads into LDS in front of it have staged: a vmcnt wait lies between.  The one
    # barrier inside a panel of the left-looking update (nb > 64) comes while the next panel is on its way.
    seen = 0
    for lines in listings:
        for name, body in functions(lines):
            if not re.search("update_task|apply_task|panel_task", name):
                continue
            at = [-1] + [i for i, s in enumerate(body) if s.startswith("s_barrier")]
            unwaited = 0
            for a, b in zip(at, at[1:]):
                loads = [i for i in range(a + 1, b) if body[i].startswith("buffer_load") and
                         re.search(r"\blds\b", body[i])]
                if loads:
                    seen += 1
                    unwaited += not any("vmcnt" in s for s in body[loads[-1]:b])
            assert unwaited <= (1 if "panel_task" in name else 0), name
    assert seen > 100

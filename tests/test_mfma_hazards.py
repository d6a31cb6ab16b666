"""What the tile kernel relies on, read from the assembly of the built library (no GPU).  Its matrix instructions are inline
assembly, so the compiler does not keep the distances that their operands and results need: an accumulator is touched by
nothing but the next MFMA on it until every pass of the last one is over, and an operand is not written by a vector
instruction right ahead.  And its logit pieces rely on the bounds check of their buffers."""
import re
import shutil
import subprocess

import pytest

import paper_2605_18817_amd.build as hip_build

OBJDUMP = shutil.which("llvm-objdump") or shutil.which("llvm-objdump", path="/opt/rocm/llvm/bin")
RESULT_SLOTS = 18      # instructions or wait states until a 16-pass result may be read or overwritten
SOURCE_SLOTS = 2       # between a vector instruction's write and the MFMA that reads it


def _registers(token):
    m = re.fullmatch(r"([av])\[(\d+):(\d+)\]", token)
    if m:
        return {(m[1], r) for r in range(int(m[2]), int(m[3]) + 1)}
    m = re.fullmatch(r"([av])(\d+)", token)
    return {(m[1], int(m[2]))} if m else set()


def _kernels(text, name):
    """name -> [(address, opcode, operands)] of the functions whose symbol holds `name`."""
    out, cur = {}, None
    for ln in text.splitlines():
        m = re.match(r"^[0-9a-f]+ <(\S+)>:", ln)
        if m:
            cur = out.setdefault(m[1], []) if name in m[1] and not m[1].endswith(".kd") else None
            continue
        m = re.match(r"^\s+([a-z]\S*)\s*(.*?)\s*// ([0-9A-F]+):", ln)
        if m and cur is not None:
            cur.append((int(m[3], 16), m[1], [t.strip() for t in m[2].split(",")] if m[2] else []))
    return out


def _target(addr, op, ops):
    """Address that a scalar branch goes to, or None."""
    if op != "s_branch" and not op.startswith("s_cbranch"):
        return None
    off = int(ops[0])
    return addr + 4 + 4 * (off - 65536 if off >= 32768 else off)


def _faults(ins):
    at = {a: n for n, (a, _, _) in enumerate(ins)}
    found = []

    def walk(n, end, result, source, slot, follow):
        while n < end and n < len(ins):
            addr, op, ops = ins[n]
            slot += int(ops[0], 0) + 1 if op == "s_nop" else 1
            regs = [r for t in ops for r in _registers(t.split()[0] if t else "")]
            if op.startswith("v_mfma"):
                dst = _registers(ops[0])
                for t in ops[1:3]:
                    if any(slot - source.get(r, -99) <= SOURCE_SLOTS for r in _registers(t)):
                        found.append((hex(addr), op, ops, "operand written right ahead"))
                    if any(slot - result.get(r, -99) < RESULT_SLOTS for r in _registers(t)):
                        found.append((hex(addr), op, ops, "operand is a result in flight"))
                if _registers(ops[3]) != dst and any(slot - result.get(r, -99) < RESULT_SLOTS for r in _registers(ops[3])):
                    found.append((hex(addr), op, ops, "another result in flight as addend"))
                for r in dst:
                    result[r] = slot
            else:
                if any(slot - result.get(r, -99) < RESULT_SLOTS for r in regs):
                    found.append((hex(addr), op, ops, "result in flight"))
                if op.startswith("v_") and ops:
                    for r in _registers(ops[0]):
                        source[r] = slot
            target = at.get(_target(addr, op, ops)) if follow else None
            if target is not None:       # (what follows where a branch goes, as far as a result may be in flight)
                walk(target, target + RESULT_SLOTS, dict(result), dict(source), slot, False)
            n += 1

    walk(0, len(ins), {}, {}, 0, True)
    return found


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if OBJDUMP is None:
        pytest.skip("no llvm-objdump")
    hip_build.build(force=False)
    folder = tmp_path_factory.mktemp("lib")
    lib = folder / "lib.so"
    shutil.copy(hip_build.LIB, lib)
    subprocess.run([OBJDUMP, "--offloading", str(lib)], check=True, stdout=subprocess.DEVNULL, cwd=folder)
    found = {}
    for image in sorted(folder.glob("lib.so.*gfx950*")):
        text = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", str(image)], check=True, stdout=subprocess.PIPE, text=True).stdout
        found.update(_kernels(text, "tiled_gemm_kernel"))
    assert len(found) >= 60
    return found


def test_matrix_instructions_keep_their_distances(kernels):
    for name, ins in kernels.items():
        assert sum(op.startswith("v_mfma") for _, op, _ in ins) >= 200, name
        assert not _faults(ins), (name, _faults(ins)[:4])


def test_buffer_bounds_see_the_whole_offset(kernels):
    """A raw buffer's bounds check compares the lane's offset with the buffer's size; a scalar offset comes on top of it
    unchecked.  So rows that are not there have to be missing from the buffer's size, and the scalar offset is zero."""
    pieces = [(name, op, ops) for name, ins in kernels.items() for _, op, ops in ins if op.startswith("buffer_")]
    assert len(pieces) >= 2000
    wrong = [p for p in pieces if p[2][3].split() != ["0", "offen"]]
    assert not wrong, (len(wrong), wrong[:3])

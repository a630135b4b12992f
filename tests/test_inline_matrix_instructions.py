"""What prefill256.hip's inline matrix instructions rely on, looked up in the library that was built: the compiler takes no
part of those kernels' registers to scratch, and puts no vector instruction so close to an inline matrix instruction that the
hardware would need a wait in between -- it inserts such waits around its own matrix instructions only."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2511_10676_amd import build

LLVM = "/opt/rocm/llvm/bin"
INTO = 2       # wait states between a vector instruction and a matrix instruction that reads its result
OUT_OF = 12    # and between a 16x16x32 product (at most 8 passes) and anything but a product onto the same sum


@pytest.fixture(scope="module")
def code_object(tmp_path_factory):
    if not (os.path.exists(os.path.join(LLVM, "llvm-objdump")) and os.path.exists(build.LIB)):
        pytest.skip("no llvm-objdump, or the library is not built")
    tmp = tmp_path_factory.mktemp("code")
    shutil.copy(build.LIB, tmp / "lib.so")                   # the code objects are written beside their library
    subprocess.run([f"{LLVM}/llvm-objdump", "--offloading", "lib.so"], cwd=tmp, check=True, capture_output=True)
    found = [f for f in tmp.iterdir() if f.name.endswith("gfx950") and b"prefill256_kernel" in f.read_bytes()]
    assert len(found) == 1
    return found[0]


def _registers(operand):
    m = re.match(r"^([va])(?:\[(\d+):(\d+)\]|(\d+))$", operand)
    if not m:
        return frozenset()
    lo = int(m[2] or m[4])
    return frozenset((m[1], i) for i in range(lo, int(m[3] or lo) + 1))


def _kernels(text):
    """name -> [(operation, [registers of each operand], immediate of s_nop)]"""
    out, cur = {}, None
    for line in text.splitlines():
        if head := re.match(r"^[0-9a-f]+ <(\S+)>:$", line):
            cur = out.setdefault(head[1], [])
        elif cur is not None and (m := re.match(r"^\s+(\w+)\s*(.*?)\s*//", line)):
            ops = [o.strip().split(" ")[0] for o in m[2].split(",")]
            cur.append((m[1], [_registers(o) for o in ops], int(ops[0], 0) if m[1] == "s_nop" else 0))
    return out


def hazards(code):
    """Pairs of instructions that stand too close, in the order of the listing."""
    bad, recent = [], []                                     # recent: (operation, registers, states since)
    for op, regs, nop in code:
        product = op.startswith("v_mfma")
        touched = frozenset().union(*regs)
        for old, old_regs, since in recent:
            if old.startswith("v_mfma"):
                sums = old_regs[0]
                onto = product and regs[0] == sums and regs[3] in (sums, frozenset())
                reads = regs[1] | regs[2] if product else touched
                if since < OUT_OF and (reads & sums or (product and not onto and (regs[0] | regs[3]) & sums)):
                    bad.append((old, op, since))
            elif product and since < INTO and old_regs[0] & (regs[1] | regs[2] | regs[3]):
                bad.append((old, op, since))
        states = nop + 1
        recent = [(o, r, s + states) for o, r, s in recent if s + states < OUT_OF]
        if op.startswith("v_"):
            recent.append((op, regs, 0))
    return bad


def test_hazards_are_found():
    v, a = (lambda *i: frozenset(("v", j) for j in i)), (lambda *i: frozenset(("a", j) for j in i))
    mfma = ("v_mfma_f32_16x16x32_bf16", [a(0, 1, 2, 3), v(0, 1, 2, 3), v(4, 5, 6, 7), a(0, 1, 2, 3)], 0)
    mov, read, nop = ("v_mov_b32_e32", [v(5), v(9)], 0), ("v_accvgpr_read_b32", [v(8), a(2)], 0), lambda n: ("s_nop", [frozenset()], n)
    assert hazards([mov, mfma]) and hazards([mov, nop(0), mfma]) and not hazards([mov, nop(1), mfma])
    assert hazards([mfma, read]) and hazards([mfma, nop(10), read]) and not hazards([mfma, nop(15), read])
    other = (mfma[0], [a(4, 5, 6, 7), v(0, 1, 2, 3), v(4, 5, 6, 7), a(0, 1, 2, 3)], 0)
    assert not hazards([mfma, mfma]) and hazards([mfma, other]) and hazards([mfma, ("ds_write_b128", [v(20), a(0, 1, 2, 3)], 0)])


def test_no_vector_instruction_crowds_an_inline_matrix_instruction(code_object):
    text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", str(code_object)], check=True, capture_output=True, text=True).stdout
    seen = 0
    for name, code in _kernels(text).items():
        if "prefill256_kernel" not in name:
            continue
        seen += 1
        assert sum(op == "v_mfma_f32_16x16x32_bf16" for op, _, _ in code) >= 64
        assert not hazards(code), (name, hazards(code)[:5])
    assert seen >= 20


def test_prefill256_keeps_its_registers(code_object):
    notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", str(code_object)], check=True, capture_output=True, text=True).stdout
    kernels = [k for k in re.split(r"\n\s+- \.agpr_count:", notes)[1:] if "prefill256_kernel" in k]
    assert len(kernels) >= 20
    for k in kernels:
        name = re.search(r"\.symbol:\s+(\S+)", k)[1]
        assert re.search(r"\.private_segment_fixed_size: 0\n", k) and re.search(r"\.vgpr_spill_count: 0\n", k), name

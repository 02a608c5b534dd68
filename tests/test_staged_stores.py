"""What the build made of the kernels that pass their output through LDS, read from the library's own code: a 16-byte LDS store keeps two
wait states between itself and the next write to the registers it stores, and operand reads that the compiler does not know to be under
way are waited for before it has registers of its own to place."""
import os
import re
import struct
import subprocess

import pytest

from paper_2602_22592_amd import binding as pq

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
pytestmark = pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")


def disassemble(path, fragments, tmp):
    """{mangled name: its instructions} of the library's gfx950 kernels whose names hold one of the fragments."""
    data, out = open(path, "rb").read(), {}
    at = data.find(b"\x7fELF", 1)
    while at >= 0:
        if struct.unpack_from("<H", data, at + 18)[0] == 224:          # EM_AMDGPU
            shoff, = struct.unpack_from("<Q", data, at + 40)
            size, n = struct.unpack_from("<HH", data, at + 58)
            blob = data[at:at + shoff + size * n]
            if any(f.encode() in blob for f in fragments):
                tmp.write_bytes(blob)
                name = None
                for line in subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", str(tmp)], capture_output=True, text=True,
                                           check=True).stdout.splitlines():
                    if m := re.match(r"(?:[0-9a-f]+ )?<(\S+)>:", line):
                        name = m[1] if any(f in m[1] for f in fragments) else None
                        if name:
                            out[name] = []
                    elif name and line.startswith("\t"):
                        out[name].append(line.split("//")[0].strip())
        at = data.find(b"\x7fELF", at + 1)
    return out


def registers(operand):
    """The vector registers of an operand: ("v" or "a", number)."""
    m = re.match(r"([va])\[(\d+):(\d+)\]$", operand)
    if m:
        return {(m[1], i) for i in range(int(m[2]), int(m[3]) + 1)}
    m = re.match(r"([va])(\d+)$", operand)
    return {(m[1], int(m[2]))} if m else set()


def operands(instruction):
    op, _, rest = instruction.partition(" ")
    return op, [o.strip().split(" ")[0] for o in rest.split(",")]


STAGED = ["fixed_gemm_kernel", "16mfma_gemm_kernel", "gemm_tn_w4_kernel", "gemm_tn_192_kernel", "tile64_gemm_kernel", "tile64_grads_kernel", "tile_set_kernel"]


@pytest.fixture(scope="module")
def code(tmp_path_factory):
    if not os.path.exists(pq.LIB_PATH):
        from paper_2602_22592_amd.build import build
        build(verbose=False)
    return disassemble(pq.LIB_PATH, STAGED, tmp_path_factory.mktemp("code") / "object.elf")


@pytest.mark.parametrize("kernel", STAGED)
def test_registers_outlive_their_store(code, kernel):
    kernels = {n: ins for n, ins in code.items() if kernel in n}
    assert kernels
    stores = 0
    for name, ins in kernels.items():
        for i, x in enumerate(ins):
            op, args = operands(x)
            if op != "ds_write_b128":
                continue
            stores += 1
            held, states = registers(args[1]), 0
            for y in ins[i + 1:i + 3]:
                op, args = operands(y)
                if op == "s_nop":
                    states += int(args[0], 0)
                elif op.startswith("v_") and states < 2:
                    assert not registers(args[0]) & held, (name, x, y)
                states += 1
    assert stores


def test_operand_reads_land_before_the_output_is_formed(code):
    """The digit products read the next tile's operands with asm statements ahead of the output's conversion to fp64, which the compiler
    arranges: a register it copied or spilled there would be one that the read has not yet written."""
    (name, ins), = [k for k in code.items() if "fixed_gemm_kernel" in k[0]]
    pending, converted, reads = set(), 0, 0
    for x in ins:
        op, args = operands(x)
        if op == "ds_read_b128":
            pending |= registers(args[0])
            reads += 1
        elif op == "s_waitcnt" and "lgkmcnt(0)" in x:
            pending = set()
        elif op == "v_cvt_f64_i32_e32":
            converted += 1
            assert not pending, (name, x, sorted(pending))
        else:
            assert not pending & set().union(*map(registers, args)), (name, x)
    assert reads and converted

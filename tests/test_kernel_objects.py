"""What the compiler made of the kernels, read from the code object of the built library: how a
kernel gets its arguments and how large its argument segment is."""
import re
import struct
import subprocess

import pytest

from paper_2312_10351_amd import binding as B

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


@pytest.fixture(scope="module")
def code_object(tmp_path_factory):
    B.load()
    data = open(B.LIB_PATH, "rb").read()
    at = data.index(b"__CLANG_OFFLOAD_BUNDLE__")
    n, = struct.unpack_from("<Q", data, at + 24)
    p, found = at + 32, []
    for _ in range(n):
        off, size, length = struct.unpack_from("<QQQ", data, p)
        name = data[p + 24:p + 24 + length]
        p += 24 + length
        if name.endswith(b"gfx950") and size:
            found.append(data[at + off:at + off + size])
    assert len(found) == 1
    path = tmp_path_factory.mktemp("co") / "kernels.elf"
    path.write_bytes(found[0])
    return path


def descriptors(path):
    """{kernel: its 64-byte descriptor}"""
    image = path.read_bytes()
    sections = subprocess.run([READELF, "-S", "-W", str(path)], check=True, capture_output=True, text=True).stdout
    shift = {int(i): int(off, 16) - int(addr, 16)
             for i, addr, off in re.findall(r"\[ *(\d+)\] \S+ +PROGBITS +([0-9a-f]+) ([0-9a-f]+)", sections)}
    symbols = subprocess.run([READELF, "-s", "-W", str(path)], check=True, capture_output=True, text=True).stdout
    out = {}
    for addr, index, name in re.findall(r"^ *\d+: ([0-9a-f]+) +64 OBJECT +\w+ +\w+ +(\d+) (opara_k_\w+)\.kd$", symbols, re.M):
        begin = int(addr, 16) + shift[int(index)]
        out[name] = image[begin:begin + 64]
    return out


def test_no_kernel_takes_arguments_from_two_places(code_object):
    """Arguments come from the argument segment only: a workgroup that finds its member of a group
    from preloaded registers and reads the member's record from memory would store out of bounds if
    the two ever disagreed."""
    found = descriptors(code_object)
    assert {"opara_k_group_f16_heavy", "opara_k_attention_f16", "opara_k_token"} <= set(found)
    preloaded = {k: struct.unpack_from("<H", d, 58)[0] & 127 for k, d in found.items()}
    assert not any(preloaded.values()), {k: v for k, v in preloaded.items() if v}


def segments(path):
    """{kernel: (bytes of its argument segment, kinds of its arguments)}"""
    notes = subprocess.run([READELF, "--notes", str(path)], check=True, capture_output=True, text=True).stdout
    out = {}
    for block in re.split(r"\n  - \.agpr_count:|\n  - \.args:", notes)[1:]:
        name = re.search(r"^    \.name: +(opara_k_\w+)$", block, re.M)
        if name:
            out[name.group(1)] = (int(re.search(r"\.kernarg_segment_size: (\d+)", block).group(1)), re.findall(r"\.value_kind: +(\w+)", block))
    return out


def test_a_marker_node_has_room_for_every_kernel_it_may_be_switched_to(code_object):
    """A node of the multi-stream graph is made with the marker kernel and later switched to its
    operator's kernel in place: the argument block that the runtime holds for the node must be
    large enough for it, implicit arguments included."""
    found = segments(code_object)
    count = B.opara_kernel_count()
    planned = ["opara_k_" + B.opara_kernel_info(i)[0] for i in range(count)]
    assert set(planned) <= set(found)
    room = found["opara_k_token"][0]
    assert {k: found[k][0] for k in planned if found[k][0] > room} == {}
    assert {k for k in planned if any(kind.startswith("hidden") for kind in found[k][1])} == set()


def scalar_registers(operand):
    run = re.fullmatch(r"s\[(\d+):(\d+)\]", operand)
    if run:
        return set(range(int(run.group(1)), int(run.group(2)) + 1))
    return {int(operand[1:])} if re.fullmatch(r"s\d+", operand) else set()


def test_memory_instructions_wait_for_scalar_registers_that_vector_instructions_write(code_object):
    """A memory instruction may read a scalar register five wait states after a vector instruction
    wrote it, and a load to workgroup memory m0 one after a scalar instruction did.  The compiler
    sees to that for its own instructions, but does not look into inline assembly."""
    text = subprocess.run(["/opt/rocm/llvm/bin/llvm-objdump", "-d", "--no-show-raw-insn", str(code_object)], check=True, capture_output=True, text=True).stdout
    loads, at, written, m0 = 0, 0, {}, -9
    for line in text.splitlines():
        line = line.split("//")[0].strip()
        if line.endswith(">:"):
            written = {}
        op, _, rest = line.partition(" ")
        operands = rest.replace(",", " ").split()
        nop = re.fullmatch(r"s_nop (\d+)", line)
        at += int(nop.group(1)) + 1 if nop else 1
        if op.startswith(("v_readfirstlane", "v_readlane", "v_cmp")) and operands:
            written.update({r: at for r in scalar_registers(operands[0])})
        elif op.startswith(("buffer_", "global_", "flat_")):
            read = set().union(*map(scalar_registers, operands))
            assert not {r for r in read if at - written.get(r, -9) <= 5}, line
            if operands[-1:] == ["lds"]:
                loads += 1
                assert at - m0 >= 2, line
        elif operands[:1] == ["m0"]:
            m0 = at
    assert loads > 1000

"""The kernels of the built library, from the metadata that the compiler puts
beside their code: how many bytes of scratch memory a lane takes, and whether
the kernels built are those that a dispatch can reach."""
import os
import re
import struct
import subprocess

import pytest

msgpack = pytest.importorskip("msgpack")

from paper_2609_08384_amd.build import LIB  # noqa: E402

BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"
NOTE_SECTION, AMDGPU_METADATA = 7, 32


def _code_objects(data):
    """The gfx950 ELF images of every offload bundle in the library."""
    pos = data.find(BUNDLE)
    while pos >= 0:
        count, = struct.unpack_from("<Q", data, pos + 24)
        at = pos + 32
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, at)
            triple = data[at + 24:at + 24 + length]
            at += 24 + length
            if b"gfx950" in triple and size:
                yield data[pos + offset:pos + offset + size]
        pos = data.find(BUNDLE, pos + len(BUNDLE))


def _kernels(elf):
    """The kernel records of one ELF image's metadata note."""
    table, = struct.unpack_from("<Q", elf, 0x28)
    entry, count = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(count):
        kind, = struct.unpack_from("<I", elf, table + i * entry + 4)
        if kind != NOTE_SECTION:
            continue
        at, size = struct.unpack_from("<QQ", elf, table + i * entry + 0x18)
        end = at + size
        while at < end:
            name, desc, note = struct.unpack_from("<III", elf, at)
            at += 12 + (name + 3) // 4 * 4
            if note == AMDGPU_METADATA:
                yield from msgpack.unpackb(elf[at:at + desc], strict_map_key=False)["amdhsa.kernels"]
            at += (desc + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(LIB):
        pytest.skip("library not built")
    with open(LIB, "rb") as fh:
        data = fh.read()
    # (name, integer template arguments) -> record; names are mangled as
    # brahms::<name><int, ...>(...)
    out = {}
    for elf in _code_objects(data):
        for k in _kernels(elf):
            k["elf"] = elf
            m = re.match(r"_ZN6brahms\d+([a-z0-9_]+?)I((?:Li\d+E)+)E", k[".name"])
            name = m.group(1) if m else k[".name"]
            args = tuple(int(v) for v in re.findall(r"Li(\d+)E", m.group(2))) if m else ()
            out[name, args] = k
    assert len(out) > 1000
    return out


# bytes of scratch memory a lane may take: eight registers
SCRATCH = 32


@pytest.mark.parametrize("family", ["axis_pass", "axis_pass_batched", "axis_pass_split", "axis_pass_split_batched",
                                    "line_steps", "line_steps_batched", "adjoint_pass", "adjoint_pass_together"])
def test_passes_keep_their_values_in_registers(kernels, family):
    mine = {args: k[".private_segment_fixed_size"] for (name, args), k in kernels.items() if name == family}
    assert mine
    assert not {args: size for args, size in mine.items() if size > SCRATCH}


def test_no_kernel_without_a_dispatch(kernels):
    """Both half-steps in one pass (mode 3) run on one line, which takes the
    one-field-per-thread kernel; the adjoint takes the first split of a
    length only."""
    assert not [args for (name, args) in kernels if name == "axis_pass" and args[4] & 3 == 3]
    with open(os.path.join(os.path.dirname(LIB), "csrc", "lengths.hpp")) as fh:
        first = re.search(r"#define BRAHMS_LENGTHS\(X\)(.*?)\n\n", fh.read(), re.S).group(1)
    splits = {(int(a), int(b)) for a, b in re.findall(r"X\(\d+, (\d+), (\d+)\)", first)}
    assert len(splits) == 21
    assert {args[:2] for (name, args) in kernels if name == "adjoint_pass"} == splits


OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.mark.parametrize("split", [(16, 8), (8, 8), (12, 4), (24, 8), (9, 1)])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_tables_are_asked_for_before_the_fields(kernels, split, axis, tmp_path):
    """Linear passes: the loads of the step's tables (global) are issued ahead
    of those of the fields (buffer), none behind them; waiting for the tables,
    which the first barrier needs, then does not wait for the fields."""
    if not os.path.exists(OBJDUMP):
        pytest.skip("no disassembler")
    k = kernels["axis_pass", (*split, axis, 1, 0, 256)]
    path = tmp_path / "unit.elf"
    path.write_bytes(k["elf"])
    asm = subprocess.run([OBJDUMP, "-d", "--disassemble-symbols=" + k[".name"], str(path)], capture_output=True,
                         text=True, check=True).stdout
    loads = re.findall(r"\t(global_load|buffer_load|s_barrier)", asm)
    loads = loads[:loads.index("s_barrier")]
    assert loads.count("global_load") >= 2 and loads.count("buffer_load") == split[0]
    assert "global_load" not in loads[loads.index("buffer_load"):]

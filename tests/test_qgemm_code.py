"""What the fast kernels of the quantized layer were compiled to, read from the library that was built here: properties that
no result shows and that a change of the source loses easily."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2302_01382_amd import build

LLVM = "/opt/rocm/llvm/bin"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _tool(name):
    return shutil.which(name) or shutil.which(name, path=LLVM)


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    """The gfx950 code objects with fast kernels, one per translation unit, as files."""
    if not _tool("llvm-readelf") or not _tool("llvm-objdump"):
        pytest.skip("no LLVM tools")
    with open(build.LIB, "rb") as f:
        data = f.read()
    out, at = [], data.find(MAGIC)
    while at >= 0:
        pos = at + len(MAGIC) + 8
        for _ in range(struct.unpack_from("<Q", data, at + len(MAGIC))[0]):
            offset, size, name = struct.unpack_from("<QQQ", data, pos)
            target = data[pos + 24:pos + 24 + name]
            pos += 24 + name
            elf = data[at + offset:at + offset + size]
            if b"gfx950" in target and (b"qgemm_dma" in elf or b"qgemm_quad" in elf):
                path = tmp_path_factory.mktemp("code") / ("%d.elf" % len(out))
                path.write_bytes(elf)
                out.append(str(path))
        at = data.find(MAGIC, at + 1)
    assert len(out) == 4  # the tiles of 256, 192, 128 and 64
    return out


def test_no_register_of_a_fast_kernel_is_spilled(code_objects):
    """A reload waits for every load and store in flight (s_waitcnt vmcnt(0)): at the head of an output tile for the
    stores of the one before it, in the k loop for the prefetch."""
    kernels, spilled = 0, []
    for path in code_objects:
        notes = subprocess.run([_tool("llvm-readelf"), "--notes", path], stdout=subprocess.PIPE, text=True, check=True).stdout
        for part in notes.split("- .agpr_count:")[1:]:
            name = re.search(r"^\s+\.name:\s+(\S+)", part, re.M).group(1)
            if "qgemm" not in name:
                continue
            kernels += 1
            count = int(re.search(r"\.vgpr_spill_count:\s+(\d+)", part).group(1))
            scratch = int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", part).group(1))
            if count or scratch:
                spilled.append((name, count, scratch))
    assert kernels >= 4 * 16 and not spilled, spilled


def test_the_first_barrier_waits_for_the_first_k_tile_only(code_objects):
    """The kernels request NSTAGE k tiles and wait for the first with a counted vmcnt: a vmcnt(0) between the requests and
    the first barrier, as the compiler puts behind an ordinary load, waits for all of them."""
    kernels, full = 0, []
    for path in code_objects:
        text = subprocess.run([_tool("llvm-objdump"), "-d", "--no-show-raw-insn", "--no-leading-addr", path],
                              stdout=subprocess.PIPE, text=True, check=True).stdout
        for part in re.split(r"^(?=\S*<\S+>:$)", text, flags=re.M):
            name = re.match(r"\S*<(\S+)>:$", part, re.M)
            if not name or not re.search("qgemm_(dma|quad)", name.group(1)):
                continue
            kernels += 1
            start = part[part.index("global_load_lds_"):]
            waits = re.findall(r"vmcnt\((\d+)\)", start[:start.index("s_barrier")])
            assert waits, name.group(1)  # the counted one
            if "0" in waits:
                full.append(name.group(1))
    assert kernels >= 4 * 16 and not full, full

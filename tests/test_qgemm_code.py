"""What the kernels of the quantized layer were compiled to, read from the library that was built here: properties that
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
    """The gfx950 code objects of the library, one per translation unit, as (contents, file)."""
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
            if b"gfx950" in target:
                path = tmp_path_factory.mktemp("code") / ("%d.elf" % len(out))
                path.write_bytes(elf)
                out.append((elf, str(path)))
        at = data.find(MAGIC, at + 1)
    return out


def _metadata(code_objects, kernel):
    """(name, its metadata) of every kernel whose name contains `kernel`."""
    for elf, path in code_objects:
        if kernel.encode() not in elf:
            continue
        notes = subprocess.run([_tool("llvm-readelf"), "--notes", path], stdout=subprocess.PIPE, text=True, check=True).stdout
        for part in notes.split("- .agpr_count:")[1:]:
            name = re.search(r"^\s+\.name:\s+(\S+)", part, re.M).group(1)
            if kernel in name:
                yield name, {k: int(v) for k, v in re.findall(r"^\s+\.(\w+):\s+(\d+)$", part, re.M)}


def test_no_register_of_a_fast_kernel_is_spilled(code_objects):
    """A reload waits for every load and store in flight (s_waitcnt vmcnt(0)): at the head of an output tile for the
    stores of the one before it, in the k loop for the prefetch."""
    kernels = list(_metadata(code_objects, "qgemm_"))
    spilled = [n for n, m in kernels if m["vgpr_spill_count"] or m["private_segment_fixed_size"]]
    assert len(kernels) >= 4 * 16 + 48 and not spilled, spilled


def test_four_workgroups_of_the_any_alignment_kernel_share_a_cu(code_objects):
    """Its 64 tile: four waves a workgroup, a SIMD's 512 registers over four of them."""
    kernels = list(_metadata(code_objects, "qgemm_anyILi64E"))
    over = [(n, m["vgpr_count"]) for n, m in kernels if m["vgpr_count"] > 128 or 4 * m["group_segment_fixed_size"] > 160 * 1024]
    assert len(kernels) == 24 and not over, over


def test_the_first_barrier_waits_for_the_first_k_tile_only(code_objects):
    """The kernels request NSTAGE k tiles and wait for the first with a counted vmcnt: a vmcnt(0) between the requests and
    the first barrier, as the compiler puts behind an ordinary load, waits for all of them."""
    kernels, full = 0, []
    for elf, path in code_objects:
        if b"qgemm_dma" not in elf and b"qgemm_quad" not in elf:
            continue
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


def _instructions(path):
    """(kernel, its instructions as (address, text, address of the branch's target or None)) of a code object."""
    text = subprocess.run([_tool("llvm-objdump"), "-d", path], stdout=subprocess.PIPE, text=True, check=True).stdout
    for part in re.split(r"^(?=[0-9a-f]+ <\S+>:$)", text, flags=re.M):
        head = re.match(r"([0-9a-f]+) <(\S+)>:$", part, re.M)
        if not head:
            continue
        found = re.findall(r"^\t(.+?)\s*// ([0-9A-F]+):[0-9A-F ]+(?:<\S+?\+0x([0-9a-f]+)>|<\S+>)?$", part, re.M)
        yield head.group(2), [(int(at, 16), op, int(head.group(1), 16) + int(to, 16) if to else None) for op, at, to in found]


def test_the_last_output_tile_is_stored_without_waiting_for_requests(code_objects):
    """Behind a workgroup's last k tile only zeros are still on their way into the LDS: there is a way from the last matrix
    step to the epilogue's first access of memory without a vmcnt(0)."""
    kernels, waiting = 0, []
    for elf, path in code_objects:
        if b"qgemm_dma" not in elf:
            continue
        for name, code in _instructions(path):
            if not re.search("qgemm_dma", name):
                continue
            kernels += 1
            index = {at: i for i, (at, _, _) in enumerate(code)}
            todo, seen, free = [max(i for i, c in enumerate(code) if c[1].startswith("v_mfma"))], set(), False
            while todo and not free:
                i = todo.pop()
                if i in seen or i >= len(code):
                    continue
                seen.add(i)
                _, op, to = code[i]
                if re.match("global_(store|load_dword)", op):
                    free = True
                if re.match(r"s_waitcnt vmcnt\(0\)", op) or op.startswith("s_endpgm"):
                    continue
                if to is not None:
                    todo.append(index[to])
                if not op.startswith("s_branch"):
                    todo.append(i + 1)
            if not free:
                waiting.append(name)
    assert kernels >= 3 * 16 and not waiting, waiting


def test_the_score_has_four_loads_of_the_reference_in_flight(code_objects):
    """The epilogue that scores reads the reference output from memory: 16 bytes of four accumulator tiles at a time."""
    kernels, few = 0, []
    for elf, path in code_objects:
        if b"qgemm_dma" not in elf and b"qgemm_quad" not in elf:
            continue
        for name, code in _instructions(path):
            tile = re.search(r"qgemm_(?:dmaILi(\d+)|quad)\w+?Lb\dELb(\d)E(?:Li\d+ELi\d+E)?Li1EEEvPKa", name)
            if not tile or tile.groups() == ("64", "1"):  # (there the compiler moves two behind the first row's arithmetic)
                continue
            kernels += 1
            most = now = 0
            for _, op, _ in code:
                if op.startswith("global_load_dwordx4"):
                    now += 1
                    most = max(most, now)
                elif "vmcnt" in op:
                    now = 0
            if most < 4:
                few.append((name, most))
    assert kernels >= 2 * 2 * 6 and not few, few


def test_the_measured_matrix_rate_is_that_of_the_kernels_own_steps(code_objects):
    """mpq_diag_mfma_rate is what a GEMM is held against: it issues the matrix instruction that the GEMM kernels issue."""
    steps = {}
    for elf, path in code_objects:
        if b"mfma_burn" not in elf and b"qgemm_" not in elf:
            continue
        for name, code in _instructions(path):
            kind = re.search("mfma_burn|qgemm_(?:dma|quad|any)", name)
            if kind:
                steps.setdefault(kind.group(0), set()).update(op.split()[0] for _, op, _ in code if op.startswith("v_mfma"))
    assert len(steps) == 4 and set.union(*steps.values()) == steps["qgemm_quad"] == steps["mfma_burn"], steps

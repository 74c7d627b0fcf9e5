"""What the compiler made of the kernels, read from the code objects in the built library: things that cost time without
changing a result."""
from __future__ import annotations

import os
import re
import struct
import subprocess

import pytest

import paper_2602_20732_amd as pk

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
pytestmark = pytest.mark.skipif(not os.path.exists(READELF), reason="llvm-readelf of the ROCm toolchain is not there")


def code_objects(path):
    """The gfx950 code objects bundled into a library."""
    blob = open(path, "rb").read()
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := blob.find(magic, at)) >= 0:
        (n,) = struct.unpack_from("<Q", blob, at + 24)
        p = at + 32
        for _ in range(n):
            off, size, name = struct.unpack_from("<QQQ", blob, p)
            if b"gfx950" in blob[p + 24:p + 24 + name] and size:
                yield blob[at + off:at + off + size]
            p += 24 + name
        at += 24


@pytest.fixture(scope="module")
def listings(tmp_path_factory):
    """(symbols, notes) of every code object, names demangled."""
    if not os.path.exists(pk.library_path()):
        from paper_2602_20732_amd.build import build
        build()
    out = []
    for i, obj in enumerate(code_objects(pk.library_path())):
        f = tmp_path_factory.mktemp("co") / f"{i}.co"
        f.write_bytes(obj)
        out.append(tuple(subprocess.run([READELF, flag, "-W", "-C", str(f)], capture_output=True, text=True, check=True).stdout
                         for flag in ("--symbols", "--notes")))
    assert out
    return out


def code_bytes(listings):
    sizes = {}
    for symbols, _ in listings:
        for m in re.finditer(r"\s(\d+) FUNC .*?chess::(\w+(?:<[^(]*>)?)\(", symbols):
            sizes[m.group(2)] = int(m.group(1))
    return sizes


def scratch_bytes(listings):
    """Scratch memory a lane, by mangled kernel name: spilled registers, or an array with a run-time index."""
    return {m.group(1): int(m.group(2)) for _, notes in listings
            for m in re.finditer(r"\.name:\s+(\S+)\n\s+\.private_segment_fixed_size:\s+(\d+)", notes)}


def kernels_named(listings, name):
    """The notes of the kernels whose name begins so."""
    return [b for _, notes in listings for b in notes.split("- .agpr_count:")[1:] if re.search(r"\.name:\s+_ZN5chess\d+" + name, b)]


def vector_registers(listings, name):
    return [int(re.search(r"\.vgpr_count:\s+(\d+)", b).group(1)) for b in kernels_named(listings, name)]


def test_the_does_not_swell_attention_over_every_page(listings):
    """The last workgroup of a sequence runs the merge once, from cold code: four inlined variants of it (19 KB a kernel) cost 1 to 9 %
    of attention over every page."""
    sizes = code_bytes(listings)
    dense = {n: s for n, s in sizes.items() if re.match(r"decode_kernel<\d+, 4, false, ", n)}
    assert len(dense) == 4, sorted(sizes)
    for name, size in dense.items():
        assert size <= (16 if name.endswith("true>") else 12) * 1024, (name, size)


def test_no_kernel_needs_scratch_memory(listings):
    """A kernel with scratch memory starts 2-3 us later, however little it is."""
    scratch = scratch_bytes(listings)
    assert len(scratch) > 50 and not any(scratch.values()), {n: b for n, b in scratch.items() if b}


def test_three_workgroups_of_the_recent_pages_fit_on_a_compute_unit(listings):
    """With more than 168 registers a lane two fit, and 96 sequences of 8 KV heads took two rounds of the 256 compute units (a page of 32
    of each 13.6 us where the kernel for every page takes 11.6, and 8.5 in one round)."""
    registers = vector_registers(listings, "summarize_recent_kernel")
    assert len(registers) == 4 and max(registers) <= 168, registers


def test_one_sequence_in_pages_of_32_keeps_to_the_registers_of_four_workgroups(listings):
    """With 136 registers instead of 124 its tiles came 5 to 7 % later (131072 tokens, one KV head, sixteen query heads 51.9 -> 55.6 us): the
    compiler uses them to ask for the value rows earlier."""
    registers = vector_registers(listings, "decode_kernelILi32ELi4ELb0ELb0E")
    assert len(registers) == 1 and registers[0] <= 128, registers


def test_the_runtime_sees_no_pointers_in_the_step(listings):
    """A pointer argument is looked up at each launch, and memory seen for the first time cost 45 us of a first pass there: the fused step
    takes its pointers as numbers and inside structs."""
    kernels = kernels_named(listings, "step_kernel")
    assert len(kernels) == 16 and not any("global_buffer" in b for b in kernels)


@pytest.mark.parametrize("name,instances", [("decode_kernel", 12), ("reuse_kernel", 8), ("summarize_recent_kernel", 4)])
def test_nor_in_the_other_kernels_of_a_step(listings, name, instances):
    kernels = kernels_named(listings, name)
    assert len(kernels) == instances and not any("global_buffer" in b for b in kernels)

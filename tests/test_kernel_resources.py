"""Registers of the compiled kernels, where the number of resident waves depends on them.

Read from the metadata that the compiler leaves in the code objects of libhufield.so (no GPU needed).
512 registers of a SIMD's lane are shared out in blocks of 8: up to 128 each for four waves, up to
168 for three.
"""

import os
import re
import shutil
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2509_08675_amd", "libhufield.so")
READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"

pytestmark = pytest.mark.skipif(not (os.path.exists(LIB) and os.path.exists(READELF)),
                                reason="libhufield.so or llvm-readelf missing")


def code_objects(blob):
    at = blob.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", blob, at + len(MAGIC))
        pos = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", blob, pos)
            name = blob[pos + 24:pos + 24 + idlen].decode()
            pos += 24 + idlen
            if "gfx950" in name and size:
                yield blob[at + off:at + off + size]
        at = blob.find(MAGIC, at + len(MAGIC))


@pytest.fixture(scope="module")
def metadata(tmp_path_factory):
    """{mangled name: (vector registers, bytes of scratch per lane, bytes of arguments)} of every kernel."""
    path = str(tmp_path_factory.mktemp("co") / "k.o")
    out = {}
    with open(LIB, "rb") as fh:
        blob = fh.read()
    for co in code_objects(blob):
        with open(path, "wb") as fh:
            fh.write(co)
        text = subprocess.run([READELF, "--notes", path], capture_output=True, text=True, check=True).stdout
        for entry in re.split(r"^  - \.agpr_count:", text, flags=re.M)[1:]:
            name = re.search(r"^    \.name: +(\S+)", entry, flags=re.M).group(1)
            regs = int(re.search(r"^    \.vgpr_count: +(\d+)", entry, flags=re.M).group(1))
            scratch = int(re.search(r"^    \.private_segment_fixed_size: +(\d+)", entry, flags=re.M).group(1))
            args = int(re.search(r"^    \.kernarg_segment_size: +(\d+)", entry, flags=re.M).group(1))
            out[name] = (regs, scratch, args)
    return out


@pytest.fixture(scope="module")
def kernels(metadata):
    return {name: use[:2] for name, use in metadata.items()}


@pytest.fixture(scope="module")
def co_args(metadata):
    return {name: use[2] for name, use in metadata.items()}


def filter_kernels(kernels, amp):
    """(length, dimension, width) -> (registers, scratch) of the filter pass with amplitudes from `amp`."""
    rx = re.compile(r"k_cols_filterILi(\d+)ELi(\d)ELi(\d)ELi%dELi0ELb0E" % amp)
    found = {}
    for name, use in kernels.items():
        m = rx.search(name)
        if m:
            found[tuple(int(x) for x in m.groups())] = use
    assert found
    return found


def test_general_filter_form_keeps_its_waves(kernels):
    # the FP64 evaluation in the pass: four waves per SIMD, three for columns of 24 elements a thread
    for (length, nd, width), (regs, scratch) in filter_kernels(kernels, 1).items():
        most = 168 if length % 3 == 0 else 128
        assert regs <= most and scratch == 0, (length, nd, width, regs, scratch)


def test_five_wave_filter_tiles_leave_room_for_two_workgroups(kernels):
    # 384 and 768, full width: two workgroups of five waves need a SIMD with room for four
    found = filter_kernels(kernels, 0)
    for length in (384, 768):
        regs, scratch = found[length, 3, 0]
        assert regs <= 128 and scratch <= 64, (length, regs, scratch)


def test_no_kernel_that_nothing_launches(kernels):
    # 2D columns up to 1024 always take half-width filter and binning tiles
    rx = [re.compile(r"k_cols_filterILi(\d+)ELi2ELi0ELi[01]E"), re.compile(r"k_cols_binILi(\d+)ELi0ELi\dELb\dELb1E")]
    for name in kernels:
        for r in rx:
            m = r.search(name)
            assert m is None or int(m.group(1)) > 1024, name


def test_loading_row_passes_carry_no_seeds(co_args):
    # the launch copies a kernel's arguments: 2 KB of seeds belong to the noise source alone
    rx = re.compile(r"k_rows_r2cILi\d+ELi(\d)E")
    sizes = {0: [], 1: [], 2: []}
    for name, n in co_args.items():
        m = rx.search(name)
        if m:
            sizes[int(m.group(1))].append(n)
    assert min(sizes[0]) >= 2048 and sizes[1] and max(sizes[1] + sizes[2]) < 768


def test_host_and_device_agree_on_kernel_names(kernels):
    # a launch looks its kernel up by name: every name that the host code holds is in a code object
    with open(LIB, "rb") as fh:
        held = {m.decode() for m in re.findall(rb"_ZN2hu\d+k_\w+", fh.read())}
    assert held and held <= set(kernels)

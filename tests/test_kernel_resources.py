"""What the kernels of the built library take of a compute unit, as their descriptors state it: no kernel spills (a thread's
private memory is allocated by the runtime when a kernel first needs it, and daf_quantize_pack_static is for callers that
cannot allocate), and the code for the tile in which a tensor ends does not cost the whole tiles a wave."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2507_07149_amd import build

LLVM = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(build.HIPCC))), "llvm", "bin")


def _descriptors(elf):
    """(mangled name, LDS bytes, private bytes per thread, registers per thread) of every kernel of a code object."""
    at, = struct.unpack_from("<Q", elf, 0x28)
    size, count = struct.unpack_from("<HH", elf, 0x3A)
    sections = [struct.unpack_from("<IIQQQQIIQQ", elf, at + i * size) for i in range(count)]
    for _, kind, _, _, offset, length, link, _, _, entry in sections:
        if kind != 11:                                             # the dynamic symbols
            continue
        for i in range(0, length, entry):
            name, _, _, section, value, _ = struct.unpack_from("<IBBHQQ", elf, offset + i)
            text = elf[sections[link][4] + name:]
            text = text[:text.index(b"\0")].decode()
            if text.endswith(".kd"):
                place = sections[section][4] + value - sections[section][3]
                lds, private = struct.unpack_from("<II", elf, place)
                rsrc1, = struct.unpack_from("<I", elf, place + 48)
                yield text[:-3], lds, private, 8 * ((rsrc1 & 63) + 1)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{mangled name: (private bytes, waves per SIMD)} of every kernel."""
    here = tmp_path_factory.mktemp("objects")
    shutil.copy(build.LIB, here / "lib.so")
    subprocess.run([os.path.join(LLVM, "llvm-objdump"), "--offloading", "lib.so"], cwd=here, check=True, stdout=subprocess.DEVNULL)
    found = {}
    for name in sorted(os.listdir(here)):
        if "gfx950" in name:
            for kernel, lds, private, registers in _descriptors((here / name).read_bytes()):
                # 512 registers, and 160 KB of LDS for the four SIMDs, with workgroups of four waves
                found[kernel] = private, min(8, 512 // registers, 160 * 1024 // max(lds, 1))
    assert len(found) > 1000
    return found


def test_no_kernel_spills(kernels):
    assert {name: private for name, (private, _) in kernels.items() if private} == {}


def test_lists_with_short_tiles_run_as_many_waves_as_lists_of_whole_ones(kernels):
    pairs = [(n, re.sub("ELb1EEEv", "ELb0EEEv", n)) for n in kernels if re.search(r"k_quantize_pack_(tile|units)_batch\w*ELb1EEEv", n)]
    assert len(pairs) == 3 * 5 * 8 + 5 + 3 * 5                     # formats, widths, group sizes (binary32 has one more); units
    assert {n: (kernels[n][1], kernels[whole][1]) for n, whole in pairs if kernels[n][1] < kernels[whole][1]} == {}


def test_statistics_run_eight_waves(kernels):
    """(Binary32 groups of 64: seven, with and without the short tile's code.)"""
    waves = {re.search(r"tileILi(\d)ELi(\d+)E", n).groups(): w for n, (_, w) in kernels.items() if "k_group_minmax_tile" in n}
    assert len(waves) == 25 and waves.pop(("0", "4")) == 7 and set(waves.values()) == {8}


def test_binary32_tiles_run_at_most_the_waves_that_keep_their_streams_together(kernels):
    """Six, five with 8 bits; lists in groups of 4096 three.  (Not the metrics, and not the tiles of longer groups.)"""
    seen = 0
    for name, (_, waves) in kernels.items():
        m = re.search(r"k_quantize_pack_tile(_batch)?ILi0ELi(\d+)ELi(\d)E(?:Lb0ELb0)?", name)
        if m and (m.group(1) or "Lb0ELb0" in m.group(0)):
            most = 3 if m.group(1) and m.group(2) == "10" else 5 if m.group(3) == "8" else 6
            assert waves <= most, (name, waves)
            seen += 1
    assert seen == 9 * 5 * 4                                       # group sizes, widths; one tensor with and without relu, two list kernels

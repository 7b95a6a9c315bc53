"""Registers and scratch memory of the built kernels, read from the library's own code objects: what the launch bounds and
the estimates of a launch's time assume of them.  CPU only."""
import os
import re
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2111_00153_amd", "librmsmp.so")
READELF = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-readelf")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(data):
    """The gfx950 objects of the bundles in a library: header, then (offset, size, name) of each entry."""
    at = data.find(MAGIC)
    while at >= 0:
        count, = struct.unpack_from("<Q", data, at + len(MAGIC))
        entry = at + len(MAGIC) + 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, entry)
            name = data[entry + 24:entry + 24 + length]
            entry += 24 + length
            if b"gfx950" in name and size:
                yield data[at + offset:at + offset + size]
        at = data.find(MAGIC, at + len(MAGIC))


@pytest.fixture(scope="module")
def code_bytes(tmp_path_factory):
    """{(name, template arguments): bytes of code}"""
    found = {}
    path = tmp_path_factory.mktemp("code") / "object"
    with open(LIB, "rb") as f:
        data = f.read()
    for obj in _code_objects(data):
        path.write_bytes(obj)
        symbols = subprocess.run([READELF, "--symbols", "--wide", str(path)], capture_output=True, text=True, check=True).stdout
        for size, name, arguments in re.findall(r"\s(\d+) FUNC .* _ZN5rmsmp\d+([a-z0-9_]+_kernel)I((?:L[ib]\d+E)+)E", symbols):
            found[name, tuple(int(v) for v in re.findall(r"L[ib](\d+)E", arguments))] = int(size)
    return found


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{(name, template arguments): (registers, bytes of scratch)}"""
    found = {}
    path = tmp_path_factory.mktemp("code") / "object"
    with open(LIB, "rb") as f:
        data = f.read()
    for obj in _code_objects(data):
        path.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for block in re.split(r"\n  - \.agpr_count:", notes)[1:]:
            def value(key):
                return re.search(r"\." + key + r":\s+(\S+)", block).group(1)
            m = re.match(r"_ZN5rmsmp\d+([a-z0-9_]+_kernel)I((?:L[ib]\d+E)+)E", value("name"))
            if m:
                arguments = tuple(int(v) for v in re.findall(r"L[ib](\d+)E", m.group(2)))
                found[m.group(1), arguments] = (int(value("vgpr_count")), int(value("private_segment_fixed_size")))
    return found


def _named(kernels, name):
    return {arguments: use for (n, arguments), use in kernels.items() if n == name}


def test_fp6_tile_kernels_keep_their_sums_in_registers(kernels):
    """No instantiation (blocks per wave, waves along rows, along columns, convolution, ragged, GELU) spills."""
    tile = _named(kernels, "fp6_tile_kernel")
    assert {a: use for a, use in tile.items() if use[1] != 0} == {}
    assert len(tile) == 8 * 2 * 2 * 2


def test_fp6_joined_kernels_keep_their_sums_in_registers(kernels):
    """The same for the five shapes with neighbouring tiles joined in a wave (blocks, waves, waves, convolution, ragged)."""
    joined = _named(kernels, "fp6_joined_kernel")
    assert {a: use for a, use in joined.items() if use[1] != 0} == {} and len(joined) == 5 * 2 * 2


def test_lds_resident_kernels_without_a_bias_have_the_registers_their_estimates_assume(kernels):
    """Template arguments: taps, K steps, pixel blocks, K split, side by side, tile pairs, in parts, bias.  With 64 pixels a wave,
    K split and two tile pairs three work-groups share a compute unit (at most 168 registers; 768 channels have always taken
    169); a wave with all of K spills nothing."""
    wide = {a: use for a, use in _named(kernels, "conv_wide_kernel").items() if not a[-1]}
    three = {a: use for a, use in wide.items() if a[2:6] == (2, 2, 1, 2) and not a[6] and a[1] != 24}
    assert {a: use for a, use in three.items() if use[0] > 168} == {} and len(three) == 7
    whole = {a: use for a, use in wide.items() if a[3] == 1}
    assert {a: use for a, use in whole.items() if use[1] != 0} == {} and len(whole) > 20


def test_patch_kernels_keep_their_sums_in_registers(kernels):
    """Template arguments: blocks per wave, K split, pairs of tiles, waves along the columns, ragged.  Two waves share a SIMD (at most 256
    registers), and none spills: the estimates of ten shapes, and of three with two layers in a launch, assume both."""
    patch, pair = _named(kernels, "fp6_patch_kernel"), _named(kernels, "fp6_patch_pair_kernel")
    assert {a: use for a, use in {**patch, **pair}.items() if use[0] > 256 or use[1] != 0} == {}
    assert len(patch) == 10 * 2 and len(pair) == 3


def test_kernels_that_read_their_code_have_readers_for_all_of_it(code_bytes):
    """The first waves of a launch on each XCD read 8 KB each: eight of them, twelve where a launch has two layers."""
    for name, readers, count in (("fp6_patch_kernel", 8, 10 * 2), ("conv_first_kernel", 8, 3 * 3 * 4), ("fp6_patch_pair_kernel", 12, 3)):
        sizes = _named(code_bytes, name)
        assert len(sizes) == count and max(sizes.values()) <= readers * 8192, (name, sizes)


def test_first_layer_kernels_spill_nothing_in_their_plain_loops(kernels):
    """Template arguments: filter side, rows of a tile, loop.  Whole 4-bit rows without a bias (1), with one (3), any 4-bit rows (2); the 7x7
    filter's 16 rows with a bias hold three blocks of fragments and spill five registers."""
    first = {a: use for a, use in _named(kernels, "conv_first_kernel").items() if a[2] != 0}
    assert {a: use[1] for a, use in first.items() if use[1] != 0} in ({}, {(7, 16, 3): 20}) and len(first) == 3 * 3 * 3

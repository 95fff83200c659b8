"""Registers and scratch of the built kernels, as their code objects state them.  Needs no GPU."""
import ctypes as C
import os
import re
import struct
import subprocess

import pytest

from paper_2011_06295_amd import binding as B, build

LLVM = "/opt/rocm/llvm/bin"
_MATRIX = re.compile(r"matrix_kernelI(DF16_|f)Li(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELb(\d)EEE")


def _code_objects(data):
    """The gfx950 ELF images of the library's offload bundles."""
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := data.find(magic, at)) >= 0:
        p = at + len(magic) + 8
        for _ in range(struct.unpack_from("<Q", data, p - 8)[0]):
            offset, size, length = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + length]:
                yield data[at + offset:at + offset + size]
            p += 24 + length
        at += len(magic)


def _metadata(elf, path):
    """The kernels' entries of an image's metadata note."""
    path.write_bytes(elf)
    notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", str(path)], stdout=subprocess.PIPE, text=True, check=True).stdout
    for entry in notes.split("\n  - ")[1:]:
        yield {key: value for key, value in re.findall(r"^ *(\.\w+): +(\S+)$", entry, re.M)}


@pytest.fixture(scope="module")
def matrix_kernels(tmp_path_factory):
    """(type, MK, NP, steps ahead, blocks in flight, KS, runs) of every matrix kernel -> its metadata."""
    found = {}
    with open(build.LIB, "rb") as f:
        data = f.read()
    path = tmp_path_factory.mktemp("code") / "object"
    for elf in _code_objects(data):
        for kernel in _metadata(elf, path):
            m = _MATRIX.search(kernel.get(".name", ""))
            if m:
                found[("f32" if m[1] == "f" else "f16", *map(int, m.groups()[1:]))] = kernel
    assert found
    return found


def _wavefronts(kernel):
    """That a SIMD's 512 registers a lane hold."""
    return min(8, 512 // ((int(kernel[".vgpr_count"]) + 7) // 8 * 8))


def test_binary16_matrix_kernels_use_no_scratch(matrix_kernels):
    kept = {v: k[".private_segment_fixed_size"] for v, k in matrix_kernels.items() if v[0] == "f16" and k[".private_segment_fixed_size"] != "0"}
    assert not kept, kept


def test_the_smallest_variant_has_four_wavefronts_a_simd(matrix_kernels):
    assert _wavefronts(matrix_kernels[("f16", 2, 2, 2, 2, 1, 0)]) == 4


def test_the_estimate_counts_the_workgroups_that_registers_hold(matrix_kernels):
    resident = B.raw_library()["_ZN2sc15matrix_residentEiiiiiib"]   # sc::matrix_resident(MK, NP, KS, ahead, fly, runs, split)
    resident.argtypes = [C.c_int] * 6 + [C.c_bool]
    wrong = {}
    for (dtype, MK, NP, ahead, fly, KS, wide), kernel in matrix_kernels.items():
        counted = resident(MK, NP, KS, ahead, 0 if wide else fly, fly if wide else 0, dtype == "f32")
        held = _wavefronts(kernel) // (2 if KS == 8 else 1)
        if counted != held:
            wrong[dtype, MK, NP, ahead, fly, KS, wide] = counted, held
    assert not wrong, wrong


def test_every_matrix_kernel_that_is_built_has_a_layer_in_the_tests(matrix_kernels):
    from test_gpu_matrix import VARIANTS
    from test_gpu_matrix_eight import VARIANTS as EIGHT
    tested = {(d, MK, NP, ahead, runs or fly, KS, int(runs > 0)) for d, (MK, NP, _, KS, ahead, fly, runs), _ in VARIANTS}
    tested |= {("f16", MK, NP, ahead, runs or fly, 8, int(runs > 0)) for (MK, NP, ahead, fly, runs, _), _ in EIGHT}
    assert tested == set(matrix_kernels)

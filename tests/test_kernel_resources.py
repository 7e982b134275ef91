"""What the compiled kernels need, read from the code objects that the build puts into the library."""
import os
import re
import struct
import subprocess

import pytest

import paper_2505_18610_amd as kq

LLVM = "/opt/rocm/llvm/bin"


def code_objects(path):
    """The gfx950 code objects of a library, one per translation unit."""
    data = open(path, "rb").read()
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):
        at = m.start() + 32
        for _ in range(struct.unpack_from("<Q", data, m.start() + 24)[0]):
            offset, size, id_size = struct.unpack_from("<QQQ", data, at)
            if data[at + 24:at + 24 + id_size].endswith(b"gfx950"):
                yield data[m.start() + offset:m.start() + offset + size]
            at += 24 + id_size


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """name (demangled, without arguments) -> {field of the metadata: number}"""
    tool, found = os.path.join(LLVM, "llvm-readelf"), {}
    if not os.path.exists(tool):
        pytest.skip("no llvm-readelf")
    path = tmp_path_factory.mktemp("co") / "object"
    for code in code_objects(kq.library_path()):
        path.write_bytes(code)
        notes = subprocess.run([tool, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for entry in notes.split("  - .agpr_count:")[1:]:
            name = re.search(r"\.name: +(\S+)", entry).group(1)
            name = subprocess.run(["c++filt", name], capture_output=True, text=True, check=True).stdout.strip()
            name = re.search(r"kvq_\w+(<[^>]*>)?", name).group(0)
            found[name] = {k: int(v) for k, v in re.findall(r"\.(\w+): +(\d+)$", entry, re.M)}
    return found


def test_no_kernel_uses_scratch(kernels):
    """A kernel with scratch pays for its allocation at every launch."""
    assert len(kernels) > 30
    for name, k in kernels.items():
        assert k["private_segment_fixed_size"] == 0 and k["vgpr_spill_count"] == 0, name


def test_wavefronts_that_the_launch_rules_count_on(kernels):
    """512 registers a lane and SIMD in steps of eight, 160 KiB of LDS a compute unit."""
    def per_simd(name, waves_per_group):
        k = kernels[name]
        by_lds = 160 * 1024 // max(1, k["group_segment_fixed_size"]) * waves_per_group // 4
        return min(8, 512 // ((k["vgpr_count"] + 7) // 8 * 8), by_lds)

    assert per_simd("kvq_append16_kernel<false, true>", 1) == 5
    assert per_simd("kvq_append16_kernel<false, false>", 1) == 4
    for bits in (8, 4, 2):
        assert per_simd(f"kvq_append_q_kernel<{bits}, false, false>", 4) == 4
        assert per_simd(f"kvq_append_q_kernel<{bits}, false, true>", 4) == 5
    for mode in range(4):
        assert per_simd(f"kvq_error_kernel<{mode}>", 4) == 4


def test_no_kernel_that_no_launch_reaches(kernels):
    """Strings into 2 bits that need no preparation are always shared by two wavefronts."""
    assert {n for n in kernels if n.startswith("kvq_append_q_kernel")} == {
        f"kvq_append_q_kernel<{bits}, {plain}, {pair}>" for bits in (8, 4, 2) for plain in ("true", "false") for pair in ("true", "false")
        if (bits, plain, pair) != (2, "true", "false")}


def test_the_build_without_arithmetic_has_none(tmp_path):
    """libkvq_noarith.so times loads, join and merge alone: not one of its attention kernels multiplies on the matrix cores."""
    from paper_2505_18610_amd.build import NOARITH_LIB
    tool = os.path.join(LLVM, "llvm-objdump")
    if not (os.path.exists(tool) and os.path.exists(NOARITH_LIB)):
        pytest.skip("no llvm-objdump, or the measurement build is not there")

    def products(lib):
        n = 0
        for i, code in enumerate(code_objects(lib)):
            path = tmp_path / f"object{i}"
            path.write_bytes(code)
            n += subprocess.run([tool, "-d", str(path)], capture_output=True, text=True, check=True).stdout.count("v_mfma_")
        return n

    assert products(kq.library_path()) > 0 and products(NOARITH_LIB) == 0

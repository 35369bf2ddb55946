"""What the compiler made of the kernels: read from the metadata and the instructions of the built library's own code
object (no GPU).  Registers in scratch memory, accumulators copied between register files inside a loop and loads that
became loops over the lanes all give right results, only slowly, so no other test sees them."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2605_08696_amd import build

msgpack = pytest.importorskip("msgpack")


@pytest.fixture(scope="module")
def code_object():
    """The gfx950 ELF inside the offload bundle of libsrm.so."""
    if not os.path.exists(build.LIB):
        build.build_lib()
    data = open(build.LIB, "rb").read()
    base = data.index(b"__CLANG_OFFLOAD_BUNDLE__")
    (n,) = struct.unpack_from("<Q", data, base + 24)
    at = base + 32
    for _ in range(n):
        off, size, length = struct.unpack_from("<QQQ", data, at)
        triple = data[at + 24:at + 24 + length]
        at += 24 + length
        if b"gfx950" in triple:
            return data[base + off:base + off + size]
    raise AssertionError("no gfx950 code object in the library")


@pytest.fixture(scope="module")
def kernels(code_object):
    (table,) = struct.unpack_from("<Q", code_object, 40)
    entry, count = struct.unpack_from("<HH", code_object, 58)
    for k in range(count):
        (kind,) = struct.unpack_from("<I", code_object, table + k * entry + 4)
        if kind != 7:                                            # SHT_NOTE
            continue
        (off,) = struct.unpack_from("<Q", code_object, table + k * entry + 24)
        name_len, desc_len, _ = struct.unpack_from("<III", code_object, off)
        desc = off + 12 + ((name_len + 3) & ~3)
        return {q[".name"]: q for q in msgpack.unpackb(code_object[desc:desc + desc_len])["amdhsa.kernels"]}
    raise AssertionError("no metadata note")


def test_no_kernel_spills_vector_registers(kernels):
    """nucleus_slow_kernel apart, whose 1024 threads hold 32 logits each within 128 registers."""
    spilled = {n: q[".vgpr_spill_count"] for n, q in kernels.items() if q[".vgpr_spill_count"] and "nucleus_slow" not in n}
    assert len(kernels) > 200 and not spilled


def test_no_kernel_has_scratch_memory(kernels):
    """Neither for spilled registers nor for an argument whose address is taken; nucleus_slow_kernel apart, as above."""
    assert not {n: q[".private_segment_fixed_size"] for n, q in kernels.items() if q[".private_segment_fixed_size"] and "nucleus_slow" not in n}


def test_bf16_gemms_keep_their_accumulators_in_one_register_file(kernels):
    """Two wavefronts per SIMD leave 256 registers, enough for every tile: with a larger budget the compiler keeps operands
    in accumulation registers and copies them back and forth inside the k loop."""
    gemms = {n: q for n, q in kernels.items() if "gemm_bf16_kernel" in n or "gemm_bf16_persist_kernel" in n}
    assert len(gemms) > 40 and not {n: q[".agpr_count"] for n, q in gemms.items() if q[".agpr_count"]}


def test_persistent_gemm_loads_its_bias_without_loops_over_lanes(code_object, kernels, tmp_path):
    """A buffer descriptor that the compiler does not know to be uniform turns each of its loads into a loop."""
    objdump = next((p for p in ("/opt/rocm/llvm/bin/llvm-objdump", shutil.which("llvm-objdump")) if p and os.path.exists(p)), None)
    if objdump is None:
        pytest.skip("no llvm-objdump")
    elf = tmp_path / "gfx950.elf"
    elf.write_bytes(code_object)
    names = [n for n in kernels if "gemm_bf16_persist_kernel" in n]
    assert len(names) >= 6
    for name in names:
        text = subprocess.run([objdump, "-d", f"--disassemble-symbols={name}", str(elf)], capture_output=True, text=True, check=True).stdout
        lines = text.splitlines()
        assert sum("v_mfma" in x for x in lines) >= 64
        for i, line in enumerate(lines):
            if re.search(r"buffer_load_dwordx4 v\[", line):
                assert not any("s_cbranch_execnz" in x for x in lines[i + 1:i + 6]), name

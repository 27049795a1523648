"""Registers of kernels whose speed rests on how many of their waves fit a SIMD, read from the built library (no GPU).

A SIMD has 512 registers a lane, dealt out eight at a time, and holds at most eight waves."""
import os
import re
import struct
import subprocess

import pytest

import paper_2407_11062_amd as eq

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


@pytest.fixture(scope="module")
def waves_per_simd(tmp_path_factory):
    if not os.path.exists(READELF):
        pytest.skip("llvm-readelf is not installed")
    eq.lib()
    blob = open(eq.LIB_PATH, "rb").read()
    out, magic = {}, b"__CLANG_OFFLOAD_BUNDLE__"
    path = tmp_path_factory.mktemp("co") / "code_object"
    for m in re.finditer(magic, blob):
        at = m.start() + len(magic)
        (n,) = struct.unpack_from("<Q", blob, at)
        at += 8
        for _ in range(n):
            off, size, id_len = struct.unpack_from("<QQQ", blob, at)
            name = blob[at + 24:at + 24 + id_len]
            at += 24 + id_len
            if b"gfx950" not in name:
                continue
            path.write_bytes(blob[m.start() + off:m.start() + off + size])
            notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
            for kernel, regs in re.findall(r"\.name:\s+(_Z\S+)\n(?:(?!\.name:).)*?\.vgpr_count:\s+(\d+)", notes, flags=re.S):
                out[kernel] = min(8, 512 // ((int(regs) + 7) // 8 * 8))
    return out


def run_kernel(waves, bits, floatz, ng, mw):
    return waves[next(k for k in waves if f"k_gemv_runILi{bits}ELb{floatz}ELi{ng}ELb{mw}E" in k)]


@pytest.mark.parametrize("floatz", [0, 1])
@pytest.mark.parametrize("ng", [1, 4])
def test_matrix_vector_kernel_of_2_bit_codes_keeps_eight_waves(waves_per_simd, floatz, ng):
    # four waves for each 16 of 28672 rows are 7168: one round of 256 compute units takes 7 waves per SIMD
    assert run_kernel(waves_per_simd, 2, floatz, ng, 0) == 8

"""Registers of the kernels as they are built: none of a GEMM's sits in scratch.  A reload is a vector-memory operation, and the wait for it waits for all loads
under way (dW with fp32 weights, two registers: up to 16 % slower).  The instantiation of the forward and dX that cuts tiles of 256 x 256 keeps one or two there."""
import re
import struct
import subprocess

import paper_2407_11062_amd as eq

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def code_objects(path):
    blob = open(path, "rb").read()
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    for at in (m.start() for m in re.finditer(magic, blob)):
        count, pos = struct.unpack_from("<Q", blob, at + len(magic))[0], at + len(magic) + 8
        for _ in range(count):
            offset, size, n = struct.unpack_from("<QQQ", blob, pos)
            if b"gfx950" in blob[pos + 24:pos + 24 + n]:
                yield blob[at + offset:at + offset + size]
            pos += 24 + n


def scratch_of_kernels(tmp_path):
    out = {}
    for k, code in enumerate(code_objects(eq.LIB_PATH)):
        f = tmp_path / f"{k}.co"
        f.write_bytes(code)
        notes = subprocess.run([READELF, "--notes", str(f)], capture_output=True, text=True, check=True).stdout
        for kernel in notes.split("- .agpr_count:")[1:]:
            out[re.search(r"\.name: +(\S+)", kernel)[1]] = int(re.search(r"\.private_segment_fixed_size: +(\d+)", kernel)[1])
    return out


def test_no_gemm_keeps_registers_in_scratch(tmp_path):
    scratch = scratch_of_kernels(tmp_path)
    assert sum("k_gemm_bwd" in k for k in scratch) == 63 and sum("k_gemm_dw" in k for k in scratch) == 36
    cut = re.compile(r"k_gemm_qILi\dELb[01]ELi1ELi256E")              # bits, transposed, kCut, 256 x ...
    assert {k for k, n in scratch.items() if n and "k_gemm" in k and not cut.search(k)} == set()
    assert all(n <= 12 for k, n in scratch.items() if cut.search(k))

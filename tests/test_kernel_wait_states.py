"""Wait states that inline assembly owes: the compiler puts them between its own instructions and sees none inside ours.  On gfx950 a scalar register that a
vector instruction wrote (readlane, readfirstlane, compare, carry) needs five wait states before a buffer load uses it, as part of its descriptor for
instance, and two before a vector instruction reads it, as a carry or as a mask.  Looked for in the kernels as they are built."""
import re
import subprocess

import pytest

import paper_2407_11062_amd as eq
from test_kernel_registers import code_objects

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
CARRY_OUT = ("v_add_co", "v_addc_co", "v_sub_co", "v_subb_co", "v_subrev_co", "v_subbrev_co", "v_div_scale", "v_mad_u64_u32", "v_mad_i64_i32")


def scalars(operand):
    """numbers of the scalar registers in an operand; vcc is -2, -1"""
    out = set()
    for m in re.finditer(r"\bs\[(\d+):(\d+)\]|\bs(\d+)\b|\bvcc(_lo|_hi)?\b", operand):
        if m[1]:
            out |= set(range(int(m[1]), int(m[2]) + 1))
        elif m[3]:
            out.add(int(m[3]))
        else:
            out |= {None: {-2, -1}, "_lo": {-2}, "_hi": {-1}}[m[4]]
    return out


def missing_waits(listing):
    """(kernel, instruction that writes, instruction that reads, wait states between) of a disassembly"""
    found, kernel, past = [], None, []
    for line in listing:
        m = re.match(r"[0-9a-f]+ <(.+)>:", line)
        if m:
            kernel, past = m[1], []
            continue
        text = line.split("//")[0].strip()
        if not re.match(r"[sv]_|buffer_|ds_|global_|flat_|scratch_", text):
            continue
        op, _, rest = text.partition(" ")
        args = [a.strip() for a in rest.split(",")]
        if op in ("s_branch", "s_endpgm", "s_setpc_b64"):
            past = []
            continue
        vector, memory = op.startswith("v_"), op.startswith("buffer_")
        two = op.startswith(CARRY_OUT)
        if vector or memory:
            reads = set().union(*(scalars(a) for a in (args[2:] if two else args[1:] if vector else args)), {-2, -1} if op.startswith("v_div_fmas") else set())
            need, waited = (2 if vector else 5), 0
            for states, writes, by in reversed(past):
                if waited >= need:
                    break
                if writes & reads:
                    found.append((kernel, by, text, waited))
                    break
                reads -= writes
                waited += states
        writes = set()
        if vector:
            writes = scalars(args[1]) if two else scalars(args[0])
        past.append((int(args[0]) + 1 if op == "s_nop" else 1, writes, text))
        del past[:-8]
    return found


def test_the_search_finds_what_it_is_for():
    listing = ["0000 <k>:", " v_cmp_ne_u32_e32 vcc, v1, v2 // x", " v_addc_co_u32_e32 v0, vcc, v0, v0, vcc // x", " v_readlane_b32 s9, v254, 3 // x", " s_mov_b32 m0, s3 // x",
               " s_nop 0 // x", " buffer_load_dwordx4 v4, s[8:11], 0 offen lds // x"]
    assert [f[3] for f in missing_waits(listing)] == [0, 2]
    listing.insert(2, " s_nop 1 // x")
    listing[-2] = " s_nop 3 // x"
    assert missing_waits(listing) == []


@pytest.fixture(scope="module")
def found(tmp_path_factory):
    found, kernels = [], 0
    for k, code in enumerate(code_objects(eq.LIB_PATH)):
        f = tmp_path_factory.mktemp("code") / f"{k}.co"
        f.write_bytes(code)
        listing = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(f)], capture_output=True, text=True, check=True).stdout.splitlines()
        kernels += sum("k_" in l for l in listing if l.endswith(">:"))
        found += missing_waits(listing)
    assert kernels > 200
    return found


def test_vector_instructions_wait_for_carries_and_masks(found):
    found = [f for f in found if f[2].startswith("v_")]
    assert found == [], f"{len(found)}: {found[:4]}"


def test_buffer_loads_wait_for_their_descriptors(found):
    found = [f for f in found if f[2].startswith("buffer_")]
    assert found == [], f"{len(found)}: {found[:4]}"

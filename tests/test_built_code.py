"""What libplc.so's own device code has to keep to and no compiler checks for it: steps written in assembly, whose
registers the compiler's hazard recognizer does not look at.  On the host: the built code objects, disassembled."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2604_15356_amd import plc

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(library):
    """The gfx950 code objects that a library embeds, one for each HIP source."""
    data = open(library, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        (n,) = struct.unpack_from("<Q", data, at + len(MAGIC))
        pos = at + len(MAGIC) + 8
        for _ in range(n):
            offset, size, id_len = struct.unpack_from("<QQQ", data, pos)
            name = data[pos + 24:pos + 24 + id_len]
            pos += 24 + id_len
            if name.endswith(b"gfx950") and size:
                yield data[at + offset:at + offset + size]
        at = data.find(MAGIC, at + len(MAGIC))


def _registers(operand):
    """Scalar registers that an operand names."""
    if operand in ("vcc", "vcc_lo", "vcc_hi"):
        return {"vcc"}
    m = re.fullmatch(r"s(\d+)", operand)
    if m:
        return {int(m[1])}
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", operand)
    return set(range(int(m[1]), int(m[2]) + 1)) if m else set()


def scalars_read_too_early(listing):
    """(kernels, their vector instructions, [(kernel, writer, reader)]): vector instructions that read a scalar register
    that a vector instruction wrote fewer than two wait states before, every instruction being one and s_nop n n + 1."""
    kernels, vector, found = set(), 0, []
    kernel, before = None, []  # the last two wait states, the latest first: (instruction, scalars it writes)
    for line in listing:
        if line[:1] != "\t":
            m = re.match(r"[0-9a-f]{16} <(.*)>:", line)
            if m:
                kernel, before = m[1], []
                kernels.add(kernel)
            continue
        text = line.split("//", 1)[0].strip()
        op, _, rest = text.partition(" ")
        operands = [x.split()[0] if x.split() else "" for x in rest.split(",")]
        writes = set()
        if op.startswith("v_"):
            vector += 1
            # (add with carry, division and 64-bit multiply-add write a scalar behind the result)
            n_out = 2 if re.match(r"v_(add|sub|subrev|addc|subb|subbrev)_co|v_div_scale|v_mad_[iu]64", op) else 1
            for x in operands[:n_out]:
                writes |= _registers(x)
            reads = set().union(*(_registers(x) for x in operands[n_out:])) if len(operands) > n_out else set()
            found += [(kernel, w, text) for w, written in before if written & reads]
        before = ([(text, writes)] + before)[:2]
        if op == "s_nop":
            before = ([("", set())] * int(operands[0], 0) + before)[:2]
    return kernels, vector, found


def _listings(library):
    objdump = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")
    objdump = objdump if os.path.exists(objdump) else shutil.which("llvm-objdump")
    if not objdump:
        pytest.skip("needs llvm-objdump")
    for code in _code_objects(library):
        out = subprocess.run([objdump, "-d", "--no-show-raw-insn", "-"], input=code, stdout=subprocess.PIPE, check=True)
        yield out.stdout.decode().splitlines()


def test_two_wait_states_between_a_scalar_written_and_read_by_vector_instructions():
    """gfx950 gives a vector instruction the old value of a scalar that another wrote less than two wait states before.
    The compiler keeps its own instructions apart, but not those in assembly (the encoders' steps: a compare at the end of
    one and a select on its mask in the next)."""
    kernels, vector, found = set(), 0, []
    for listing in _listings(plc.LIB_PATH):
        k, v, f = scalars_read_too_early(listing)
        kernels, vector, found = kernels | k, vector + v, found + f
    assert sum("rans_encode_pipe_kernel" in k for k in kernels) >= 5 and sum("rans_encode_short_kernel" in k for k in kernels) >= 3
    assert vector > 100_000
    assert not found, f"{len(found)}, the first: {found[0]}"


def test_the_check_sees_what_it_is_for():
    listing = ["0000000000000000 <kernel>:", "\tv_cmp_gt_u32_e32 vcc, v1, v2 // 0: 00", None,
               "\tv_cndmask_b32_e32 v3, v4, v5, vcc // 8: 00"]
    for between, early in (([], 1), (["\ts_waitcnt lgkmcnt(4)"], 1), (["\ts_nop 0"], 1), (["\ts_nop 1"], 0),
                           (["\ts_waitcnt lgkmcnt(4)", "\tv_add_u32_e32 v4, v6, v7"], 0)):
        assert len(scalars_read_too_early(listing[:2] + between + listing[3:])[2]) == early
    wide = ["0000000000000000 <kernel>:", "\tv_cmp_lt_u32_e64 s[4:5], v1, v2", "\tv_bcnt_u32_b32 v3, s5, 0"]
    assert len(scalars_read_too_early(wide)[2]) == 1

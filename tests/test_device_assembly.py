"""What the compiler cannot see in hand-written assembly: registers that it changes, and products whose results take
longer than an instruction.  The first is looked for in the sources, the second in the code the compiler makes of them."""
from __future__ import annotations

import glob
import os
import re
import struct
import subprocess

import pytest

from paper_2406_06220_amd import build

CSRC = os.path.join(build.PKG, "csrc")


def asm_statements():
    for path in sorted(glob.glob(os.path.join(CSRC, "*.h*"))):
        src = open(path).read()
        for m in re.finditer(r"\basm\s+volatile\s*\((.*?)\);", src, flags=re.S):
            yield os.path.basename(path), m.group(1)


def test_assembly_that_writes_m0_says_so():
    writes = [(f, s) for f, s in asm_statements() if re.search(r"\bs_\w+ m0\b", s)]
    assert writes
    for f, s in writes:
        assert re.search(r':[^:]*"m0"[^:]*$', s), f"{f}: {s}"


def instructions(source, kernel, out):
    """The instructions of one kernel of a file, in order: (mnemonic, operands)."""
    flags = [f for f in build.HIPCC_FLAGS if f != "-shared"]
    subprocess.run(["hipcc", *flags, "-I", os.path.join(build.ROOT, "include"), "-I", CSRC, "-S", "--cuda-device-only", source,
                    "-o", out], check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    code, inside = [], False
    for line in open(out):
        line = line.split(";")[0].strip()
        if re.match(rf"\w*{kernel}\w*:", line):
            inside = True
        elif inside and line and not line.startswith(".") and not line.endswith(":"):
            op, _, rest = line.partition(" ")
            code.append((op, [o.strip() for o in rest.split(",")]))
            if op == "s_endpgm":
                return code
    raise AssertionError("the kernel was not found")


@pytest.fixture(scope="module")
def big_kernel(tmp_path_factory):
    return instructions(os.path.join(CSRC, "enc_proj.hip"), "enc_proj_bf16_big_kernel", str(tmp_path_factory.mktemp("asm") / "enc_proj.s"))


WORDS = r"""
#include "exchange.h"
using namespace tdt;
__global__ void words_kernel(const unsigned long long *a, unsigned long long *b, int n)
{
    const int lane = threadIdx.x * 8;
    const __amdgpu_buffer_rsrc_t in = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned long long *>(a), 0, n, 0x00020000);
    const __amdgpu_buffer_rsrc_t out = __builtin_amdgcn_make_buffer_rsrc(b, 0, n, 0x00020000);
    const unsigned long long x = ld_co64(a + threadIdx.x);
    const unsigned long long y = ld_word64(in, lane, 4096);
    st_co64(b + 64 + threadIdx.x, y);
    st_word64(out, lane, 0, x);
}
"""


def test_words_move_like_atomics(tmp_path):
    """An 8-byte word through a buffer descriptor is one access of the width and the scope that an agent-scope atomic of 8
    bytes is."""
    src = tmp_path / "words.hip"
    src.write_text(WORDS)
    code = instructions(str(src), "words_kernel", str(tmp_path / "words.s"))
    moves = {op: o for op, o in code if re.match(r"(global|flat|buffer)_(load|store|atomic)", op)}
    assert sorted(moves) == ["buffer_load_dwordx2", "buffer_store_dwordx2", "global_load_dwordx2", "global_store_dwordx2"]
    scope = lambda op: [w for w in moves[op][-1].split() if w in ("sc0", "sc1", "nt")]   # noqa: E731
    assert all(scope(op) == ["sc1"] for op in moves)


def registers(operand):
    m = re.match(r"([va])\[(\d+):(\d+)\]$", operand)
    if m:
        return {f"{m[1]}{i}" for i in range(int(m[2]), int(m[3]) + 1)}
    return {operand} if re.match(r"[va]\d+$", operand) else set()


def test_products_are_read_behind_their_wait(big_kernel):
    """Sixteen cycles a product and more: nothing but another product touches an accumulator from the first product to the
    wait behind the last."""
    products = [i for i, (op, _) in enumerate(big_kernel) if op.startswith("v_mfma")]
    waits = [i for i, (op, o) in enumerate(big_kernel) if op == "s_nop" and o == ["15"]]
    assert len(products) == 80 and len(waits) == 2 and waits[1] == waits[0] + 1 and products[-1] < waits[0]
    for op, operands in big_kernel[products[0]:waits[0]]:
        if not op.startswith("v_mfma"):
            assert not any(r[0] == "a" for o in operands for r in registers(o)), (op, operands)
    assert any(r[0] == "a" for op, operands in big_kernel[waits[1]:] for o in operands for r in registers(o))


def test_products_do_not_follow_what_makes_their_operands(big_kernel):
    """A product may read a vector register two instructions after the vector ALU wrote it: fragments come from LDS, and no
    copy of one stands that close in front of a product."""
    for i, (op, operands) in enumerate(big_kernel):
        if op.startswith("v_mfma"):
            needs = registers(operands[1]) | registers(operands[2])
            for before, o in big_kernel[max(0, i - 2):i]:
                if before.startswith("v_") and not before.startswith("v_mfma"):
                    assert not registers(o[0]) & needs, (before, o, op, operands)


def scratch_bytes(library, directory):
    """Bytes of scratch memory a lane of every kernel of a library takes, as its code objects say."""
    data, magic, found, at = open(library, "rb").read(), b"__CLANG_OFFLOAD_BUNDLE__", {}, -1
    while (at := data.find(magic, at + 1)) >= 0:
        n, = struct.unpack_from("<Q", data, at + len(magic))
        entry = at + len(magic) + 8
        for _ in range(n if n < 16 else 0):   # (more: the name alone, not a bundle)
            off, size, length = struct.unpack_from("<QQQ", data, entry)
            target = data[entry + 24:entry + 24 + length]
            entry += 24 + length
            if b"gfx950" in target and size:
                path = directory / "code.o"
                path.write_bytes(data[at + off:at + off + size])
                notes = subprocess.run(["/opt/rocm/llvm/bin/llvm-readelf", "--notes", str(path)], check=True,
                                       stdout=subprocess.PIPE, text=True).stdout
                names = re.findall(r"^ +\.name: +(_Z\S+)$", notes, re.M)
                sizes = re.findall(r"^ +\.private_segment_fixed_size: +(\d+)$", notes, re.M)
                assert len(names) == len(sizes)
                found.update(zip(names, map(int, sizes)))
    return found


def test_scratch_memory_of_the_label_loop(tmp_path):
    """A value in scratch memory is a trip to memory in the middle of a label, so the forms of the kernel that have any are
    known: chunks in float32 of larger groups with two rounds, and of one bfloat16 layer to 1024."""
    if not os.path.exists(build.LIB):
        pytest.skip("the library has not been built")
    label = {n: b for n, b in scratch_bytes(build.LIB, tmp_path).items() if "label_kernel" in n}
    assert len(label) > 40
    known = ("IfLi1ELb1ELi10ELi4ELi4ELi16E", "ItLi1ELb1ELi8ELi4ELi2ELi16E")
    for name, size in label.items():
        assert size == 0 or (size <= 64 and any(k in name for k in known)), (name, size)

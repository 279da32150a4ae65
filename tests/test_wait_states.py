"""Matrix products of the built library: nothing reads or overwrites a product's registers before they are written, on any path.

The hardware does not wait for them; the compiler puts the wait in, but where two paths of different length meet it has been seen to
count the longer one only (sums read three instructions behind their last product came out without it). A product by 16-bit
operands is readable its passes + 4 instructions later, one by floats its passes + 2 (what the compiler keeps within a block)."""
import bisect
import os
import re
import shutil
import subprocess

import pytest

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
SLOTS = {"v_mfma_f32_16x16x32_bf16": 8, "v_mfma_f32_16x16x32_f16": 8, "v_mfma_f32_32x32x16_bf16": 12, "v_mfma_f32_32x32x16_f16": 12,
         "v_mfma_f32_32x32x2_f32": 18}
READERS = ("v_", "ds_", "buffer_", "global_", "flat_", "scratch_")


def _registers(text):
    out = set()
    for kind, first, last, one in re.findall(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+))", text):
        out.update((kind, i) for i in (range(int(first), int(last) + 1) if not one else (int(one),)))
    return out


def _decode(text):
    """(operation, registers of the first operand, of the next two, of all, instructions that it counts for)"""
    op, _, rest = text.partition(" ")
    parts = rest.split(", ")
    return op, _registers(parts[0]), _registers(" ".join(parts[1:3])), _registers(rest), int(rest, 0) + 1 if op == "s_nop" else 1


def _functions(listing):
    """name -> [(address, text, branch target or None)]"""
    out, now = {}, None
    for line in listing.splitlines():
        head = re.match(r"^([0-9a-f]+) <(.*)>:$", line)
        if head:
            now = out.setdefault(head.group(2), [])
            continue
        m = re.match(r"^\s+(\S.*?)\s*// ([0-9A-F]+):", line)
        if m and now is not None:
            text, at = m.group(1), int(m.group(2), 16)
            jump = re.match(r"^s_c?branch\S* (\d+)", text)
            offset = int(jump.group(1)) if jump else 0
            now.append((at, text, at + 4 + 4 * (offset - 65536 if offset >= 32768 else offset) if jump else None))
    return out


def _early(code):
    """[(product, reader, instructions between)]"""
    address = [x[0] for x in code]
    decoded = [_decode(x[1]) for x in code]
    found = []
    for i, (op, dst, _, _, _) in enumerate(decoded):
        if not op.startswith("v_mfma"):
            continue
        paths, seen = [(i + 1, 0)], set()
        while paths:
            j, slots = paths.pop()
            if j >= len(code) or slots >= SLOTS[op] or (j, slots) in seen:
                continue
            seen.add((j, slots))
            other, first, operands, every, count = decoded[j]
            if other.startswith("v_mfma"):
                if operands & dst:
                    found.append((code[i][1], code[j][1], slots))
                if first & dst:
                    continue          # an accumulator is handed on
            elif other.startswith(READERS) and every & dst:
                found.append((code[i][1], code[j][1], slots))
                continue
            if code[j][2] is not None:
                paths.append((bisect.bisect_left(address, code[j][2]), slots + count))
            if not other.startswith(("s_branch", "s_endpgm")):
                paths.append((j + 1, slots + count))
    return found


def _listing(lines):
    return "\n".join(["0000000000000000 <k>:"] + [f"\t{text}  // {4 * i:012X}: 00000000" for i, text in enumerate(lines)])


def test_paths_of_different_length():
    product = "v_mfma_f32_32x32x16_bf16 v[0:15], v[16:19], v[20:23], 0"
    body = [product, "s_cbranch_scc1 4"] + ["s_add_i32 s0, s0, 1"] * 4

    def early(wait, reader="v_add_f32_e32 v30, v15, v31"):
        return _early(_functions(_listing(body + [f"s_nop {wait}", reader, "s_endpgm"]))["k"])
    assert early(10) == []                                   # the branch and eleven more
    assert [x[2] for x in early(6)] == [8]                   # enough for the path that takes no branch
    assert early(6, "v_add_f32_e32 v30, v29, v31") == []     # other registers
    assert [x[2] for x in early(9, "v_mfma_f32_32x32x16_bf16 v[32:47], v[12:15], v[20:23], 0")] == [11]
    assert early(0, "v_mfma_f32_32x32x16_bf16 v[0:15], v[24:27], v[20:23], v[0:15]") == []


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
def test_built_library(tmp_path):
    import paper_2507_17245_amd.build as build
    if not os.path.exists(build.OUT):
        build.build()
    shutil.copy(build.OUT, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp_path, check=True, stdout=subprocess.DEVNULL)
    products = 0
    for name in sorted(x for x in os.listdir(tmp_path) if "amdgcn" in x):
        text = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", name], cwd=tmp_path, check=True, stdout=subprocess.PIPE, text=True).stdout
        for kernel, code in _functions(text).items():
            products += sum(x[1].startswith("v_mfma") for x in code)
            assert _early(code) == [], kernel
    assert products > 1000

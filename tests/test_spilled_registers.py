"""Registers that the bf16 forward kernels of the built library spill: none but where a tile's scores and outputs do not fit the file,
and there no more than the products themselves take (code beside the loop that keeps its addresses alive through it has doubled them)."""
import os
import re
import shutil
import subprocess

import pytest

BIN = "/opt/rocm/llvm/bin/"
# <d, Br, Bc, contraction, mode (0 exact, 1 K_f, 2 Q~), groups, halves>
SPILLED = {(128, 128, 64, 16, 1, 8, 1): 14, (128, 128, 64, 16, 1, 8, 2): 18, (128, 256, 128, 128, 0, 128, 1): 35,
           (128, 256, 128, 128, 2, 128, 1): 52, (128, 256, 128, 16, 1, 16, 1): 229, (128, 256, 128, 32, 1, 32, 1): 156,
           (128, 256, 128, 64, 1, 64, 1): 175, (128, 256, 64, 16, 1, 8, 1): 12, (128, 64, 128, 32, 1, 32, 1): 19,
           (128, 64, 128, 64, 1, 64, 1): 49, (128, 64, 64, 16, 1, 8, 1): 18, (128, 64, 64, 16, 1, 8, 2): 18,
           (64, 128, 128, 32, 1, 32, 1): 4, (64, 64, 128, 16, 1, 16, 1): 33}


@pytest.mark.skipif(not os.path.exists(BIN + "llvm-readelf"), reason="no reader of the metadata")
def test_forward_kernels(tmp_path):
    import paper_2507_17245_amd.build as build
    if not os.path.exists(build.OUT):
        build.build()
    shutil.copy(build.OUT, tmp_path / "lib.so")
    subprocess.run([BIN + "llvm-objdump", "--offloading", "lib.so"], cwd=tmp_path, check=True, stdout=subprocess.DEVNULL)
    seen = {}
    for name in sorted(x for x in os.listdir(tmp_path) if "amdgcn" in x):
        notes = subprocess.run([BIN + "llvm-readelf", "--notes", name], cwd=tmp_path, check=True, stdout=subprocess.PIPE, text=True).stdout
        for kernel, spilled in re.findall(r"\.name: +(_Z\S+)\n(?:.*\n)*?.*\.vgpr_spill_count: +(\d+)", notes):
            m = re.search(r"attn_bf16_kernelI((?:Li\d+E)+)", kernel)
            if m:
                key = tuple(map(int, re.findall(r"\d+", m.group(1))))
                seen[key] = max(seen.get(key, 0), int(spilled))
    assert len(seen) > 50 and SPILLED.keys() <= seen.keys()
    assert {k: n for k, n in seen.items() if n > SPILLED.get(k, 0)} == {}

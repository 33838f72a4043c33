"""What the compiler made of the device code of the built library (gfx950 assembly of this
repository's own sources)."""
from __future__ import annotations

import os
import re
import subprocess

import pytest

from paper_2507_03092_amd import build

LLVM = os.path.join(os.path.dirname(os.path.dirname(build.HIPCC)), "llvm", "bin")


@pytest.fixture(scope="module")
def functions(tmp_path_factory):
    """Instructions by (mangled) name of the library's device functions."""
    tool = {t: os.path.join(LLVM, t) for t in ("llvm-objcopy", "clang-offload-bundler", "llvm-objdump")}
    if not all(os.path.exists(t) for t in tool.values()):
        pytest.skip("llvm tools not available")
    lib = build.build(force=False)
    tmp = tmp_path_factory.mktemp("device_code")
    fat, obj = str(tmp / "fat.bin"), str(tmp / "dev.o")
    subprocess.check_call([tool["llvm-objcopy"], "--dump-section", f".hip_fatbin={fat}", lib, str(tmp / "copy.so")])
    subprocess.check_call([tool["clang-offload-bundler"], "--unbundle", "--type=o", f"--input={fat}", f"--output={obj}",
                           "--targets=hipv4-amdgcn-amd-amdhsa--gfx950"])
    text = subprocess.check_output([tool["llvm-objdump"], "-d", "--no-show-raw-insn", "--no-leading-addr", obj], text=True)
    out, name = {}, None
    for line in text.splitlines():
        m = re.match(r"<(\S+)>:$", line)
        if m:
            name = m[1]
            out[name] = []
        elif name and line.startswith("\t"):
            out[name].append(line.split("//")[0].strip())
    return out


@pytest.mark.parametrize("part", ["batch_segment", "batch_window", "batch_measure_fast", "batch_dets", "batch_measure_slow"])
def test_parts_of_the_batch_kernel_save_no_registers(functions, part):
    """A part's callee-saved vector registers (every other eight from v40 on) are not stored at its entry."""
    found = {n: f for n, f in functions.items() if re.search(rf"\d{part}I", n)}
    assert found
    for name, f in found.items():
        saved = []
        for ins in f[:80]:
            m = re.match(r"scratch_store_dword off, v(\d+), s32", ins)
            if m:
                saved.append(int(m[1]))
        # (a few spilled scalars go through registers of their own, from the top down)
        assert len(saved) <= 8, (name, saved)

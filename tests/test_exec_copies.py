"""The compiled code of every kernel, checked on the CPU for one compiler fault: a
register saved (to an accumulation register or to scratch memory) in the block
where a divergent region ends, before that block gives the other lanes back.  Only
the region's lanes then hold the saved value; a store through it in another lane
goes anywhere."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2609_01864_amd import credit

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def saves_before_restore(lines):
    """(kernel, instruction) of each save between a label and the block's restore of exec."""
    out, kernel, held = [], None, None
    for line in lines:
        if line.endswith(">:"):
            name = line[line.index("<") + 1:-2]
            if name.startswith("_Z"):
                kernel = name
            held = []
            continue
        text = line.split("//")[0].strip()
        if held is None or not text:
            continue
        if text.startswith("s_or_b64 exec, exec,"):
            out += [(kernel, h) for h in held]
            held = None
        elif text.startswith(("s_cbranch", "s_branch", "s_endpgm", "s_and_saveexec", "s_mov_b64 exec,")):
            held = None
        elif text.startswith(("v_accvgpr_write", "v_accvgpr_mov", "scratch_store")):
            held.append(text)
    return out


def test_the_scan_sees_such_a_copy():
    head = ["0000000000001000 <_Zk>:", "<L48>:"]
    save, back = "\tv_accvgpr_write_b32 a43, v7 // 0", "\ts_or_b64 exec, exec, s[58:59] // 2"
    assert saves_before_restore(head + [save, "\ts_nop 0 // 1", back]) == [("_Zk", "v_accvgpr_write_b32 a43, v7")]
    assert saves_before_restore(head + ["\ts_nop 0 // 1", back, save]) == []


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
def test_no_kernel_saves_a_register_before_its_lanes_are_back(lib_built, tmp_path):
    shutil.copy(credit.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)
    kernels, found = set(), []
    for f in sorted(tmp_path.glob("lib.so.*gfx950")):
        p = subprocess.run([OBJDUMP, "-d", "--symbolize-operands", "--no-show-raw-insn", f.name], cwd=tmp_path,
                           check=True, capture_output=True, text=True)
        kernels |= set(re.findall(r"^[0-9a-f]+ <(_Z\w+)>:", p.stdout, re.M))
        found += saves_before_restore(p.stdout.splitlines())
    assert any("k_resident" in k for k in kernels) and any("k_stream" in k for k in kernels)
    assert found == []

"""The library's own gfx950 code, disassembled: instructions that stand in inline assembly, where the compiler keeps no wait states."""
import glob
import os
import re
import shutil
import subprocess

import pytest

import paper_1901_06887_amd as mt

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_wide_stores_in_asm_wait_until_their_data_may_be_overwritten(tmp_path):
    """A vector instruction may overwrite the data of a store wider than 8 bytes two wait states behind it (the compiler puts `s_nop 1`
    there, on gfx950 as on gfx942); behind a store in inline assembly it puts nothing, so the assembly brings them."""
    mt.load_library()
    lib = shutil.copy(os.path.join(os.path.dirname(mt.__file__), "libmt.so"), tmp_path)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, stdout=subprocess.DEVNULL, cwd=tmp_path)
    seen = 0
    for obj in glob.glob(str(tmp_path / "*gfx950*")):
        code = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", obj], check=True, stdout=subprocess.PIPE, text=True).stdout.splitlines()
        for store, behind in zip(code, code[1:]):
            if re.search(r"global_store_dwordx4 .* off sc1", store):
                nop = re.search(r"s_nop (\d+)", behind)
                assert nop and int(nop.group(1)) >= 1, (store, behind)
                seen += 1
    assert seen > 0

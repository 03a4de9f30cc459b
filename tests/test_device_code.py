"""The library's own gfx950 code, disassembled: instructions that stand in inline assembly, where the compiler keeps no wait states."""
import glob
import os
import re
import shutil
import subprocess

import pytest

import paper_1901_06887_amd as mt

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
READELF = "/opt/rocm/llvm/bin/llvm-readelf"


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


def kernel_resources(tmp_path):
    """{mangled kernel name: (bytes of scratch memory a lane, vector registers)} of the library, from its code objects' notes."""
    mt.load_library()
    lib = shutil.copy(os.path.join(os.path.dirname(mt.__file__), "libmt.so"), tmp_path)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, stdout=subprocess.DEVNULL, cwd=tmp_path)
    found = {}
    for obj in glob.glob(str(tmp_path / "*gfx950*")):
        notes = subprocess.run([READELF, "--notes", obj], check=True, stdout=subprocess.PIPE, text=True).stdout
        for entry in re.split(r"\n  - ", notes)[1:]:
            name = re.findall(r"\.name:\s+(_Z\w+)", entry)
            if name:
                found[name[-1]] = tuple(int(re.search(r"\.%s:\s+(\d+)" % key, entry).group(1)) for key in ("private_segment_fixed_size", "vgpr_count"))
    return found


@pytest.mark.skipif(not os.path.exists(READELF), reason="no llvm-readelf")
def test_narrow_fc_kernels_keep_to_the_registers_of_four_workgroups(tmp_path):
    """Every FC launch of a small run takes one of these: what only last layers of 33 to 128 classes need has kernels of its own, and no register of either goes to scratch memory."""
    narrow = {n: r for n, r in kernel_resources(tmp_path).items() if re.search(r"9fc_kernelI\w+Lb1ELi\d", n)}
    assert len(narrow) >= 12
    assert all(scratch == 0 for scratch, _ in narrow.values()), narrow
    assert all(registers <= 107 for n, (_, registers) in narrow.items() if not re.search(r"Lb1ELi0ELb\dELb1E", n)), narrow

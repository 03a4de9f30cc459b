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
    """{mangled kernel name: (bytes of scratch memory a lane, vector registers, bytes of LDS)} of the library, from its code objects' notes."""
    mt.load_library()
    lib = shutil.copy(os.path.join(os.path.dirname(mt.__file__), "libmt.so"), tmp_path)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, stdout=subprocess.DEVNULL, cwd=tmp_path)
    found = {}
    for obj in glob.glob(str(tmp_path / "*gfx950*")):
        notes = subprocess.run([READELF, "--notes", obj], check=True, stdout=subprocess.PIPE, text=True).stdout
        for entry in re.split(r"\n  - ", notes)[1:]:
            name = re.findall(r"\.name:\s+(_Z\w+)", entry)
            if name:
                found[name[-1]] = tuple(int(re.search(r"\.%s:\s+(\d+)" % key, entry).group(1)) for key in ("private_segment_fixed_size", "vgpr_count", "group_segment_fixed_size"))
    return found


@pytest.mark.skipif(not os.path.exists(READELF), reason="no llvm-readelf")
def test_narrow_fc_kernels_keep_to_the_registers_of_four_workgroups(tmp_path):
    """Every FC launch of a small run takes one of these: what only last layers of 33 to 128 classes need has kernels of its own, and no register of either goes to scratch memory."""
    narrow = {n: r for n, r in kernel_resources(tmp_path).items() if re.search(r"9fc_kernelI\w+Lb1ELi\d", n)}
    assert len(narrow) >= 12
    assert all(r[0] == 0 for r in narrow.values()), narrow
    assert all(r[1] <= 107 for n, r in narrow.items() if not re.search(r"Lb1ELi0ELb\dELb1E", n)), narrow


@pytest.mark.skipif(not os.path.exists(READELF), reason="no llvm-readelf")
def test_facts_ahead_cost_no_frame_tile_its_place(tmp_path):
    """LDS is dealt out in 1280 bytes, 160 KiB to a compute unit.  What a frame tile has beside its input rows leaves room for as many workgroups as the lookup's 16 bytes did,
    unless the whole launch starts at once; the kernels hold what the rule reckons with."""
    fixed = {n: r[2] for n, r in kernel_resources(tmp_path).items() if re.search(r"15conv_img_kernel", n)}
    assert {f for n, f in fixed.items() if not re.search(r"Lb1EEEvNS", n)} == {16}
    with_facts = {f for n, f in fixed.items() if re.search(r"Lb1EEEvNS", n)}
    assert len(with_facts) == 1 and with_facts.pop() == 32 * 36 * 4
    fit = lambda lds, blocks: min(4 if blocks == 2 else 3, 128 // -(-lds // 1280))  # noqa: E731
    taken = 0
    for blocks in (2, 3, 4):
        for frame in range(8 * 1024, 96 * 1024 + 1, 208):
            without, ahead = fit(frame + 16, blocks), fit(frame + 32 * 36 * 4, blocks)
            for grid in (8, 256 * ahead, 256 * ahead + 8, 1 << 16):
                got = mt.debug_conv_frame_ahead(32, blocks, frame, grid)
                assert got == (ahead == without or grid <= 256 * ahead), (blocks, frame, grid)
                taken += got and ahead < without
                assert not mt.debug_conv_frame_ahead(33, blocks, frame, grid) and not mt.debug_conv_frame_ahead(32, 1, frame, grid)
    assert taken > 0


@pytest.mark.skipif(not os.path.exists(READELF), reason="no llvm-readelf")
def test_no_kernel_keeps_registers_in_scratch_memory(tmp_path):
    kernels = kernel_resources(tmp_path)
    assert len(kernels) > 100
    assert not {n: r for n, r in kernels.items() if r[0]}

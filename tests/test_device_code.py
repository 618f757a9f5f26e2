"""What the compiler made of the kernels, read from the gfx950 assembly of the library's own source.  CPU only."""
import os
import re
import subprocess

import pytest

from paper_2302_02599_amd import build


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("asm") / "ckpt_dp.s")
    flags = [f for f in build.HIPCC_FLAGS if f != "-shared"]
    subprocess.check_call([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "--cuda-device-only", "-S", "-I",
                           os.path.join(build.ROOT, "include"), "-x", "hip", os.path.join(build.CSRC, "ckpt_dp.hip"), "-o", out],
                          stderr=subprocess.DEVNULL)
    return open(out, encoding="utf-8").read()


def kernels(assembly):
    for part in assembly[assembly.index("amdhsa.kernels:"):].split("  - .agpr_count")[1:]:
        name = re.search(r"\.name: +(_Z\S+)", part)[1]
        yield name, {k: int(v) for k, v in re.findall(r"\.(\w+): +(\d+)\n", part)}


def test_no_kernel_spills_vector_registers(assembly):
    """A spilled register is a store and a load of its own, which wait for the accesses before them: in the block product
    they undid the order of requests and stores."""
    seen = dict(kernels(assembly))
    assert sum("gemm_kernel" in n for n in seen) == 6 and sum("tile_rows_kernel" in n for n in seen) == 6
    for name, k in seen.items():
        assert k["vgpr_spill_count"] == 0, (name, k["vgpr_spill_count"])
        assert k["private_segment_fixed_size"] == 0, (name, k["private_segment_fixed_size"])


WIDE_STORE = re.compile(r"^\s*buffer_store(?:_format)?_(?:dwordx[34]|xyzw?)\s+(.*)$", re.M)


def scalar_offsets(assembly):
    """The scalar offset of every buffer store of more than 8 bytes: the operand behind data, address and descriptor."""
    for operands in WIDE_STORE.findall(assembly):
        m = re.match(r"[va](?:\[\d+:\d+\]|\d+), *(?:v\d+|v\[\d+:\d+\]|off), *s\[\d+:\d+\], *(\S+)", operands)
        assert m, operands
        yield m[1]


def test_no_wide_store_has_a_scalar_offset_register(assembly):
    """Behind a buffer store of more than 8 bytes a lane with a scalar offset register the compiler keeps no distance to an
    instruction that overwrites its data, and the overwritten value was seen in memory.  Without that register it does."""
    planted = "\tbuffer_store_dwordx4 v[2:5], v21, s[16:19], s7 offen nt\n\tbuffer_store_dwordx3 v[2:4], off, s[0:3], 0\n"
    assert list(scalar_offsets(planted)) == ["s7", "0"]
    found = list(scalar_offsets(assembly))
    assert len(found) >= 2 * 3  # the wide rows of three variants of the block product
    assert all(re.fullmatch(r"\d+|0x[0-9a-f]+", o) for o in found), sorted(set(found))


def test_wide_stores_to_a_table_go_through_the_one_function():
    """That function takes no scalar offset."""
    text = open(os.path.join(build.CSRC, "ckpt_dp.hip"), encoding="utf-8").read()
    calls = re.findall(r"__builtin_amdgcn_raw_buffer_store_b(?:96|128)\(.*", text)
    assert calls == ["__builtin_amdgcn_raw_buffer_store_b128(v, tab, voff, 0, policy);"]

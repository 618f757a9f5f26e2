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

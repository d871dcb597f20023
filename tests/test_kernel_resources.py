"""Registers of the built kernels, from the library's own metadata: no kernel that
runs every sweep keeps registers in memory, and the argument layout still spares the
FP64 sweep kernels most of their scalar spills (see SweepParams::pad)."""
import glob
import os
import re
import subprocess

import pytest

from paper_2311_02101_amd import hp

LLVM = "/opt/rocm/llvm/bin/"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not (os.path.exists(hp.LIB_PATH) and os.path.exists(LLVM + "llvm-readelf")):
        pytest.skip("needs the built library and ROCm's LLVM tools")
    d = str(tmp_path_factory.mktemp("code"))
    os.symlink(hp.LIB_PATH, os.path.join(d, "lib.so"))
    subprocess.run([LLVM + "llvm-objdump", "--offloading", "lib.so"], cwd=d, check=True, capture_output=True)
    notes = "".join(subprocess.run([LLVM + "llvm-readelf", "--notes", f], check=True, capture_output=True,
                                   text=True).stdout for f in glob.glob(d + "/*gfx950"))
    found = re.findall(r"\.name:\s+(\S+)\n.*?\.private_segment_fixed_size: (\d+).*?\.sgpr_spill_count: (\d+)", notes,
                       re.S)
    return {name: (int(private), int(sgpr)) for name, private, sgpr in found}


def test_no_registers_in_memory(kernels):
    assert len(kernels) > 80
    # the FP64 pull kernel with four averages per thread parks two registers
    bad = {k: v[0] for k, v in kernels.items() if v[0] > (16 if "sweep_pull_kernelIdLi4E" in k else 0)}
    assert not bad


# scalar spills with the eight bytes of padding / without: 79 / 117 in the padded
# split, 46 / 55 in the size-clustered one, 73 / 85 with one variable per thread
@pytest.mark.parametrize("kernel,most", [("sweep_split_kernelIdLi1ELb0ELb0ELb0E", 90),
                                         ("sweep_split_kernelIdLi1ELb1ELb0ELb0E", 50),
                                         ("sweep_push_kernelIdLin1ELi1ELb0ELb0ELb0E", 79)])
def test_argument_layout_spares_scalar_spills(kernels, kernel, most):
    got = [v[1] for k, v in kernels.items() if kernel in k]
    assert len(got) == 1 and got[0] <= most

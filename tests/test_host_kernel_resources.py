"""Registers of the built kernels: waves per SIMD that a kernel must not lose, read
from the resource notes of the library's own code objects."""
import os
import re
import subprocess

import pytest

from paper_2310_16298_amd import build as hipbuild
from paper_2310_16298_amd import stencil as st

LLVM = os.path.join(os.path.dirname(hipbuild.HIPCC), "..", "llvm", "bin")


@pytest.fixture(scope="module")
def registers(tmp_path_factory):
    """Mangled kernel name -> vector registers (accumulation registers included), spilled scalar ones."""
    st.load_library()
    tmp = tmp_path_factory.mktemp("kernels")
    fat = str(tmp / "fat")
    subprocess.run([os.path.join(LLVM, "llvm-objcopy"), "--dump-section", ".hip_fatbin=" + fat, hipbuild.LIB,
                    str(tmp / "rest")], check=True)
    data = open(fat, "rb").read()
    at = [m.start() for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__|CCOB", data)] + [len(data)]
    regs = {}
    for k in range(len(at) - 1):
        bundle, obj = str(tmp / f"bundle{k}"), str(tmp / f"obj{k}")
        with open(bundle, "wb") as f:
            f.write(data[at[k]:at[k + 1]])
        res = subprocess.run([os.path.join(LLVM, "clang-offload-bundler"), "--type=o", "--unbundle", "--input=" + bundle,
                              "--output=" + obj, "--targets=hipv4-amdgcn-amd-amdhsa--gfx950"], capture_output=True)
        if res.returncode != 0 or not os.path.getsize(obj):
            continue
        notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", obj], capture_output=True, text=True,
                               check=True).stdout
        for m in re.finditer(r"\.sgpr_spill_count:\s+(\d+)\s+\.symbol:\s+'?([^\s']+)\.kd.*?\.vgpr_count:\s+(\d+)",
                             notes, re.S):
            regs[m.group(2)] = (int(m.group(3)), int(m.group(1)))
    assert len(regs) > 500
    return regs


def _of(registers, *parts):
    found = {n: v for n, v in registers.items() if all(p in n for p in parts)}
    assert found, parts
    return found


def test_batched_fp64_order1_outer_products_run_two_waves(registers):
    # 512 vector registers per SIMD lane
    for name, v in _of(registers, "mfma2d_batchIdLi1E").items():
        assert v[0] <= 256, (name, v)


def test_two_step_stream_of_order_3_runs_two_waves(registers):
    for name, v in _of(registers, "tb3d_stream_kernelIfLi3E").items():
        assert v[0] <= 256, (name, v)
    for name, v in _of(registers, "tb3d_stream_kernelIfLi4E").items():
        assert v[0] <= 300, (name, v)  # one wave; vector weights took 327


def test_batched_two_step_stream_fits_its_workgroups(registers):
    # 5 and 6 waves a workgroup: a CU takes one less past 128 registers
    for part in ("IfLi2ELb0E", "IfLi1ELb1E"):
        for name, v in _of(registers, "tb3d_stream_batch" + part).items():
            assert v[0] <= 128, (name, v)


def test_batched_ring_of_fp64_order_4_boxes_keeps_its_scalars(registers):
    # 57 with a search that stays in scalar registers, 429 with one across the lanes
    for name, v in _of(registers, "gather3d_batchIdLi4ELb1ELb1E").items():
        assert v[1] <= 100, (name, v)

"""The forward GroupNorm kernels form the normalised value with the explicit
fused multiply-add that the backward recomputes the ReLU mask with, not by
leave of the compiler's contraction: read off the compiled kernels (CPU)."""
import os
import re
import subprocess

import pytest

from paper_1911_00357_amd import build as B


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Kernel name -> LLVM IR of norm.hip for gfx950."""
    ll = tmp_path_factory.mktemp("ir") / "norm.ll"
    flags = [f for f in B.FLAGS if f != "-fPIC"]
    subprocess.run([B.HIPCC, *flags, "-O1", "--cuda-device-only", "-S", "-emit-llvm", "-o", str(ll),
                    os.path.join(B.CSRC, "norm.hip")], check=True, capture_output=True)
    return {m.group(1): m.group(0)
            for m in re.finditer(r"^define [^\n]*@(\w+)\(.*?^}", ll.read_text(), re.S | re.M)}


def fmas(ir):
    return len(re.findall(r"call [^\n]*@llvm\.fma\.f32", ir))


def test_one_launch_forward_forms_every_value_explicitly(kernels):
    fused = {k: ir for k, ir in kernels.items() if "gn_fused_kernel" in k}
    assert len(fused) == 20  # 10 sizes, with and without a second GroupNorm
    for k, ir in fused.items():
        npt, nt, dual = (int(v) for v in re.search(r"ILi(\d+)ELi(\d+)ELb(\d)E", k).groups())
        assert fmas(ir) >= npt * (1 + dual), k


def test_three_launch_forward_and_backward_do_too(kernels):
    want = {"gn_apply_kernel": 4, "gnb_partial_kernelILi2E": 4, "gnb_apply_kernelILi2E": 4,
            "gnb_partial_kernelILi3E": 4, "gnb_apply_kernelILi3E": 4}
    for what, n in want.items():
        ir = [v for k, v in kernels.items() if what in k]
        assert len(ir) == 1 and fmas(ir[0]) >= n, what

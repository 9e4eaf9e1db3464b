"""What the compiler makes of the kernels where no result would show a loss (no GPU)."""
import os
import re
import subprocess

import pytest

from paper_2502_01068_amd import build


def _device_code(source, tmp_path, *extra):
    """The device side of a source, compiled as the library is, to the form that `extra` asks for; and what the compiler said."""
    out = str(tmp_path / "device.out")
    flags = [f for f in build.FLAGS if f not in ("-fPIC", "-shared")]
    res = subprocess.run([build.HIPCC, *flags, "--cuda-device-only", os.path.join(build.CSRC, source), *extra, "-o", out],
                         check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    return out, res.stdout


@pytest.mark.parametrize("source", ["fkv_score.hip", "fkv_score_fused.hip", "fkv_score_keep.hip"])
def test_pooling_forms_can_be_reached(source, tmp_path):
    """Kernel 7 takes two tokens per lane up to 128 owned tokens: a kernel whose rows hold no more (six slots of a row are halo)
    has no code for four."""
    ir = open(_device_code(source, tmp_path, "-S", "-emit-llvm", "-Xclang", "-disable-llvm-passes")[0]).read()
    forms = {(int(stride), int(per)) for stride, per in re.findall(r"^define .*pool7_groupILi(\d+)ELb[01]ELi(\d)E", ir, re.M)}
    assert {per for _, per in forms} == {2, 4}, forms
    assert all(stride - 6 > 128 for stride, per in forms if per == 4), forms


@pytest.mark.parametrize("source", ["fkv_score.hip", "fkv_score_fused.hip", "fkv_score_keep.hip", "fkv_decode.hip", "fkv_wout.hip"])
def test_no_register_goes_to_scratch(source, tmp_path):
    """The kernels whose loops fill the vector registers keep all of them there: a spill is a trip to memory between the loads."""
    said = _device_code(source, tmp_path, "-c", "-Rpass-analysis=kernel-resource-usage")[1]
    kernels = re.findall(r"Function Name: (\S+)", said)
    scratch = [int(n) for n in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", said)]
    spilled = [int(n) for n in re.findall(r" VGPRs Spill: (\d+)", said)]
    assert kernels and len(kernels) == len(scratch) == len(spilled)
    assert not any(scratch) and not any(spilled), list(zip(kernels, scratch, spilled))

"""Registers and scratch memory of the kernels as built: what the build refuses."""
import re

import pytest

from paper_2601_16032_amd import build as hip_build

from .util import device_code, llvm_tool

NAMES = [f"_ZN7sawattn15attn_fwd_kernelILi128ELb{bf16}ELb{causal}ELi2ELb0ELi2EEEvNS_6ParamsE" for bf16 in (0, 1) for causal in (0, 1)]
NAMES += [f"_ZN7sawattn15attn_fwd_kernelILi{d}ELb0ELb0ELi1ELb{halves}ELi2EEEvNS_6ParamsE" for d, halves in ((128, 1), (64, 0))]
NAMES += ["_ZN7sawattn22attn_fwd_shared_kernelILi64ELb0ELb0ELb1EEEvNS_6ParamsE"]


def remarks(**of_one):
    """The compiler's remarks for NAMES, each without scratch or spills but for what `of_one` says of the one at index `at`."""
    lines = []
    for i, name in enumerate(NAMES + ["_ZN7sawattn18bf16_to_f16_kernelEPKDv4_jS2_PS0_S3_m"]):
        mine = of_one if i == of_one.get("at") else {}
        lines += [f"x.hip:1:1: remark: {text} [-Rpass-analysis=kernel-resource-usage]" for text in (
            f"Function Name: {name}", "    VGPRs: 168", f"    ScratchSize [bytes/lane]: {mine.get('scratch', 0)}",
            "    SGPRs Spill: 60", f"    VGPRs Spill: {mine.get('spills', 0)}")]
    return hip_build.kernel_resources("\n".join(lines))


def test_build_refuses_attention_kernels_with_scratch():
    hip_build.check_scratch(remarks())
    for at, name in enumerate(NAMES):
        with pytest.raises(RuntimeError, match=name):
            hip_build.check_scratch(remarks(at=at, scratch=4))
    with pytest.raises(RuntimeError, match="no kernels"):
        hip_build.check_scratch({})


def test_build_refuses_wide_kernels_that_spill_without_scratch():
    """Spills into accumulation registers take no scratch memory but copy registers like others."""
    hip_build.check_wide_kernels(remarks())
    for at, name in enumerate(NAMES[:4]):
        with pytest.raises(RuntimeError, match=f"must not spill.*{name}"):
            hip_build.check_wide_kernels(remarks(at=at, spills=3))


def test_built_kernels_use_no_scratch(tmp_path):
    """The built library's own record of its kernels: no attention kernel has a private segment, none with 256-row tiles spills."""
    notes = llvm_tool("llvm-readelf", "--notes", device_code(tmp_path))
    fields = r"\.name:\s+(_Z\S+)\s+\.private_segment_fixed_size:\s+(\d+).*?\.vgpr_spill_count:\s+(\d+)"
    kernels = {k: (int(scratch), int(spills)) for k, scratch, spills in re.findall(fields, notes, re.S) if "attn_fwd_" in k}
    assert len(kernels) >= 40 and not any(scratch for scratch, _ in kernels.values()), kernels
    wide = {k: spills for k, (_, spills) in kernels.items() if "attn_fwd_kernel" in k and "ELi2ELb" in k}
    assert len(wide) == 4 and not any(wide.values()), wide

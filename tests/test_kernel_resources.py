"""The build refuses kernels whose in-flight LDS reads could be spilled: the
compiler's resource remarks of the present sources, and texts with a fault."""

import os

import pytest

from paper_2609_19868_amd import build

SOUND = """\
x.hip:9:1: remark: Function Name: _Z1kv [-Rpass-analysis=kernel-resource-usage]
    9 | __global__ void k() {
      | ^
x.hip:9:1: remark:     VGPRs: 219 [-Rpass-analysis=kernel-resource-usage]
x.hip:9:1: remark:     ScratchSize [bytes/lane]: 0 [-Rpass-analysis=kernel-resource-usage]
x.hip:9:1: remark:     SGPRs Spill: 21 [-Rpass-analysis=kernel-resource-usage]
x.hip:9:1: remark:     VGPRs Spill: 0 [-Rpass-analysis=kernel-resource-usage]
x.hip:12:3: warning: something
   12 | code
"""


def device_resources(name):
    out = build._run([build._hipcc(), *build.HIPCC_FLAGS, build.RESOURCE_FLAG, "--cuda-device-only", "-c",
                      os.path.join(build.CSRC, name + ".hip"), "-o", os.devnull])
    build.check_kernels(out)
    return build.kernel_resources(out)


def test_check_refuses_scratch_and_vector_spills():
    build.check_kernels(SOUND)
    for good, bad in (("bytes/lane]: 0", "bytes/lane]: 16"), ("VGPRs Spill: 0", "VGPRs Spill: 3")):
        with pytest.raises(RuntimeError, match="_Z1kv"):
            build.check_kernels(SOUND.replace(good, bad))
    assert build.without_remarks(SOUND).splitlines() == ["x.hip:12:3: warning: something", "   12 | code"]


@pytest.mark.parametrize("source,kernel,at_least", [("slot_attn", "slot_attn_bf16_kernel", 4),
                                                    ("slot_conf", "slot_conf_bf16_kernel", 8)])
def test_present_kernels_are_seen_and_sound(source, kernel, at_least):
    r = device_resources(source)
    assert sum(kernel in k for k in r) >= at_least  # every instantiation is looked at
    assert all("VGPRs" in v for v in r.values())


def test_attention_of_64_elements_fits_four_waves_a_simd():
    r = {k: v for k, v in device_resources("slot_attn").items() if "slot_attn_bf16_kernelILi64E" in k}
    assert len(r) == 2 and all(v["VGPRs"] + v["AGPRs"] <= 128 for v in r.values())

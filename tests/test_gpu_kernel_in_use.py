"""info's kernel name is that of the kernel run() launches: joined steps of
small problems, the one-launch and the two-launch form of the split
contraction, and the tiles otherwise."""
import re

import pytest

from paper_2305_07187_amd import instances

from gpu_common import announce, ensure_built, to_dev

pytestmark = pytest.mark.gpu


def _launched(m, steps):
    """Names of the device kernels of one run."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        m.run(steps)
        torch.cuda.synchronize()
    return {e.name for e in prof.events() if "kernel" in e.name}


@pytest.mark.parametrize("n,r,kind,kw,name,kernel", [
    (20, 8, "pm1", {}, "step_f32_small_32x16_w8_mfma16", "small_steps_kernel"),
    (100, 8, "gauss", {}, "step_f32_small_112x16_w8_mfma16", "small_steps_kernel"),
    (200, 64, "pm1", {}, "step_f32_small_224x16_w8_mfma16", "small_steps_kernel"),
    (100, 8, "gauss", {"resident": 2}, r"step_f32_32x32_w2x2_mfma16_k32_s0_a1", "resident_f32_kernel"),
    (1000, 64, "gauss", {}, "step_f32_few_16x32_mfma16_k32_ks4", "step_few_kernel"),
    (2000, 128, "gauss", {}, "step_f32_few_32x32_mfma32_k32_ks4", "step_few_kernel"),
    (5000, 64, "gauss", {}, r"step_f32_128x64_\w+_ks4", "coupling_partial_kernel"),
    (300, 2000, "gauss", {}, r"step_f32_\d+x\d+_\w+_a\d", "step_f32_kernel"),
    (600, 100, "pm1", {}, "step_i8x4_32x16_ks4", "step_i8_few_kernel"),
    (1100, 64, "pm1", {}, "step_i8x4_32x16_ks8", "step_i8_few_kernel"),
    (700, 1001, "pm1", {}, "step_i8x4_256x32_w4_k256_s3", "step_i8_kernel"),
    (700, 961, "gauss", {}, "step_i8x10_128x64_w4_k128_s3", "step_i8_kernel")])
def test_name_and_launch(n, r, kind, kw, name, kernel):
    si = ensure_built()
    announce(f"kernel in use N={n} R={r} {kind} {kw}")
    m = si.SpringIsing(to_dev(instances.make_J(n, kind, 1)), to_dev(instances.make_x0(n, r, 1)), total_steps=40)
    if kw:
        m.set_resident(kw["resident"])
    m.run(8)
    assert re.fullmatch(name, m.info()["kernel_name"]), m.info()["kernel_name"]
    names = _launched(m, 8)
    assert any(kernel in k for k in names), names
    m.close()

"""Registers of the elementwise batch-norm kernels and of the stage boundary's weight gradient, as the compiler reports them: the
statistics rows that they add up first must not cost the waves that hide their own loads (kernel, waves a SIMD at least)."""
import os
import re
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1804_10574_amd", "csrc")
WAVES = {"kernels_elem.hip": [("bn_apply_kernel<ddg::bf16_t>", 7), ("bn_apply_kernel<float>", 7), ("bn_bwd_apply_kernel<ddg::bf16_t>", 7),
                              ("bn_bwd_apply_kernel<float>", 8), ("bn_apply_chunk_kernel<ddg::bf16_t, 1, true>", 5),
                              ("bn_apply_chunk_kernel<ddg::bf16_t, 2, true>", 4), ("bn_apply_pair_kernel<ddg::bf16_t, 4, true>", 4),
                              ("bn_apply_pair_kernel<ddg::bf16_t, 2, true>", 5), ("bn_apply_pair_kernel<ddg::bf16_t, 1, true>", 5)],
         "kernels_wgrad_tiled.hip": [("wgrad_tiled_kernel<32, 64, 8, 2, 1>", 3)]}


@pytest.mark.parametrize("source", sorted(WAVES))
def test_waves_per_simd(source):
    from paper_1804_10574_amd.build import FLAGS, HIPCC
    if not shutil.which(HIPCC) or not shutil.which("c++filt"):
        pytest.skip("needs hipcc and c++filt")
    r = subprocess.run([HIPCC] + FLAGS + ["--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c", os.path.join(CSRC, source), "-o", os.devnull],
                       check=True, capture_output=True, text=True)
    text = subprocess.run(["c++filt"], input=r.stderr, check=True, capture_output=True, text=True).stdout
    waves, name = {}, None
    for line in text.splitlines():
        m = re.search(r"remark:\s+Function Name: (?:void )?(?:ddg::)?(.*?)\(", line)
        name = m[1] if m else name
        m = re.search(r"remark:\s+Occupancy \[waves/SIMD\]: (\d+)", line)
        if m:
            waves[name] = int(m[1])
    for kernel, least in WAVES[source]:
        assert waves[kernel] >= least, (kernel, waves[kernel])

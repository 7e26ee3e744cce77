"""The prefill kernels keep everything in registers (CPU only): what the projection spilled were addresses, whose reloads waited for the rows that were
meant to be on their way during the products."""
import re

from paper_2508_15881_amd import build as b


def test_prefill_kernels_use_no_scratch():
    kernels = {}
    for part in b.device_assembly("prefill_mfma.hip").split("\n  - ")[1:]:
        name, size = re.search(r"\.name:\s+(\S*prefill\S*)", part), re.search(r"\.private_segment_fixed_size:\s+(\d+)", part)
        if name and size:
            kernels[name.group(1)] = int(size.group(1))
    assert sum("prefill_kv_project" in n for n in kernels) == 1 and len(kernels) == 3, kernels
    assert set(kernels.values()) == {0}, kernels

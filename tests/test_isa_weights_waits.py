"""The assembly LDS reads of the weights transform against their waits, with the checker of test_isa_lds_waits.py (CPU only)."""
from paper_2508_15881_amd import build as b
from test_isa_lds_waits import _kernels, check_kernel


def test_weights_transform_reads_are_waited_for():
    kernels = _kernels(b.device_assembly("transform_weights.hip"))
    reads = {n: sum(1 for t, in_asm in k if in_asm and t.startswith("ds_read")) for n, k in kernels.items()}
    assert sorted(r > 0 for r in reads.values()) == [False, False, True, True], reads      # the two column instances
    for name, insts in kernels.items():
        assert not check_kernel(insts), name

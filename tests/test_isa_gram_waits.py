"""The Gram kernel reads its tiles with inline assembly as well: no instruction may touch the destination of such a read
before its wait."""
from paper_2508_15881_amd import build as b
from test_isa_lds_waits import _kernels, check_kernel


def test_gram_kernel_waits_for_its_lds_reads():
    kernels = {n: k for n, k in _kernels(b.device_assembly("pca.hip", ())).items() if "latent_gram_mfma" in n}
    assert len(kernels) == 1
    for insts in kernels.values():
        assert sum(1 for t, in_asm in insts if in_asm and t.startswith("ds_read")) >= 32      # both kinds of block
        assert check_kernel(insts) == []

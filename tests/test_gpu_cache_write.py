"""Cache writes at the widths where the 16-byte pieces of a row are fewer than the lanes of a wave (2^k lanes per token), fill it, or fill it more than once, and at token
counts around the tokens per wave, against float64."""
import numpy as np
import pytest
import torch

import paper_2508_15881_amd as tp
from paper_2508_15881_amd import pipeline as pl
from paper_2508_15881_amd import workloads as wl
from oracle import tpla_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d_c,d_r,T", [(8, 8, 1), (72, 24, 3), (512, 64, 1), (512, 64, 17), (256, 64, 33), (264, 8, 9), (504, 64, 5), (16, 2048, 7), (520, 136, 16), (1024, 64, 5), (1536, 64, 6)])
def test_write_mla_cache_edges(dtype, d_c, d_r, T):
    print(f"[gpu] write_mla_cache {dtype} d_c={d_c} d_r={d_r} T={T}", flush=True)
    rng = np.random.default_rng(d_c + d_r + T)
    shape = tp.TplaShape(1, 16, d_c, 1, d_r, 8, 8, 16, tp.TPLA_F32 if dtype == "f32" else tp.TPLA_BF16, 1.0)
    c = wl.to_storage(rng.standard_normal((T, d_c)) * np.exp(rng.uniform(-2, 2, size=(T, 1))), dtype)
    k = wl.to_storage(rng.standard_normal((T, d_r)), dtype)
    slots = rng.permutation(64)[:T].astype(np.int32)
    if T > 2:
        slots[T // 2] = -1
    for eps in (1e-6, -1.0):
        pool = torch.zeros((4, 16, d_c + d_r), dtype=pl.torch_dtype(dtype), device="cuda")
        tp.tpla_write_mla_cache(shape, pl.to_device(c, dtype), pl.to_device(k, dtype), torch.from_numpy(slots).cuda(), T, eps, pool)
        torch.cuda.synchronize()
        got = wl.as_f64(pl.from_device_bits(pool), dtype).reshape(64, d_c + d_r)
        c64, k64 = wl.as_f64(c, dtype), wl.as_f64(k, dtype)
        ref = orc.mla_cache_rows(c64, k64, eps) if eps >= 0 else np.concatenate([c64, k64], axis=1)
        keep = slots >= 0
        tol = 2e-6 if dtype == "f32" else 2.0 ** -8          # float: the scale carries a sum of up to 1536 squares and a square root
        assert np.all(np.abs(got[slots[keep]] - ref[keep]) <= tol * np.abs(ref[keep]) + 1e-30)
        assert np.array_equal(got[slots[keep]][:, d_c:], k64[keep])
        rest = np.ones(64, dtype=bool)
        rest[slots[keep]] = False
        assert np.all(got[rest] == 0)

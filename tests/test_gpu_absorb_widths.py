"""Absorb of the query, every kernel of it against the float64 oracle: the matrix-core instances of all key widths with several blocks of 16 sequences per
workgroup and a ragged last one; the few-rows kernel over one and more rounds of 32 weight rows, remainders and the column tail, in both types; the
general kernel, which larger batches take, with a partial last group of 8 sequences.  Factors differ by slice.  Float: sums of up to 1000 products in
another order (1e-5 of the sum of their sizes); bf16: half a step of the output beside it."""
import numpy as np
import pytest
import torch

import paper_2508_15881_amd as tp
from oracle import tpla_oracle as orc
from paper_2508_15881_amd import pipeline as pl
from paper_2508_15881_amd import workloads as wl

pytestmark = pytest.mark.gpu

# dtype, B, H, d_n, d_c, g
CASES = [("bf16", 270, 2, d_n, 128, 4) for d_n in range(32, 257, 32)] + [("bf16", 37, 5, d_n, 256, 2) for d_n in (32, 96, 160, 224, 256)]
CASES += [(dt, 1, 3, d_n, d_c, g) for dt in ("bf16", "f32") for d_n, d_c, g in ((8, 24, 3), (24, 72, 3), (40, 72, 1), (128, 200, 5), (256, 64, 8), (250, 192, 2), (33, 520, 1))
          if dt == "f32" or d_n % 32 or d_c % 128]
CASES += [(dt, 21, 5, d_n, d_c, g) for dt in ("bf16", "f32") for d_n, d_c, g in ((40, 192, 2), (128, 328, 1), (24, 264, 3))] + [("f32", 53, 3, 256, 512, 4), ("f32", 3, 2, 264, 64, 2),
                                                                                                                      ("bf16", 2, 2, 1000, 128, 4)]


@pytest.mark.parametrize("dtype,B,H,d_n,d_c,g", CASES, ids=["%s_b%d_h%d_n%d_c%d_g%d" % c for c in CASES])
def test_absorb_against_the_oracle(dtype, B, H, d_n, d_c, g):
    print(f"[gpu] absorb {dtype} B={B} H={H} d_n={d_n} d_c={d_c} g={g}", flush=True)
    rng = np.random.default_rng(B + d_n + d_c)
    shape = tp.TplaShape(B, H, d_c, g, 16, d_n, 32, 64, tp.TPLA_F32 if dtype == "f32" else tp.TPLA_BF16, 1.0)
    q = wl.to_storage(rng.standard_normal((B, H, d_n)), dtype)
    W = wl.to_storage(rng.standard_normal((H, d_n, d_c)) * 0.05, dtype)
    mu = [0.5 + 0.75 * i for i in range(g)]
    q_lat = torch.full((g, B, H, d_c // g), float("nan"), dtype=pl.torch_dtype(dtype), device="cuda")
    tp.tpla_absorb_query(shape, pl.to_device(q, dtype), pl.to_device(W, dtype), mu, q_lat)
    got = wl.as_f64(pl.from_device_bits(q_lat), dtype)
    q64, W64, m64 = wl.as_f64(q, dtype), wl.as_f64(W, dtype), np.asarray(mu, dtype=np.float32).astype(np.float64)
    want, size = orc.absorb_query(q64, W64, g, m64), orc.absorb_query(np.abs(q64), np.abs(W64), g, m64)
    assert np.all(np.abs(got - want) <= 1e-5 * size + (0.0 if dtype == "f32" else 2.0 ** -8) * np.abs(want))

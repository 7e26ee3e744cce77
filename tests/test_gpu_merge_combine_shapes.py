"""Merge and combine as one kernel, latent widths that are a multiple of 512 (and the combine alone, multiples of 256): every way its units of work are dealt over the waves (sequences
per workgroup, slice widths) and every column width of a workgroup, with page ranges of one, some and many slots.  o_lat and lse against the
stand-alone merge, o against the product in 64 bits of the o_lat that the same call returned: two bf16 terms carry at least 16 bits of a float
(2^-16), the float sums of up to 1024 products add at most as much again."""
import numpy as np
import pytest
import torch

import paper_2508_15881_amd as tp
from paper_2508_15881_amd import pipeline as pl
from paper_2508_15881_amd import workloads as wl

pytestmark = pytest.mark.gpu

# heads, g, d_c, d_v, lengths
CASES = [(H, g, 512, d_v, lens)
         for H, d_v in ((64, 128), (16, 64), (16, 192), (128, 128))
         for g, lens in ((1, [1300]), (2, [64]), (2, [1300, 0]), (2, [9000, 65, 700]), (4, [5000]), (4, [90, 20000]), (8, [3000]), (8, [130, 1, 4097]))]
CASES += [(64, 2, 512, 128, [64 * i + 1 for i in range(n)]) for n in (4, 5, 8, 9, 16, 23)]
CASES += [(64, 4, 512, 128, [40 * i + 7 for i in range(n)]) for n in (6, 10, 16, 17)]
CASES += [(64, 8, 512, 128, [40 * i + 7 for i in range(n)]) for n in (6, 17)] + [(16, 2, 1024, 128, [2000, 100]), (64, 8, 1024, 64, [700])]
CASES += [(H, g, d_c, 128, lens) for d_c in (256, 768) for H, g, lens in ((64, 1, [500] * 9), (16, 2, [1300, 0, 70]), (128, 4, [40 * i + 7 for i in range(17)]))
          if d_c // g % 64 == 0]
# two rounds of workgroups
CASES += [(64, 2, 512, 128, [130 + i for i in range(70)]), (128, 1, 512, 128, [65 + i for i in range(40)])]


@pytest.mark.parametrize("H,g,d_c,d_v,lens", CASES, ids=["h%d_g%d_c%d_v%d_%dx%d" % (*c[:4], len(c[4]), max(c[4])) for c in CASES])
@pytest.mark.parametrize("n_splits", [0, 5])
def test_merge_and_combine_against_the_separate_kernels(H, g, d_c, d_v, lens, n_splits):
    print(f"[gpu] merge-and-combine H={H} g={g} d_c={d_c} d_v={d_v} lens={lens[:4]} B={len(lens)} n_splits={n_splits}", flush=True)
    B, dl = len(lens), d_c // g
    shape = pl.make_shape(wl.scaled(wl.CONFIGS["dsv3_4k"], B=B, H=H, g=g, d_c=d_c, d_v=d_v))
    pages = [(n + 63) // 64 for n in lens]
    width, P = max(pages) + 3, sum(pages)
    gen = torch.Generator(device="cuda").manual_seed(H + d_v + B)
    normal = lambda *s: torch.randn(*s, generator=gen, device="cuda", dtype=torch.bfloat16)
    bt, at = torch.zeros(B, width, dtype=torch.int32), 0
    for b, n in enumerate(pages):
        bt[b, :n] = torch.arange(at, at + n)
        at += n
    bt, lens_d = bt.cuda(), torch.tensor(lens, dtype=torch.int32, device="cuda")
    q_lat, q_pe, W = normal(g, B, H, dl), normal(B, H, 64), normal(H, d_c, d_v)
    pools = [normal(P, 64, dl + 64) for _ in range(g)]
    ws_b = tp.tpla_workspace_bytes_all(shape, width, n_splits)
    ws = torch.full((ws_b,), 0xFF, dtype=torch.uint8, device="cuda")
    new = lambda *s: torch.full(s, float("nan"), device="cuda")
    o, o_lat, lse, ref_lat, ref_lse = new(B, H, d_v), new(g, B, H, dl), new(g, B, H), new(g, B, H, dl), new(g, B, H)
    o16 = torch.full((B, H, d_v), float("nan"), dtype=torch.bfloat16, device="cuda")
    tp.tpla_decode_shards_combine_to(shape, q_lat, q_pe, pools, bt, width, lens_d, n_splits, ws, ws_b, W, o16, tp.TPLA_BF16, o_lat, lse)
    o_lat.fill_(float("nan"))
    tp.tpla_decode_shards_combine(shape, q_lat, q_pe, pools, bt, width, lens_d, n_splits, ws, ws_b, W, o, o_lat, lse)
    tp.tpla_decode_shards(shape, q_lat, q_pe, pools, bt, width, lens_d, n_splits, ws, ws_b, ref_lat, ref_lse)
    torch.testing.assert_close(o_lat, ref_lat, rtol=2e-5, atol=2e-6)        # the same sums in another order
    torch.testing.assert_close(lse, ref_lse, rtol=1e-6, atol=2e-6)
    x, w = o_lat.double().permute(1, 2, 0, 3).reshape(B, H, d_c).cpu(), W.double().cpu()
    exact = torch.einsum("bhk,hkj->bhj", x, w)
    bound = torch.einsum("bhk,hkj->bhj", x.abs(), w.abs()) * 2.0 ** -15 + 1e-30
    assert bool(((o.double().cpu() - exact).abs() <= bound).all())
    assert torch.equal(o16, o.to(torch.bfloat16))
    o2 = torch.full_like(o, float("nan"))
    tp.tpla_combine_shards(shape, o_lat, W, o2)
    assert bool(((o2.double().cpu() - exact).abs() <= bound).all())

"""Prefill at the ends of the projection's blocks of 64 and 512 rows: latents past the last token are not used, nothing is written past the last row of the
workspace, and the outputs hold against float64 (bf16 keys, values and weights of the softmax: 2^-8 each, 1e-2 of the 2-norm)."""
import math

import pytest
import torch

import paper_2508_15881_amd as tp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,d_c", [(3, 128), (2, 512)])
@pytest.mark.parametrize("T", [1, 15, 63, 65, 448, 449, 513, 1090])
def test_prefill_row_edges(H, d_c, T):
    print(f"[gpu] prefill rows T={T} H={H} d_c={d_c}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(T)
    normal = lambda *s: torch.randn(*s, generator=gen, device="cuda", dtype=torch.bfloat16)
    q_nope, q_pe, c, k_pe = normal(T, H, 128), normal(T, H, 64), normal(T + 64, d_c), normal(T, 64)
    c[T:] = float("nan")
    W_UK, W_UV = normal(H, 128, d_c) * 0.05, normal(H, d_c, 128) * 0.05
    scale = 1 / math.sqrt(192)
    shape = tp.TplaShape(1, H, d_c, 1, 64, 128, 128, 64, tp.TPLA_BF16, scale)
    ws_b = tp.tpla_prefill_workspace_bytes(shape, T)
    ws = torch.full((ws_b + 64 * H * 512,), 0x5A, dtype=torch.uint8, device="cuda")
    o = torch.full((T, H, 128), float("nan"), device="cuda")
    cu = torch.tensor([0, T], dtype=torch.int32, device="cuda")
    tp.tpla_prefill_attention(shape, q_nope, q_pe, c, k_pe, W_UK, W_UV, cu, T, T, ws, ws_b, o)
    assert bool((ws[ws_b:] == 0x5A).all())
    x = c[:T].double().cpu()
    for h in range(H):
        k = torch.cat([x @ W_UK[h].double().cpu().t(), k_pe.double().cpu()], 1)
        q = torch.cat([q_nope[:, h], q_pe[:, h]], 1).double().cpu()
        s = (scale * q @ k.t()).masked_fill(torch.ones(T, T, dtype=torch.bool).triu(1), float("-inf"))
        want = torch.softmax(s, 1) @ (x @ W_UV[h].double().cpu())
        assert float((o[:, h].double().cpu() - want).norm() / want.norm()) <= 1e-2

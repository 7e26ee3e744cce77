"""W_O in passes of 32, 64 and 128 rows: batches at the edges of the three, and one past the largest, with k-ranges of one,
two and more chunks (the ring holds two or three ahead), against the oracle."""
import numpy as np
import pytest
import torch

import paper_2508_15881_amd as tp
from gpu_common import rel_err
from oracle import tpla_oracle as orc
from paper_2508_15881_amd import pipeline as pl
from paper_2508_15881_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,d_v,D", [(2, 64, 256), (24, 128, 2048), (16, 128, 7168), (16, 128, 2048), (8, 128, 2048)])   # 1, 3, 8; all compute units 2 and 1 chunks per k-range
@pytest.mark.parametrize("Bn", [16, 17, 32, 33, 64, 65, 112, 113, 128, 129, 192, 193])
def test_rows_at_the_edges_of_a_pass(Bn, H, d_v, D):
    print(f"output projection rows: B={Bn} H={H} d_v={d_v} D={D}", flush=True)
    rng = np.random.default_rng(Bn * 8 + H)
    shape = tp.TplaShape(Bn, H, 64, 2, 16, 8, d_v, 64, tp.TPLA_BF16, 1.0)
    x = rng.standard_normal((Bn, H, d_v)).astype(np.float32)
    W = wl.to_storage(rng.standard_normal((H * d_v, D)) * 0.02, "bf16")
    ws_b = tp.tpla_output_projection_workspace_bytes(shape, D)
    ws = torch.empty(max(ws_b, 16), dtype=torch.uint8, device="cuda")
    out = torch.full((Bn, D), float("nan"), dtype=torch.float32, device="cuda")
    tp.tpla_output_projection(shape, torch.from_numpy(x).cuda(), pl.to_device(W, "bf16"), D, ws, ws_b, out)
    torch.cuda.synchronize()
    # x is carried by two bf16 terms: 2^-16 of each product, and float sums over K <= 3072 of them
    assert rel_err(out.cpu().numpy(), orc.output_projection(x.astype(np.float64), wl.as_f64(W, "bf16"))) <= 1e-5

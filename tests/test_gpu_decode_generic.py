"""The generic decode kernel at the widths where its tiles change: rows that leave 64, 32, 8 or fewer tokens per tile, column
groups that do and do not divide a wave, head counts around four, one and several chunks per sequence; against float64."""
import numpy as np
import pytest
import torch

import paper_2508_15881_amd as tp
from paper_2508_15881_amd import workloads as wl

from gpu_common import TOL, build_shard_problem, oracle_decode_shard, rel_err, run_decode_shard

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("dl,d_r,H,pt", [(8, 8, 1, 64), (32, 16, 4, 64), (40, 24, 5, 16), (144, 8, 3, 64), (256, 64, 2, 64), (512, 64, 4, 48),
                                         (1024, 64, 1, 64), (264, 2104, 2, 64)])
@pytest.mark.parametrize("n_splits", [0, 1, 3])
def test_generic_decode_edges(dtype, dl, d_r, H, pt, n_splits):
    print(f"[gpu] generic decode {dtype} dl={dl} d_r={d_r} H={H} page={pt} n_splits={n_splits}", flush=True)
    w = wl.Workload("edges", B=5, H=H, d_c=dl, g=1, d_r=d_r, d_n=16, d_v=16, dtype=dtype, page_tokens=pt, seed=dl + H, unit_variance_rows=True)
    if dtype == "bf16" and pt == 64 and d_r == 64 and dl in (128, 256, 512):
        w = wl.scaled(w, H=3)                                  # a head count the matrix-core kernel does not take
    prob = build_shard_problem(w, [130, 0, 1, 63, 257])
    o, lse = run_decode_shard(prob, n_splits)
    r_o, r_lse = oracle_decode_shard(prob)
    assert rel_err(o, r_o) <= TOL[dtype]
    assert np.array_equal(np.isneginf(lse), np.isneginf(r_lse))
    live = ~np.isneginf(r_lse)
    assert np.max(np.abs(lse[live] - r_lse[live])) <= TOL[dtype]

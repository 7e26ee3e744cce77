"""Batched prefill: the tiles of 2 to 64 sequences share one grid (an upper bound of T / 128 + B tiles) where that is
fewer workgroups, other batches keep a grid of tiles x sequences.  Lengths at the tile edges, empty sequences at both ends, a batch at and past
64, and token counts at the edges of the projection's blocks of 512 rows, each against the oracle."""
import numpy as np
import pytest

from gpu_common import TOL, rel_err
from oracle import tpla_oracle as orc
from paper_2508_15881_amd import workloads as wl
from test_gpu_parity import _prefill_problem, _run_prefill

pytestmark = pytest.mark.gpu

CASES = {
    "edges": [127, 128, 129, 1, 255, 256, 257],
    "empty first and last": [0, 0, 130, 0, 5, 0],
    "two": [1, 511],
    "64 sequences": [1 + (37 * i) % 19 for i in range(63)] + [140],
    "65 sequences": [1 + (37 * i) % 19 for i in range(64)] + [140],
    "as many as the longest needs": [128, 100, 127],
    "one, 512 rows": [512],
    "one, 513 rows": [513],
}


@pytest.mark.parametrize("H,d_c", [(2, 128), (3, 256)])
@pytest.mark.parametrize("name", list(CASES))
def test_packed_sequences_match_the_oracle(name, H, d_c):
    lens = CASES[name]
    print(f"prefill packing: {name} H={H} d_c={d_c}", flush=True)
    p = _prefill_problem(len(lens) * 7 + H, lens, H, d_c)
    f64 = {k: wl.as_f64(p[k], "bf16") for k in ("q_nope", "q_pe", "c", "k_pe", "W_UK", "W_UV")}
    ref = orc.mla_prefill(f64["q_nope"], f64["q_pe"], f64["W_UK"], f64["W_UV"], f64["c"], f64["k_pe"], p["cu"],
                                 1.0 / np.sqrt(192.0))
    o, _ = _run_prefill(p, H, d_c, len(lens), max(lens))
    assert np.all(np.isfinite(o))                            # every row of every sequence was written
    # the bound of the parity tests: keys, values, queries and probabilities are bf16 (up to 2^-8 relative each)
    assert rel_err(o, ref) <= TOL["bf16"]


@pytest.mark.parametrize("lens", [[300, 1, 640, 129, 0, 513, 384, 385], [40] * 40 + [257] * 3 + [256, 0, 700],
                                  [30 + 7 * (i * 37 % 64) for i in range(64)], [128, 1000]])
def test_sequences_ranked_by_their_tiles(lens):
    """The sequences are laid end to end by falling number of query tiles, ties by index, empty ones last, each with two groups of heads
    of its own (16 heads): every tile of every sequence and head is computed once."""
    H, d_c = 16, 128
    print(f"prefill order: {len(lens)} sequences", flush=True)
    p = _prefill_problem(len(lens), lens, H, d_c)
    f64 = {k: wl.as_f64(p[k], "bf16") for k in ("q_nope", "q_pe", "c", "k_pe", "W_UK", "W_UV")}
    ref = orc.mla_prefill(f64["q_nope"], f64["q_pe"], f64["W_UK"], f64["W_UV"], f64["c"], f64["k_pe"], p["cu"],
                                 1.0 / np.sqrt(192.0))
    o, _ = _run_prefill(p, H, d_c, len(lens), max(lens))
    assert np.all(np.isfinite(o))
    # as above, and for every head by itself: a head left out or taken twice would show in one of them alone
    assert max(rel_err(o[:, h], ref[:, h]) for h in range(H)) <= TOL["bf16"]

"""Merge of the split decode's partial results over the page ranges of the automatic plan: lengths far below what the
block table could hold (fewer pages than workgroups, one page per range), single and odd batches, long sequences of
many partial results beside empty ones, every slice width; against the float64 oracle."""
import numpy as np
import pytest
import torch

import paper_2508_15881_amd as tp
from paper_2508_15881_amd import pipeline as pl
from paper_2508_15881_amd import workloads as wl
from oracle import tpla_oracle as orc

from gpu_common import TOL, build_shard_problem, rel_err

pytestmark = pytest.mark.gpu

CASES = [  # lengths, g, heads, pages of a block-table row (0: as many as the longest sequence needs), d_v
    ([1], 2, 64, 64, 128),
    ([1237], 2, 64, 64, 128),
    ([4100, 0], 4, 16, 512, 128),
    ([20000], 1, 16, 0, 128),
    ([33000], 2, 16, 600, 128),
    ([65, 0, 9000], 2, 32, 200, 128),
    ([64 * 300 + 1] + [70] * 4, 2, 32, 1000, 72),
    ([700, 3, 64, 1500, 129, 0, 2048, 64, 65], 4, 64, 80, 128),
    ([300] * 17, 2, 16, 40, 200),
    ([2500] * 33, 1, 16, 0, 64),
    ([5000], 2, 128, 128, 128),
    # the last workgroup has one to three sequences, the others eight (the lengths of those: several page ranges)
    ([70 + 11 * i for i in range(24)] + [3000], 2, 64, 0, 128),
    ([130] * 32 + [2000], 2, 64, 64, 128),
    ([65, 0] * 16 + [700, 0, 1900], 2, 64, 0, 128),
    ([90] * 40 + [4000], 4, 64, 0, 128),
    ([200] * 26 + [2500], 1, 64, 0, 128),
    ([100 + 64 * i for i in range(9)], 2, 128, 0, 128),
    ([129] * 16 + [64, 1000, 3], 2, 128, 0, 128),
    ([66] * 56 + [1500], 2, 32, 0, 128),
    # four heads per wave with 17, some 30 and more than 64 slots in a pair
    ([130] * 22 + [20011], 2, 64, 0, 128),
    ([300] * 21 + [9000, 5000], 2, 64, 0, 128),
    ([64] * 56 + [17 * 64], 4, 64, 0, 128),
]


@pytest.mark.parametrize("lens,g,H,table,d_v", CASES, ids=["%dx%d_g%d_h%d_t%d_v%d" % (len(c[0]), max(c[0]), *c[1:]) for c in CASES])
@pytest.mark.parametrize("n_splits", [0, 7])
def test_merge_over_short_ranges(lens, g, H, table, d_v, n_splits):
    print(f"[gpu] merge lens={lens[:4]} B={len(lens)} g={g} H={H} table={table} d_v={d_v} n_splits={n_splits}", flush=True)
    w = wl.scaled(wl.CONFIGS["dsv3_4k"], B=len(lens), H=H, g=g, d_v=d_v)
    probs = [build_shard_problem(w, lens, rng_extra=40 + i) for i in range(g)]
    p0 = probs[0]
    shape = pl.make_shape(w)
    width = max(table, p0["max_pages"])
    bt = np.zeros((len(lens), width), dtype=np.int32)
    bt[:, :p0["max_pages"]] = p0["bt"]
    pools, kpe = [], [r[:, w.dl:] for r in p0["rows64"]]
    for i in range(g):                                 # latents of every slice on the pages of the first, its RoPE key on all
        pool = p0["pool"].copy()
        for b, n in enumerate(p0["lens"]):
            for j in range((int(n) + 63) // 64):
                pool[p0["bt"][b, j], :, :w.dl] = probs[i]["pool"][probs[i]["bt"][b, j], :, :w.dl]
        pools.append(pl.to_device(pool, "bf16"))
    q_lat = pl.to_device(np.stack([p["q_lat"] for p in probs]), "bf16")
    q_pe, lens_d, bt_d = pl.to_device(p0["q_pe"], "bf16"), torch.from_numpy(p0["lens"]).cuda(), torch.from_numpy(bt).cuda()
    Wv = wl.to_storage(np.random.default_rng(5).standard_normal((H, w.d_c, d_v)) * 0.05, "bf16")
    Wv_d = pl.to_device(Wv, "bf16")
    ref = [orc.shard_attention(wl.as_f64(probs[i]["q_lat"], "bf16"), wl.as_f64(p0["q_pe"], "bf16"),
                               [r[:, :w.dl] for r in probs[i]["rows64"]], kpe, w.sm_scale) for i in range(g)]
    ref_o = orc.combine_shards(np.stack([r[0] for r in ref]), wl.as_f64(Wv, "bf16"))
    ref_lse = np.stack([r[1] for r in ref])
    ws_b = tp.tpla_workspace_bytes_all(shape, width, n_splits)
    ws = torch.full((ws_b,), 0xFF, dtype=torch.uint8, device="cuda")     # NaN wherever nothing was written
    new = lambda *s: torch.full(s, float("nan"), dtype=torch.float32, device="cuda")
    o, o_lat, lse = new(len(lens), H, d_v), new(g, len(lens), H, w.dl), new(g, len(lens), H)
    o2, o_lat2, lse2 = torch.full_like(o, float("nan")), torch.full_like(o_lat, float("nan")), torch.full_like(lse, float("nan"))
    tp.tpla_decode_shards_combine(shape, q_lat, q_pe, pools, bt_d, width, lens_d, n_splits, ws, ws_b, Wv_d, o, o_lat, lse)
    tp.tpla_decode_shards(shape, q_lat, q_pe, pools, bt_d, width, lens_d, n_splits, ws, ws_b, o_lat2, lse2)
    tp.tpla_combine_shards(shape, o_lat2, Wv_d, o2)
    D = 64                                             # the block output: the same merge and combine in front of W_O
    W_O = torch.ones((H * d_v, D), dtype=torch.bfloat16, device="cuda")
    ws3_b = tp.tpla_attention_block_workspace_bytes(shape, width, n_splits, D)
    ws3 = torch.full((ws3_b,), 0xFF, dtype=torch.uint8, device="cuda")
    o3, o_lat3, lse3, out = new(len(lens), H, d_v), new(g, len(lens), H, w.dl), new(g, len(lens), H), new(len(lens), D)
    tp.tpla_decode_shards_project(shape, q_lat, q_pe, pools, bt_d, width, lens_d, n_splits, ws3, ws3_b, Wv_d, W_O, D, out, tp.TPLA_F32,
                                  o3, o_lat3, lse3)
    torch.cuda.synchronize()
    assert torch.equal(o3, o) and torch.equal(o_lat3, o_lat) and torch.equal(lse3, lse)
    for got_o, got_lat, got_lse in ((o, o_lat, lse), (o2, o_lat2, lse2)):
        assert rel_err(got_lat.cpu().numpy(), np.stack([r[0] for r in ref])) <= TOL["bf16"]
        assert rel_err(got_o.cpu().numpy(), ref_o) <= TOL["bf16"]
        L = got_lse.cpu().numpy()
        assert np.array_equal(np.isneginf(L), np.isneginf(ref_lse))
        live = ~np.isneginf(ref_lse)
        assert np.max(np.abs(L[live] - ref_lse[live]), initial=0.0) <= 1e-2
    # same partial results, merged in the same slot order: only float rounding apart (2^-24 per slot and column)
    assert rel_err(o2.cpu().numpy(), o.cpu().numpy()) <= 1e-5 and rel_err(o_lat2.cpu().numpy(), o_lat.cpu().numpy()) <= 1e-5


@pytest.mark.parametrize("dtype,H,d_c", [("bf16", 64, 512), ("bf16", 3, 512), ("bf16", 2, 144), ("f32", 4, 128)])
@pytest.mark.parametrize("times", [1, 16])
@pytest.mark.parametrize("n_splits", [0, 1, 5, 47])
def test_scores_that_are_not_finite_are_not_an_empty_sequence(dtype, H, d_c, times, n_splits):
    """lse = -inf says that a sequence is empty.  A sequence with a NaN in one of its rows, or whose only score is infinite, has
    lse NaN and o NaN through every merge, and the other sequences do not see it."""
    print(f"[gpu] merge of non-finite scores {dtype} H={H} d_c={d_c} times={times} n_splits={n_splits}", flush=True)
    lens = [1, 3000, 130, 0] * times
    w = wl.Workload("nan", B=len(lens), H=H, d_c=d_c, g=2, d_r=64 if d_c == 512 else 24, d_n=128, d_v=128, dtype=dtype, seed=3, unit_variance_rows=True)
    p = build_shard_problem(w, lens)
    shape = pl.make_shape(w)
    hit = np.array([n in (1, 3000) for n in lens])
    bad = p["pool"].copy()
    for b, n in enumerate(lens):
        if hit[b]:
            row = bad[p["bt"][b, (n - 1) // 64], (n - 1) % 64]
            row[5 if n > 1 else w.dl] = wl.to_storage(np.array([np.nan if n > 1 else -np.inf]), dtype)[0]
    q_lat = pl.to_device(np.stack([p["q_lat"], p["q_lat"]]), dtype)
    q_pe, lens_d, bt_d = pl.to_device(p["q_pe"], dtype), torch.from_numpy(p["lens"]).cuda(), torch.from_numpy(p["bt"]).cuda()
    Wv = pl.to_device(wl.to_storage(np.random.default_rng(5).standard_normal((H, d_c, 128)) * 0.05, dtype), dtype)
    ws_b = tp.tpla_workspace_bytes_all(shape, p["max_pages"], n_splits)
    ws = torch.full((ws_b,), 0xFF, dtype=torch.uint8, device="cuda")

    def both(pool):
        pools = [pl.to_device(pool, dtype)] * 2
        new = lambda *s: torch.zeros(s, dtype=torch.float32, device="cuda")
        o, o_lat, lse = new(w.B, H, 128), new(2, w.B, H, w.dl), new(2, w.B, H)
        o_lat2, lse2 = new(2, w.B, H, w.dl), new(2, w.B, H)
        tp.tpla_decode_shards_combine(shape, q_lat, q_pe, pools, bt_d, p["max_pages"], lens_d, n_splits, ws, ws_b, Wv, o, o_lat, lse)
        tp.tpla_decode_shards(shape, q_lat, q_pe, pools, bt_d, p["max_pages"], lens_d, n_splits, ws, ws_b, o_lat2, lse2)
        torch.cuda.synchronize()
        return [t.cpu().numpy() for t in (o[None], o_lat, lse, o_lat2, lse2)]

    for clean, got in zip(both(p["pool"]), both(bad)):
        assert not np.any(np.isnan(clean))
        assert np.all(np.isnan(got[:, hit]))
        assert np.array_equal(got[:, ~hit], clean[:, ~hit])

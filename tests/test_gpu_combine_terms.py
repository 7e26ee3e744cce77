"""How many bits of the float o_lat reach the product with W_UV.  A weight matrix of single ones copies columns of o_lat to the
output, so what arrives can be compared with what went in: every bit for the widths that take three bf16 terms, 2^-17
for those that take two (a term keeps 8 bits, round to nearest).  Infinities behave as in a float product."""
import numpy as np
import pytest
import torch

import paper_2508_15881_amd as tp
from paper_2508_15881_amd import pipeline as pl
from paper_2508_15881_amd import workloads as wl

from gpu_common import build_shard_problem

pytestmark = pytest.mark.gpu

SHAPES = [  # d_c, g, d_v, H, B, all 24 bits?
    (256, 1, 128, 64, 32, True), (256, 2, 128, 16, 5, True), (128, 1, 128, 3, 1, True), (512, 2, 72, 16, 17, True), (192, 1, 64, 2, 40, True),
    (320, 1, 200, 5, 3, True), (768, 2, 128, 4, 9, True), (1024, 4, 72, 2, 33, True),
    (512, 2, 128, 64, 33, False), (1024, 2, 64, 3, 5, False), (512, 8, 192, 16, 1, False),
]


def _pick(H, d_c, d_v, seed):
    """W of single ones, and the latent column each output column copies."""
    k = np.random.default_rng(seed).integers(0, d_c, size=(H, d_v))
    W = np.zeros((H, d_c, d_v), dtype=np.float32)
    W[np.arange(H)[:, None], k, np.arange(d_v)[None]] = 1.0
    return W, k


def _rows(o_lat):
    """[g, B, H, dl] -> [B, H, d_c]"""
    return np.moveaxis(o_lat, 0, 2).reshape(o_lat.shape[1], o_lat.shape[2], -1)


def _compare(o, o_lat, k, exact):
    ref = np.take_along_axis(_rows(o_lat), np.broadcast_to(k[None], o.shape), axis=2)
    if exact:
        assert np.array_equal(o, ref)
    else:
        assert np.all(np.abs(o - ref) <= 2.0 ** -17 * np.abs(ref))


@pytest.mark.parametrize("d_c,g,d_v,H,B,exact", SHAPES)
def test_bits_of_the_latent_output_in_the_combine(d_c, g, d_v, H, B, exact):
    print(f"[gpu] combine terms d_c={d_c} g={g} d_v={d_v} H={H} B={B}", flush=True)
    rng = np.random.default_rng(d_c + d_v + B)
    shape = tp.TplaShape(B, H, d_c, g, 64, 128, d_v, 64, tp.TPLA_BF16, 0.1)
    o_lat = (rng.standard_normal((g, B, H, d_c // g)) * np.exp(rng.uniform(-6, 6, size=(g, B, H, 1)))).astype(np.float32)
    W, k = _pick(H, d_c, d_v, 7)
    W_d = pl.to_device(wl.to_storage(W, "bf16"), "bf16")

    def combine(x, w):
        o = torch.full((B, H, d_v), float("nan"), dtype=torch.float32, device="cuda")
        tp.tpla_combine_shards(shape, torch.from_numpy(x).cuda(), w, o)
        torch.cuda.synchronize()
        return o.cpu().numpy()

    _compare(combine(o_lat, W_d), o_lat, k, exact)
    # an infinite latent output and positive weights; then positive latent outputs (most of them with low terms of zero) and an infinite weight
    pos = np.abs(W) + 0.5
    x = o_lat.copy()
    x[0, B - 1, 0, 3] = np.inf
    got = combine(x, pl.to_device(wl.to_storage(pos, "bf16"), "bf16"))
    assert np.all(got[B - 1, 0] == np.inf) and np.isfinite(np.delete(got.reshape(B * H, d_v), (B - 1) * H, axis=0)).all()
    pos[H - 1, 5, d_v - 1] = np.inf
    x = 1.0 + (rng.random(o_lat.shape) < 0.3) * rng.random(o_lat.shape)
    got = combine(x.astype(np.float32), pl.to_device(wl.to_storage(pos, "bf16"), "bf16"))
    assert np.all(got[:, H - 1, d_v - 1] == np.inf) and np.isfinite(got[:, :, : d_v - 1]).all()


@pytest.mark.parametrize("d_c,g,d_v,H,exact", [(256, 1, 128, 16, True), (256, 2, 72, 32, True), (512, 2, 72, 64, True), (512, 1, 40, 16, True),
                                               (512, 2, 128, 64, False), (1024, 4, 64, 16, False)])
@pytest.mark.parametrize("B", [1, 11, 25])
def test_bits_of_the_latent_output_in_the_fused_combine(d_c, g, d_v, H, exact, B):
    print(f"[gpu] fused combine terms d_c={d_c} g={g} d_v={d_v} H={H} B={B}", flush=True)
    w = wl.Workload("terms", B=B, H=H, d_c=d_c, g=g, d_r=64, d_n=128, d_v=d_v, seed=d_c + B)
    p = build_shard_problem(w, [70 + 37 * i for i in range(B)])
    shape = pl.make_shape(w)
    W, k = _pick(H, d_c, d_v, 9)
    new = lambda *s: torch.full(s, float("nan"), dtype=torch.float32, device="cuda")
    o, o_lat, lse = new(B, H, d_v), new(g, B, H, w.dl), new(g, B, H)
    ws_b = tp.tpla_workspace_bytes_all(shape, p["max_pages"], 0)
    ws = torch.full((ws_b,), 0xFF, dtype=torch.uint8, device="cuda")
    q_lat = pl.to_device(np.stack([np.roll(p["q_lat"], i, axis=1) for i in range(g)]), "bf16")
    tp.tpla_decode_shards_combine(shape, q_lat, pl.to_device(p["q_pe"], "bf16"), [pl.to_device(p["pool"], "bf16")] * g,
                                  torch.from_numpy(p["bt"]).cuda(), p["max_pages"], torch.from_numpy(p["lens"]).cuda(), 0, ws, ws_b,
                                  pl.to_device(wl.to_storage(W, "bf16"), "bf16"), o, o_lat, lse)
    torch.cuda.synchronize()
    _compare(o.cpu().numpy(), o_lat.cpu().numpy(), k, exact)

"""Second moments over ragged pages: last tiles, empty pages, page sizes on both sides of the tile height, more and fewer
pages than splits, more than 64 pages in a split, against float64: rounding on normal latents, and every row exactly
once on small whole numbers."""
import numpy as np
import pytest
import torch

import paper_2508_15881_amd as tp
from paper_2508_15881_amd import pipeline as pl
from paper_2508_15881_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_c,pt,P", [(128, 64, 1), (256, 64, 700), (512, 64, 130), (512, 16, 37), (384, 48, 61), (512, 100, 23), (128, 32, 600), (1024, 4, 1300),
                                      (512, 2, 9000)])
def test_moments_of_ragged_pages(d_c, pt, P):
    print(f"[gpu] latent moments d_c={d_c} page_tokens={pt} pages={P}", flush=True)
    rng = np.random.default_rng(d_c + pt + P)
    G, s, rows = _moments(rng, rng.standard_normal((P + 2, pt, d_c + 64)) + 0.25, d_c, pt, P)
    # products of bf16 are exact in float; float sums inside a split of at most 16384 rows (2^-24 per addition), doubles after it
    n = min(len(rows), 16384)
    assert np.all(np.abs(G - rows.T @ rows) <= n * 2.0 ** -24 * (np.abs(rows).T @ np.abs(rows)) + 1e-12)
    assert np.all(np.abs(s - rows.sum(0)) <= n * 2.0 ** -24 * np.abs(rows).sum(0) + 1e-12)
    # whole numbers of 1 to 4: 16 x 16384 rows stay below 2^24, so every sum is exact, and a row lost or taken twice shows
    G, s, rows = _moments(rng, rng.integers(1, 5, size=(P + 2, pt, d_c + 64)).astype(np.float64), d_c, pt, P)
    assert np.array_equal(G, rows.T @ rows) and np.array_equal(s, rows.sum(0))


def _moments(rng, values, d_c, pt, P):
    """(gram, sum, the rows that count) of the library over shuffled, partly filled pages of `values`."""
    shape = tp.TplaShape(1, 16, d_c, 1, 64, 8, 8, pt, tp.TPLA_BF16, 1.0)
    pool = wl.to_storage(values, "bf16")
    ids = rng.permutation(P + 2)[:P].astype(np.int32)
    fill = rng.integers(0, pt + 1, size=P).astype(np.int32)
    fill[: P // 3] = pt
    fill[-1] = 0 if P > 1 else 5
    bits = pool.copy()
    for p, f in zip(ids, fill):
        bits[p, f:] = 0x7FC0                                 # what lies past the fill is never read
    rows = np.concatenate([wl.as_f64(pool[p, :f, :d_c], "bf16") for p, f in zip(ids, fill)])
    ws_b = tp.tpla_latent_moments_workspace_bytes(shape, P)
    ws = torch.full((ws_b,), 0xFF, dtype=torch.uint8, device="cuda")
    s = torch.full((d_c,), float("nan"), dtype=torch.float64, device="cuda")
    G = torch.full((d_c, d_c), float("nan"), dtype=torch.float64, device="cuda")
    tp.tpla_latent_moments(shape, pl.to_device(bits, "bf16"), torch.from_numpy(ids).cuda(), torch.from_numpy(fill).cuda(), P, ws, ws_b, s, G)
    torch.cuda.synchronize()
    assert torch.equal(G, G.t())
    return G.cpu().numpy(), s.cpu().numpy(), rows

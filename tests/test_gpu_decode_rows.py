"""Narrow float rows in short tables (automatic splits) against the general kernel, which explicit splits still take: block and page edges, every
row width, one to eight slices, empty sequences, the combine inside and outside the kernel.  Float sums in another order: 1e-5 of the largest
value of a row, lse 1e-5."""
import pytest
import torch

import paper_2508_15881_amd as tp

pytestmark = pytest.mark.gpu

# B, H, d_c, g, d_r, d_v, page_tokens, table pages, lengths
CASES = [
    (1, 4, 64, 2, 16, 32, 64, 2, [128]),
    (5, 2, 64, 1, 16, 32, 64, 8, [0, 1, 15, 16, 17]),
    (4, 3, 64, 4, 64, 64, 16, 256, [4096, 63, 65, 2000]),
    (2, 1, 128, 8, 32, 16, 128, 16, [2048, 129]),
    (3, 5, 32, 1, 32, 24, 64, 64, [4096, 1000, 255]),        # d_v without the combine in the kernel
    (2, 2, 256, 4, 16, 128, 32, 20, [640, 33]),
    (2, 4, 64, 2, 16, 256, 64, 64, [4095, 64]),
    (64, 4, 32, 2, 16, 32, 64, 5, [(37 * i) % 320 + 1 for i in range(64)]),
    # all 64 blocks of a wave (taken where 256 pairs keep the device busy)
    (16, 16, 64, 4, 16, 32, 64, 64, [4096, 0, 4095, 4081] + [1, 16, 63, 64, 65, 300] * 2),
    (32, 8, 128, 8, 32, 16, 128, 16, [2048, 1921, 0, 2047] + [(29 * i) % 400 + 1 for i in range(28)]),
    (32, 8, 64, 4, 64, 64, 16, 256, [4096, 63, 65, 2000] + [(31 * i) % 500 for i in range(28)]),
]


@pytest.mark.parametrize("B,H,d_c,g,d_r,d_v,pt,width,lens", CASES, ids=["b%d_h%d_c%d_g%d_r%d_v%d_p%d_t%d" % c[:8] for c in CASES])
def test_rows_against_the_general_kernel(B, H, d_c, g, d_r, d_v, pt, width, lens):
    print(f"[gpu] rows B={B} H={H} d_c={d_c} g={g} d_r={d_r} d_v={d_v} pt={pt} width={width}", flush=True)
    dl, d_n = d_c // g, 24
    shape = tp.TplaShape(B, H, d_c, g, d_r, d_n, d_v, pt, tp.TPLA_F32, 0.2)
    gen = torch.Generator(device="cuda").manual_seed(B * H + d_c)
    normal = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    pages = [(n + pt - 1) // pt for n in lens]
    P = sum(pages) + 2
    ids = torch.randperm(P, generator=torch.Generator().manual_seed(3)).to(torch.int32)
    bt, at = torch.full((B, width), 2 ** 30, dtype=torch.int32), 0          # entries past a sequence are nobody's
    for b, n in enumerate(pages):
        bt[b, :n] = ids[at:at + n]
        at += n
    pools = [normal(P, pt, dl + d_r) for _ in range(g)]
    for p in pools:
        p[ids[at:].long().cuda()] = float("nan")
        for b, n in enumerate(lens):                                        # slots past the end of a sequence are never read
            if n % pt:
                p[int(bt[b, pages[b] - 1]), n % pt:] = float("nan")
    bt, lens_d = bt.cuda(), torch.tensor(lens, dtype=torch.int32, device="cuda")
    q_nope, W_UK, q_pe, W = normal(B, H, d_n), normal(H, d_n, d_c) * 0.2, normal(B, H, d_r), normal(H, d_c, d_v)
    mu = [1.0 + 0.5 * i for i in range(g)]
    q_lat = torch.full((g, B, H, dl), float("nan"), device="cuda")
    tp.tpla_absorb_query(shape, q_nope, W_UK, mu, q_lat)
    exact_q = torch.einsum("bhn,hnc->bhc", q_nope.double().cpu(), W_UK.double().cpu()).reshape(B, H, g, dl).permute(2, 0, 1, 3)
    exact_q = exact_q * torch.tensor(mu, dtype=torch.float64)[:, None, None, None]
    torch.testing.assert_close(q_lat.double().cpu(), exact_q, rtol=1e-5, atol=1e-5)
    got = {}
    for n_splits in (0, 1):
        ws_b = tp.tpla_workspace_bytes_all(shape, width, n_splits)
        ws = torch.full((max(ws_b, 16),), 0xFF, dtype=torch.uint8, device="cuda")
        new = lambda *s: torch.full(s, float("nan"), device="cuda")
        o, o_lat, lse, o_lat2, lse2 = new(B, H, d_v), new(g, B, H, dl), new(g, B, H), new(g, B, H, dl), new(g, B, H)
        tp.tpla_decode_shards_combine(shape, q_lat, q_pe, pools, bt, width, lens_d, n_splits, ws, ws_b, W, o, o_lat, lse)
        tp.tpla_decode_shards(shape, q_lat, q_pe, pools, bt, width, lens_d, n_splits, ws, ws_b, o_lat2, lse2)
        assert torch.equal(o_lat, o_lat2) and torch.equal(lse, lse2)
        got[n_splits] = (o, o_lat, lse)
    for a, b in zip(got[0], got[1]):
        inf = torch.isinf(b)
        assert torch.equal(torch.isinf(a), inf)
        assert float((a - b).masked_fill(inf, 0.0).abs().max()) <= 1e-5 * max(1.0, float(b.masked_fill(inf, 0.0).abs().max()))


@pytest.mark.parametrize("g,d_r", [(1, 16), (2, 16), (2, 32), (4, 16), (4, 64)])
def test_rows_with_scores_that_are_not_finite(g, d_r):
    """Against the softmax in 64 bits: tokens whose score is -inf weigh nothing, whichever blocks, waves and parts of a block they fill; a sequence
    of such tokens alone is NaN and not empty; a NaN row or a score of +inf makes its sequence NaN and no other; rows past the end, infinite and
    NaN here, count for nothing."""
    print(f"[gpu] rows that are not finite g={g} d_r={d_r}", flush=True)
    H, d_c, d_v, pt, width, L = 3, 64, 32, 64, 12, 700
    dl, inf, nan = d_c // g, float("inf"), float("nan")
    # sequence: [tokens, value of the first position column]
    edits = [[], [(range(0, 16), -inf)], [(range(0, L, 2), -inf)], [(range(1, L), -inf)], [(range(0, L - 1), -inf)], [(range(64, 400), -inf)],
             [(range(i, L, 256), -inf) for i in range(64)], [(range(0, L), -inf)], [(range(333, 334), inf)], [(range(699, 700), nan)], [(range(0, 1), nan)],
             [(range(0, L), -inf), (range(5, 6), inf)]]
    bad = [7, 8, 9, 10, 11]
    B = len(edits) + 1                                                      # the last one is empty
    shape = tp.TplaShape(B, H, d_c, g, d_r, 24, d_v, pt, tp.TPLA_F32, 0.2)
    gen = torch.Generator(device="cuda").manual_seed(g + d_r)
    normal = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    n_pages = (L + pt - 1) // pt
    pools = [normal(B * n_pages, pt, dl + d_r) for _ in range(g)]
    for b, edit in enumerate(edits):
        for p in pools:
            rows = p[b * n_pages:(b + 1) * n_pages].view(-1, dl + d_r)
            for tokens, x in edit:
                rows[list(tokens), dl] = x
            rows[L:] = nan
            rows[L + 1::2] = -inf
            rows[L + 2::4] = inf
    bt = torch.arange(B * n_pages, dtype=torch.int32, device="cuda").view(B, n_pages)
    bt = torch.nn.functional.pad(bt, (0, width - n_pages), value=2 ** 30).contiguous()
    lens_d = torch.tensor([L] * (B - 1) + [0], dtype=torch.int32, device="cuda")
    q_lat, q_pe, W = normal(g, B, H, dl), normal(B, H, d_r), normal(H, d_c, d_v)
    q_pe[:, :, 0] = 1.0
    ws_b = tp.tpla_workspace_bytes_all(shape, width, 0)
    ws = torch.full((max(ws_b, 16),), 0xFF, dtype=torch.uint8, device="cuda")
    new = lambda *s: torch.full(s, 7.0, device="cuda")
    o, o_lat, lse = new(B, H, d_v), new(g, B, H, dl), new(g, B, H)
    tp.tpla_decode_shards_combine(shape, q_lat, q_pe, pools, bt, width, lens_d, 0, ws, ws_b, W, o, o_lat, lse)
    rows = torch.stack([p.view(B, n_pages * pt, dl + d_r)[:, :L] for p in pools]).double().cpu()
    q = torch.cat([q_lat, q_pe.expand(g, B, H, d_r)], dim=3).double().cpu()
    score = torch.matmul(q, rows.transpose(2, 3).contiguous()) * 0.2        # (nan, +inf and rows of -inf alone stay NaN through the softmax)
    ref_lat, ref_lse = torch.matmul(torch.softmax(score, 3), rows[..., :dl].contiguous()), torch.logsumexp(score, 3)
    ref_lse[:, bad] = nan
    ref_lat[:, -1], ref_lse[:, -1] = 0.0, -inf
    ref_o = torch.matmul(ref_lat.permute(1, 2, 0, 3).reshape(B, H, 1, d_c), W.double().cpu()).squeeze(2)
    for got, ref in ((o_lat, ref_lat), (lse, ref_lse), (o, ref_o)):
        dim = 0 if got is o else 1
        want_nan = torch.zeros(B, dtype=torch.bool)
        want_nan[bad] = True
        got = got.double().cpu().movedim(dim, 0)
        ref = ref.movedim(dim, 0)
        assert bool(torch.isnan(got[want_nan]).all()) and bool(torch.isnan(ref[want_nan]).all())
        torch.testing.assert_close(got[~want_nan], ref[~want_nan], rtol=1e-5, atol=1e-5)

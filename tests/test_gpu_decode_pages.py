"""The split kernel of 256-wide slices (a page per step, 32 heads per wave, weights swapped between waves) at the sizes where it can
go wrong, against the float64 oracle: first and last tokens of every 16-token quarter of a page, items of one page, more pairs than
a wave scans at once, scores that move the shared reference on many pages and between the items of a workgroup, pages without a finite
score, large latents, ranges long enough to keep their pages in L2, more static chunks than compute units; and the order of its pages."""
import numpy as np
import pytest
import torch

import paper_2508_15881_amd as tp
from gpu_common import TOL, build_shard_problem, oracle_decode_shard, rel_err, run_decode_shard
from paper_2508_15881_amd import workloads as wl

pytestmark = pytest.mark.gpu
DSV3 = wl.CONFIGS["dsv3_32k"]


def score_error(prob):
    """What a score [B, H] may err by: float sums of its products, (d_c/g + d_r) roundings of up to 2^-24 of the sum of their sizes."""
    w = prob["w"]
    q = np.abs(np.concatenate([wl.as_f64(prob["q_lat"], "bf16"), wl.as_f64(prob["q_pe"], "bf16")], axis=2))
    return np.stack([(q[b] @ np.abs(r).T).max(axis=1) if len(r) else np.zeros(w.H) for b, r in enumerate(prob["rows64"])]) \
        * w.sm_scale * (w.dl + w.d_r) * 2.0 ** -24


def check(prob, n_splits):
    o, lse = run_decode_shard(prob, n_splits)
    ro, rl = oracle_decode_shard(prob)
    nz = prob["lens"] > 0
    assert rel_err(o, ro) <= TOL["bf16"]
    # Weights are rounded to bf16 (half a step is 2^-9 of them at most), everything else is float: an output errs by at most
    # 2^-9 of the weighted mean of |v|, so of the largest |v| of its sequence, and by what the scores err (a weight and the sum of all).
    v = np.array([np.abs(r[:, :prob["w"].dl]).max() if len(r) else 0.0 for r in prob["rows64"]])
    d = score_error(prob)
    assert np.all(np.abs(o - ro) <= ((2.0 ** -9 + 1e-4 + 2 * d) * v[:, None])[:, :, None])
    assert np.all(np.abs(lse[nz] - rl[nz]) <= d[nz] + 2.0 ** -20 * (1 + np.abs(rl[nz])))
    assert np.all(o[~nz] == 0) and np.all(np.isneginf(lse[~nz]))
    o2, lse2 = run_decode_shard(prob, n_splits)
    assert np.array_equal(o, o2) and np.array_equal(lse, lse2)


@pytest.mark.parametrize("H", [16, 32, 64, 128])
@pytest.mark.parametrize("n_splits", [0, 2])
def test_edges_of_pages_and_quarters(H, n_splits):
    check(build_shard_problem(wl.scaled(DSV3, H=H), [1, 15, 16, 17, 0, 33, 48, 49, 63, 64, 65, 81, 127, 128, 129, 4097]), n_splits)


@pytest.mark.parametrize("H", [16, 64])
def test_more_pairs_than_lanes_and_several_items_per_workgroup(H):
    lens = np.random.default_rng(5).integers(0, 300, size=520)
    lens[7], lens[300] = 5000, 0
    check(build_shard_problem(wl.scaled(DSV3, H=H), lens), 0)


def peaky(prob):
    """Queries 24 times larger: scores spread over several hundred log2 units, so that later pages exceed the reference of the
    earlier ones by far more than it may be exceeded by, in most heads."""
    for k in ("q_lat", "q_pe"):
        prob[k] = wl.to_storage(wl.as_f64(prob[k], "bf16") * 24.0, "bf16")
    return prob


@pytest.mark.parametrize("H", [16, 32, 64, 128])
def test_reference_moves_on_later_pages(H):
    """Chunks of up to 15 pages, one to a workgroup."""
    check(peaky(build_shard_problem(wl.scaled(DSV3, H=H), [900, 130, 64])), 1)


def moves_of_the_reference(prob, workgroups):
    """(range, items of the range, item, pages of the item, pages on which the reference moves, whether the last of them is a partial one)
    for every item of the automatic plan with at least one such page: equal ranges, an item's pages from a fraction of
    it on (PageOrder), the reference the highest score of the first, moved when one exceeds it by 8 log2 units."""
    w, out, items = prob["w"], [], {}
    q = np.concatenate([wl.as_f64(prob["q_lat"], "bf16"), wl.as_f64(prob["q_pe"], "bf16")], axis=2)
    pages = (prob["lens"].astype(np.int64) + 63) // 64
    total, e = int(pages.sum()), 0
    for b, n in enumerate(pages):
        for k in range(workgroups):
            p0, p1 = max(k * total // workgroups, e) - e, min((k + 1) * total // workgroups, e + int(n)) - e
            if p0 < p1:
                items.setdefault(k, []).append((b, p0, p1))
        e += int(n)
    for k, work in items.items():
        for i, (b, p0, p1) in enumerate(work):
            s = (q[b] @ prob["rows64"][b].T) * w.sm_scale / np.log(2.0)
            first = p0 + (((k * 12337) & 65535) * (p1 - p0) >> 16)
            order = list(range(first, p1)) + list(range(p0, first))
            top = np.stack([s[:, 64 * p:64 * p + 64].max(axis=1) for p in order])
            ref, moved = top[0], []
            for t in range(1, len(order)):
                if np.any(top[t] > ref + 8.01):          # (a hair more: not within rounding)
                    moved.append(order[t])
                    ref = np.maximum(ref, top[t])
            if moved:
                out.append((k, len(work), i, p1 - p0, moved, (moved[-1] + 1) * 64 > prob["lens"][b]))
    return out


@pytest.mark.parametrize("H", [16, 32, 64, 128])
def test_reference_moves_between_the_items_of_a_workgroup(H):
    """The two extra barriers of a moved reference in ranges of several sequences: before, between and after the queries and the
    pending sums of other items, on whole and on partial pages, several times in an item."""
    lens = np.random.default_rng(5).integers(0, 300, size=520)
    lens[7], lens[300] = 5000, 0
    prob = peaky(build_shard_problem(wl.scaled(DSV3, H=H), lens))
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    moves = moves_of_the_reference(prob, cus if H <= 64 else cus // 2)
    several = [m for m in moves if m[1] > 1]
    assert sum(m[2] == 0 for m in several) >= 10 and sum(0 < m[2] < m[1] - 1 for m in several) >= 5 and sum(m[2] == m[1] - 1 for m in several) >= 10
    assert sum(m[5] for m in several) >= 10 and sum(not m[5] for m in several) >= 10 and sum(len(m[4]) > 1 for m in several) >= 5
    check(prob, 0)


def set_rows(prob, edit):
    """Replaces the cache rows of every sequence b by edit(b, rows)."""
    pt = prob["w"].page_tokens
    for b, rows in enumerate(prob["rows64"]):
        stored = wl.to_storage(edit(b, rows.copy()), "bf16")
        wl.place_rows(prob["pool"], prob["bt"][b, :(len(rows) + pt - 1) // pt], stored)
        prob["rows64"][b] = wl.as_f64(stored, "bf16")


@pytest.mark.parametrize("H", [16, 64])
def test_log_sum_exp_of_one_token_is_its_score(H):
    """One product per score, so that it is exact, and |score| < 1: log-sum-exp errs by four roundings of it (the scale, its
    product, the conversion to base e and back: 4 x 2^-24) and by one of a weight near 1 (2^-23), 3e-7 together."""
    prob = build_shard_problem(wl.scaled(DSV3, H=H), [1] * 16)
    dl = prob["w"].dl
    prob["q_lat"] = wl.to_storage(np.zeros_like(wl.as_f64(prob["q_lat"], "bf16")), "bf16")
    q_pe = np.zeros((16, H, 64))
    q_pe[:, :, 0] = np.linspace(-13.0, 13.0, 16 * H).reshape(16, H)
    prob["q_pe"] = wl.to_storage(q_pe, "bf16")
    one = lambda b, rows: np.concatenate([rows[:, :dl], np.ones_like(rows[:, dl:])], axis=1)
    set_rows(prob, one)
    _, lse = run_decode_shard(prob)
    _, ref = oracle_decode_shard(prob)
    assert np.max(np.abs(ref)) < 1 and np.max(np.abs(lse - ref)) <= 2.0 ** -21


@pytest.mark.parametrize("H", [16, 64, 128])
@pytest.mark.parametrize("n_splits", [0, 1])
def test_large_latents_under_scores_far_apart(H, n_splits):
    """Latents of 2^112 and a page whose scores lie 47 log2 units above (even heads) or below the others': sums of the weighted latents
    are finite as long as a weight may not exceed the reference's by many powers of two."""
    prob = build_shard_problem(wl.scaled(DSV3, H=H), [192, 192, 192])
    w = prob["w"]
    prob["q_lat"] = wl.to_storage(np.zeros_like(wl.as_f64(prob["q_lat"], "bf16")), "bf16")
    q_pe = np.zeros((3, H, 64))
    q_pe[:, :, 0] = np.where(np.arange(H) % 2 == 0, 8.0, -8.0)
    prob["q_pe"] = wl.to_storage(q_pe, "bf16")

    def edit(b, rows):
        rows[:, :w.dl] = np.abs(rows[:, :w.dl]) * 2.0 ** 112
        rows[:, w.dl:] = 0
        rows[64 * b:64 * b + 64, w.dl] = 47 * np.log(2.0) / 8.0 / w.sm_scale
        return rows

    set_rows(prob, edit)
    o, lse = run_decode_shard(prob, n_splits)
    ro, rl = oracle_decode_shard(prob)
    assert np.all(np.isfinite(o)) and rel_err(o, ro) <= TOL["bf16"] and np.max(np.abs(lse - rl)) <= 1e-4


@pytest.mark.parametrize("dl,H,times", [(256, 16, 1), (256, 32, 1), (256, 64, 1), (256, 128, 1), (256, 16, 30), (256, 32, 30), (256, 64, 30), (256, 64, 60), (256, 128, 20),
                                        (128, 64, 1), (512, 16, 1), (512, 64, 1), (512, 128, 40)])
@pytest.mark.parametrize("n_splits", [1, 2])
def test_pages_without_a_finite_score(dl, H, times, n_splits):
    """Pages whose scores are all -inf (a masked RoPE component) weigh nothing, wherever they lie in a range; a range of such
    pages alone is NaN, like its softmax.  times > 1: more chunks than compute units, on every kernel that takes them."""
    masked = [(0,), (1,), (2,), (3,), (4,), (0, 1), (2, 4), (1, 2), ()] * times + [(0, 1, 2, 3, 4)]
    prob = build_shard_problem(wl.scaled(DSV3, H=H, g=512 // dl), [300] * len(masked))
    w = prob["w"]
    q_pe = wl.as_f64(prob["q_pe"], "bf16")
    q_pe[:, :, 0] = 1.0
    prob["q_pe"] = wl.to_storage(q_pe, "bf16")

    def edit(b, rows):
        for p in masked[b]:
            rows[64 * p:64 * p + 64, w.dl] = -np.inf
        return rows

    set_rows(prob, edit)
    o, lse = run_decode_shard(prob, n_splits)
    for k in ("rows64", "q_lat", "q_pe"):
        prob[k] = prob[k][:-1]
    prob["w"] = wl.scaled(w, B=len(masked) - 1)
    ro, rl = oracle_decode_shard(prob)
    # with two ranges (pages 0-2 and 3-4) none of the sequences before the last has a range of masked pages alone
    assert rel_err(o[:-1], ro) <= TOL["bf16"] and np.max(np.abs(lse[:-1] - rl)) <= 1e-2
    assert np.all(np.isnan(o[-1])) and np.all(np.isnan(lse[-1]))


@pytest.mark.parametrize("B,L", [(32, 32768), (8, 131072), (32, 32832)])
def test_pools_in_sequence_order_are_read_as_fast_as_scattered_ones(B, L):
    """Ranges of equal length over pages in sequence order: workgroups that begin at unlucky distances share memory channels (12 to
    20 % slower than over scattered pages).  Both on the same card in turn; the medians are within 5 % where the order is good."""
    print(f"page order: {B} x {L}", flush=True)
    shape = tp.TplaShape(B, 64, 256, 1, 64, 128, 128, 64, tp.TPLA_BF16, 192.0 ** -0.5)
    W = (L + 63) // 64
    gen = torch.Generator(device="cuda").manual_seed(B)
    draw = lambda *s: torch.randn(*s, generator=gen, device="cuda", dtype=torch.bfloat16)
    pool, q_lat, q_pe = draw(B * W, 64, 320), draw(B, 64, 256) * 0.35, draw(B, 64, 64)
    lens = torch.full((B,), L, dtype=torch.int32, device="cuda")
    ids = torch.arange(B * W, dtype=torch.int32).reshape(B, W)
    scattered = torch.randperm(B * W, generator=torch.Generator().manual_seed(B)).to(torch.int32).reshape(B, W)
    tables = [ids.cuda(), scattered.cuda()]
    n = tp.tpla_workspace_bytes(shape, W, 0)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    o, lse = torch.empty(B, 64, 256, device="cuda"), torch.empty(B, 64, device="cuda")
    times = []
    for rounds in (100, 60):             # the first settles the clocks
        tp.tpla_profile_enable(2 * rounds)
        for _ in range(rounds):
            for bt in tables:
                tp.tpla_decode_shard(shape, q_lat, q_pe, pool, bt, W, lens, 0, ws, n, o, lse)
        torch.cuda.synchronize()
        times = tp.tpla_profile_collect(2 * rounds)
        tp.tpla_profile_enable(0)
    in_order, over_all = np.median(times[0::2]), np.median(times[1::2])
    print(f"in order {in_order * 1e3:.1f} us, scattered {over_all * 1e3:.1f} us", flush=True)
    assert in_order <= 1.1 * over_all


def test_128_heads_long_ranges():
    """Ranges of 128 pages and more of two rows of workgroups take their own copy of the kernel: chunks of a whole sequence against the
    oracle, balanced ranges (64 sequences over one set of pages) against chunks too short for it, which differ in the order of sums."""
    check(build_shard_problem(wl.scaled(DSV3, H=128), [8192, 8191, 130, 8129, 9000]), 1)
    B, L, W = 64, 16384, 256
    shape = tp.TplaShape(B, 128, 256, 1, 64, 128, 128, 64, tp.TPLA_BF16, 192.0 ** -0.5)
    gen = torch.Generator(device="cuda").manual_seed(3)
    draw = lambda *s: torch.randn(*s, generator=gen, device="cuda", dtype=torch.bfloat16)
    pool, q_lat, q_pe = draw(W, 64, 320), draw(B, 128, 256) * 0.35, draw(B, 128, 64)
    bt = torch.arange(W, dtype=torch.int32, device="cuda").repeat(B, 1).contiguous()
    lens = torch.full((B,), L, dtype=torch.int32, device="cuda")
    got = []
    for n_splits in (0, 4):
        n = tp.tpla_workspace_bytes(shape, W, n_splits)
        ws = torch.empty(n, dtype=torch.uint8, device="cuda")
        o, lse = torch.empty(B, 128, 256, device="cuda"), torch.empty(B, 128, device="cuda")
        tp.tpla_decode_shard(shape, q_lat, q_pe, pool, bt, W, lens, n_splits, ws, n, o, lse)
        torch.cuda.synchronize()
        got.append((o.cpu().numpy(), lse.cpu().numpy()))
    # both round their weights to bf16, relative to different references
    assert rel_err(got[0][0], got[1][0]) <= TOL["bf16"] and np.max(np.abs(got[0][1] - got[1][1])) <= 1e-4


@pytest.mark.parametrize("dl,H", [(256, 16), (256, 32), (256, 64), (256, 128), (512, 128)])
@pytest.mark.parametrize("n_splits", [1, 3, 11])
def test_more_chunks_than_compute_units(dl, H, n_splits):
    """Static launches of one to four and of more chunks per compute unit have kernels or grids of their own: against the oracle, with
    empty sequences (the first and the last too), fewer pages than chunks, chunks of one page and a long sequence among them."""
    lens = np.random.default_rng(H + n_splits).integers(0, 400, size=260 if n_splits < 11 else 140)
    lens[3], lens[0], lens[50:70], lens[-1] = 1500, 0, 0, 0
    check(build_shard_problem(wl.scaled(DSV3, H=H, g=512 // dl), lens), n_splits)


@pytest.mark.parametrize("H", [16, 64, 128])
@pytest.mark.parametrize("lens", [[0] * 1100, [0] * 500 + [130] + [0] * 598 + [1], [3] * 1030 + [700]])
def test_dealt_chunks_that_hardly_exist(H, lens):
    """Enough chunks by the sizes for dealing, of which none, two or one of each sequence exist."""
    prob = build_shard_problem(wl.scaled(DSV3, H=H), lens)
    if sum(lens) == 0:
        o, lse = run_decode_shard(prob, 1)
        assert np.all(o == 0) and np.all(np.isneginf(lse))
    else:
        for n_splits in (1, 2):
            check(prob, n_splits)

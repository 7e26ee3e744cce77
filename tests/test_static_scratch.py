"""Batches whose partial results fit the library's fixed scratch with one page range per 8 pages (not below one per
compute unit) fit it with the plan that is used, whatever more ranges that plan would like."""
import pytest

import paper_2508_15881_amd as tp

LIMIT = 64 << 20
CUS = 256


@pytest.mark.parametrize("H,dl", [(16, 128), (32, 128), (64, 128), (16, 256), (32, 256), (64, 256), (128, 256)])
@pytest.mark.parametrize("g", [1, 2, 4])
def test_plan_stays_inside_the_fixed_scratch(H, dl, g):
    for rows in range(64, 6000, 97):
        B = max(1, rows // g)
        for pages in (1, 2, 3, 5, 8, 16, 64):
            most = g * B * pages
            n_wg = min(max(most // 8, CUS), most)
            shape = tp.TplaShape(B, H, dl * g, g, 64, 128, 128, 64, tp.TPLA_BF16, 0.07)
            if n_wg <= 2 * CUS and (n_wg + g * B) * H * (dl + 2) * 4 + 12 * g * B + 24 <= LIMIT:
                assert tp.tpla_workspace_bytes_all(shape, pages, 0) <= LIMIT, (B, g, H, dl, pages)

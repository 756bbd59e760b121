"""Kernels at the sizes where their splits of the work can go wrong (edges of
tiles, remainders, the smallest and largest of a variant's range), against the
oracle or fp64 torch."""
import numpy as np
import pytest
import torch

import oracle as O
from tests._gpu import bf16_dev, f32_np, mask_np, rel_close

pytestmark = pytest.mark.gpu

zf = pytest.importorskip("paper_2505_12242_amd")


def gbits(n, m, seed, spread=1.5):
    """bf16 bit patterns of independent normals times a lognormal column scale."""
    rng = np.random.default_rng(seed)
    g = rng.standard_normal((n, m)) * np.exp(spread * rng.standard_normal(m))
    return O.bf16_round(g.astype(np.float32))


# Row-major scores, second stage: 64 columns a block, eight waves that share a
# column's row-block partials, eight loads at a time.  n gives 0, 1, 7, 8, 9
# and 65 partials (16 rows each on grids this small) and a last row block of
# one row; m the edges of a 64-column block.
@pytest.mark.parametrize("n", [0, 1, 16 * 7, 16 * 8, 16 * 9, 16 * 65 + 1])
@pytest.mark.parametrize("m", [1, 63, 64, 65, 513])
def test_row_major_scores_second_stage(n, m):
    g = gbits(n, m, 7 * n + m)
    got = f32_np(zf.colnorm(bf16_dev(g)))
    # fp64 sums of exact squares in another order, rounded once to fp32: half
    # an ulp on either side
    ok, worst = rel_close(got, (O.widen(g).astype(np.float64) ** 2).sum(0), 2.0 ** -23)
    assert ok, (n, m, worst)


# Selection: columns at the edges of the register variants (1, 4, 8, 16 and 32
# words of 64 columns for each of 16 waves) and beyond the last; scores that
# spread, that share one radix digit, and that tie.
@pytest.mark.parametrize("m", [1, 64, 1023, 1024, 1025, 4096, 4097, 8193, 16384, 16385, 32768,
                               32769, 70001])
@pytest.mark.parametrize("kind", ["spread", "narrow", "ties", "constant", "signed"])
def test_selection_variants(m, kind):
    rng = np.random.default_rng(m)
    if kind == "spread":
        s = np.exp(3.0 * rng.standard_normal(m)).astype(np.float32)
    elif kind == "narrow":
        s = (np.float32(1.0).view(np.uint32) + rng.integers(0, 900, m)).astype(np.uint32).view(np.float32)
    elif kind == "ties":
        s = rng.integers(0, 4, m).astype(np.float32)
    elif kind == "constant":
        s = np.full(m, 2.5, np.float32)
    else:  # negative scores, both zeros and infinities order like the floats
        s = np.where(rng.random(m) < 0.2, 0.0, rng.standard_normal(m)).astype(np.float32)
        s = np.where(rng.random(m) < 0.1, -s, s)
        s[rng.integers(0, m, 3)] = [np.inf, -np.inf, np.float32(3.4e38)]
    dev = torch.from_numpy(s).cuda()
    for ratio in (0.0, 0.1, 0.5, 1.0 - 1.0 / max(m, 2), 1.0):
        k = zf.k_from_ratio(ratio, m)
        got, want = zf.topk_select(dev, ratio), O.select_topk(s, k)
        assert np.array_equal(got.sel_idx.cpu().numpy(), want.sel), (m, kind, ratio)
        assert np.array_equal(got.unsel_idx.cpu().numpy(), want.unsel), (m, kind, ratio)
        assert np.array_equal(mask_np(got.mask), want.mask), (m, kind, ratio)
        assert np.array_equal(got.prefix.cpu().numpy(), want.prefix), (m, kind, ratio)

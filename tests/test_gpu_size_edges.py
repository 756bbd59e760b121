"""Kernels at the sizes where their splits of the work can go wrong (edges of
tiles, remainders, the smallest and largest of a variant's range), against the
oracle or fp64 torch."""
import numpy as np
import pytest
import torch

import oracle as O
from tests._gpu import bf16_dev, bits_np, f32_np, rel_close, same_bits

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

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


# Row-major Zen-auto: the 16-byte update with its statistics (and on a refresh
# the packing pass with them, after the per-column Adam) against the
# per-column update with the separate statistics pass, which buffers off the
# 16-byte path run.  Same fp64 partials in the same order: identical bits.
# Rows at the edges of the row batches and row blocks, columns at the edges of
# the tiles (multiples of 64 up to 960, else of 8 up to 1000).
@pytest.mark.parametrize("n", [1, 15, 17, 129])
@pytest.mark.parametrize("m", [8, 960, 961, 1000, 1921])
def test_row_major_zen_paths_agree(n, m):
    k = zf.k_from_ratio(0.1, m)
    dev = torch.device("cuda")
    rng = np.random.default_rng(n + 7 * m)
    g = [gbits(n, m, 11 * n + m + t) for t in range(3)]
    w0 = O.bf16_round((0.02 * rng.standard_normal((n, m))).astype(np.float32))
    master = torch.from_numpy(rng.standard_normal((n, m)).astype(np.float32)).to(dev)
    scores = [torch.from_numpy(rng.random(m).astype(np.float32)).to(dev) for _ in range(2)]
    got = []
    for aligned in (True, False):
        def bf16(b):
            return bf16_dev(b, ld=-(-m // 8) * 8) if aligned else bf16_dev(b, offset=1)

        sels = [zf.topk_select(s, 0.1) for s in scores]
        w = bf16(w0)
        acc = zf.alloc_stored(zf.ROW_MAJOR, n, m - k)
        st = [[zf.alloc_stored(zf.ROW_MAJOR, n, k) for _ in range(3)] for _ in range(2)]
        sq = torch.zeros(k, device=dev), torch.zeros(m - k, device=dev)
        totals = torch.zeros(zf.ZEN_TOTALS_BYTES // 8, dtype=torch.int64, device=dev)
        out = []
        # init, in place, remap (from the master) to another selection
        for t, (mode, p) in enumerate([(zf.STATES_INIT, 0), (zf.STATES_INPLACE, 0),
                                       (zf.STATES_REMAP, 1)]):
            src = zf.StateSource(prev=sels[1 - p], prev_master=st[1 - p][0],
                                 prev_exp_avg=st[1 - p][1], prev_exp_avg_sq=st[1 - p][2],
                                 init_master=master)
            plan = zf.Plan([zf.MatrixBuffers(
                grad=bf16(g[t]), k=k, sel=sels[p], weight=w, master=st[p][0], exp_avg=st[p][1],
                exp_avg_sq=st[p][2], acc=acc, src=src, sel_sq=sq[0], acc_sq=sq[1])])
            plan.update_zen(zf.AdamHparams(lr=1e-3), t + 1, mode, 1 + (t == 1), 4, 1.0, totals)
            torch.cuda.synchronize()
            out += [x.clone() for x in (w, acc, *st[p], *sq, totals)]
            plan.close()
        got.append(out)
    for i, (a, b) in enumerate(zip(*got)):
        assert torch.equal(a.view(torch.int16) if a.dtype == torch.bfloat16 else a,
                           b.view(torch.int16) if b.dtype == torch.bfloat16 else b), (n, m, i)

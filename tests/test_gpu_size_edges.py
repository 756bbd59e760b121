"""Kernels at the sizes where their splits of the work can go wrong (edges of
tiles, remainders, the smallest and largest of a variant's range), against the
oracle or fp64 torch."""
import numpy as np
import pytest
import torch

import oracle as O
from tests._gpu import bf16_dev, bits_np, f32_np, mask_np, rel_close, same_bits

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


# ... and so many columns that blocks of eight waves would pass the work-items
# of one launch (one partial a column: exact squares, rounded once).
def test_row_major_scores_of_a_very_wide_row():
    m = (1 << 29) + 5
    g = torch.randn(1, m, device="cuda", dtype=torch.bfloat16)
    assert torch.equal(zf.colnorm(g), (g[0].float() ** 2))


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


# Row-major Zen-auto on 16-byte rows (the 16-byte update with its statistics, on a
# refresh the packing pass with them after the per-column Adam) and off them (at
# these sizes the per-column update and a statistics pass), against the
# channel-major kernels: identical states, weights and sums, statistics up to
# the order of the fp64 sums (half an ulp of fp32 on either side).  Rows at the
# edges of the row batches and row blocks, columns at the edges of the tiles
# (multiples of 64 up to 960, else of 8 up to 1000).
@pytest.mark.parametrize("n", [1, 15, 17, 129])
@pytest.mark.parametrize("m", [8, 960, 961, 1000, 1921])
def test_row_major_zen_against_channel_major(n, m):
    k = zf.k_from_ratio(0.1, m)
    dev = torch.device("cuda")
    rng = np.random.default_rng(n + 7 * m)
    g = [gbits(n, m, 11 * n + m + t) for t in range(3)]
    w0 = O.bf16_round((0.02 * rng.standard_normal((n, m))).astype(np.float32))
    master = torch.from_numpy(rng.standard_normal((n, m)).astype(np.float32)).to(dev)
    scores = [torch.from_numpy(rng.random(m).astype(np.float32)).to(dev) for _ in range(2)]
    got = []
    for form in ("channel", "aligned", "unaligned"):
        cm = form == "channel"
        L = zf.CHANNEL_MAJOR if cm else zf.ROW_MAJOR

        def bf16(b):
            if cm:
                return bf16_dev(np.ascontiguousarray(b.T))
            return bf16_dev(b, offset=1) if form == "unaligned" else bf16_dev(b, ld=-(-m // 8) * 8)

        sels = [zf.topk_select(s, 0.1) for s in scores]
        w = bf16(w0)
        acc = zf.alloc_stored(L, n, m - k)
        st = [[zf.alloc_stored(L, n, k) for _ in range(3)] for _ in range(2)]
        sq = torch.zeros(k, device=dev), torch.zeros(m - k, device=dev)
        totals = torch.zeros(zf.ZEN_TOTALS_BYTES // 8, dtype=torch.int64, device=dev)
        out = []
        # init, in place, remap (from the master) to another selection
        for t, (mode, p) in enumerate([(zf.STATES_INIT, 0), (zf.STATES_INPLACE, 0),
                                       (zf.STATES_REMAP, 1)]):
            src = zf.StateSource(prev=sels[1 - p], prev_master=st[1 - p][0],
                                 prev_exp_avg=st[1 - p][1], prev_exp_avg_sq=st[1 - p][2],
                                 init_master=master.t().contiguous() if cm else master)
            plan = zf.Plan([zf.MatrixBuffers(
                grad=bf16(g[t]), k=k, sel=sels[p], weight=w, master=st[p][0], exp_avg=st[p][1],
                exp_avg_sq=st[p][2], acc=acc, src=src, sel_sq=sq[0], acc_sq=sq[1], layout=L)])
            plan.update_zen(zf.AdamHparams(lr=1e-3), t + 1, mode, 1 + (t == 1), 4, 1.0, totals)
            torch.cuda.synchronize()
            bits = [bits_np(w)] + [f32_np(x) for x in (acc, *st[p])]
            out.append(([x.T if cm else x for x in bits], [f32_np(x) for x in sq],
                        zf.ZenTotals.from_bytes(totals.cpu().numpy().tobytes())))
            plan.close()
        got.append(out)
    for form, other in zip(("aligned", "unaligned"), got[1:]):
        for t, ((bits, stats, tot), (bits2, stats2, tot2)) in enumerate(zip(got[0], other)):
            for i, (a, b) in enumerate(zip(bits, bits2)):
                assert same_bits(a, b), (form, n, m, t, i)
            for a, b in zip(stats, stats2):
                assert rel_close(b, a, 2.0 ** -22)[0], (form, n, m, t)
            # sums over columns of the roots of those: no column is off by more
            assert rel_close([tot2.sum_sel, tot2.sum_acc], [tot.sum_sel, tot.sum_acc], 2.0 ** -22)[0]
            assert (tot2.k_total, tot2.u_total) == (tot.k_total, tot.u_total)


# Row-major sets that are wide and large enough for the 16-byte update although
# no buffer has 16-byte rows (2^26 elements, tiles of 640 columns or more),
# against the same data in 16-byte rows: identical bits in every pass.  Columns
# at the edges of a tile, of an 8-column group and of a tile's slot quads, a last
# row block of a few rows.
@pytest.mark.parametrize("m", [641, 1000, 1921, 4001])
def test_row_major_large_sets_in_rows_of_any_alignment(m):
    n = -(-(1 << 26) // m)
    dev, hp, k = torch.device("cuda"), zf.AdamHparams(lr=1e-3, weight_decay=0.01), zf.k_from_ratio(0.1, m)
    gen = torch.Generator(device=dev).manual_seed(m)

    def buf(dtype, cols, aligned):
        if aligned:
            return zf.alloc_stored(zf.ROW_MAJOR, n, cols, dtype)
        return torch.empty(n * (cols + 1 + cols % 2) + 1, dtype=dtype, device=dev)[1:].view(
            n, cols + 1 + cols % 2)[:, :cols]

    def twins(dtype, cols, scale=1.0, fill=None):
        src = (torch.randn(n, cols, generator=gen, device=dev) * scale if fill is None
               else torch.full((n, cols), fill, device=dev))
        return [buf(dtype, cols, al).copy_(src) for al in (True, False)]

    sel = zf.topk_select(torch.rand(m, generator=gen, device=dev), 0.1)
    G = [twins(torch.bfloat16, m) for _ in range(3)]
    W = twins(torch.bfloat16, m, 0.02)
    st = [twins(torch.float32, k, 0.02), twins(torch.float32, k, 1e-3), twins(torch.float32, k, fill=1e-4)]
    acc, out = twins(torch.float32, m - k, fill=0.0), twins(torch.float32, m, fill=0.0)
    stage = [zf.alloc_stored(zf.ROW_MAJOR, n, m, torch.bfloat16).zero_() for _ in range(2)]
    sq = [(torch.zeros(k, device=dev), torch.zeros(m - k, device=dev)) for _ in range(2)]
    totals = [torch.zeros(zf.ZEN_TOTALS_BYTES // 8, dtype=torch.int64, device=dev) for _ in range(2)]
    plans = []
    for a in range(2):
        kw = dict(k=k, sel=sel, weight=W[a], master=st[0][a], exp_avg=st[1][a],
                  exp_avg_sq=st[2][a], acc=acc[a], unpacked=out[a], layout=zf.ROW_MAJOR)
        plans.append(([zf.Plan([zf.MatrixBuffers(grad=g[a], **kw)]) for g in G],
                      [zf.Plan([zf.MatrixBuffers(grad=g[a], acc_first=stage[a], **kw)]) for g in G],
                      zf.Plan([zf.MatrixBuffers(grad=G[0][a], sel_sq=sq[a][0], acc_sq=sq[a][1], **kw)])))
    I = zf.STATES_INPLACE
    calls = [("first", lambda a, P, S, Z: P[0].update(hp, 1, I, 1, 4)),
             ("later", lambda a, P, S, Z: P[1].update(hp, 2, I, 2, 4)),
             ("hand-over", lambda a, P, S, Z: P[2].update_handover(hp, 3, I, 3, 3, 1 / 3)),
             ("first, stage", lambda a, P, S, Z: S[0].update(hp, 4, I, 1, 4)),
             ("second, stage", lambda a, P, S, Z: S[1].update(hp, 5, I, 2, 4)),
             ("second, stage, hand-over", lambda a, P, S, Z: S[1].update_handover(hp, 6, I, 2, 2, 0.5)),
             ("Adam", lambda a, P, S, Z: P[1].update(hp, 7, I, 1, 4, pack=False)),
             ("packing", lambda a, P, S, Z: P[2].update(hp, 8, I, 2, 4, adam=False)),
             ("deferred", lambda a, P, S, Z: P[2].update_handover_deferred(hp, 9, P[:2], 0.25)),
             ("Zen-auto", lambda a, P, S, Z: Z.update_zen(hp, 10, I, 2, 4, 1.0, totals[a]))]
    for name, call in calls:
        for a in range(2):
            call(a, *plans[a])
        torch.cuda.synchronize()
        for i, (x, y) in enumerate([W, *st, acc, out, stage, totals, *zip(*sq)]):
            it = torch.int16 if x.dtype == torch.bfloat16 else torch.int32 if x.dtype == torch.float32 else x.dtype
            assert torch.equal(x.view(it), y.view(it)), (name, i)
    for P, S, Z in plans:
        for p in (*P, *S, Z):
            p.close()


# The runner on rows of any alignment, bit for bit against the oracle.
# Row-major: gradient rows of an odd number of elements (all phases, with and
# without the bf16 stage, the deferred hand-over).
# Channel-major: channels of n % 8 != 0 through the ragged kernels, n at the
# edges of a quad, a lane's quads, a chunk and the shortest channels that take
# quads (350 rows in the hand-over of kept gradients, else 850), next to an aligned matrix and to a long odd one.
def _odd_runner(layout, shapes, how):
    cm = layout == zf.CHANNEL_MAJOR
    R, S, T = 8, 4, 9
    hp = zf.AdamHparams(lr=1e-3, weight_decay=0.01)

    def dev(b):
        return bf16_dev(np.ascontiguousarray(b.T) if cm else b)

    def host(t):
        x = bits_np(t) if t.dtype == torch.bfloat16 else f32_np(t)
        return np.ascontiguousarray(x.T) if cm else x

    bits = [[gbits(n, m, 100 * n + m + t) for n, m in shapes] for t in range(4)]
    w = [O.bf16_round((0.02 * np.random.default_rng(n).standard_normal((n, m))).astype(np.float32))
         for n, m in shapes]
    wd = [dev(x) for x in w]
    r = zf.SelectiveUpdateRunner(shapes, 0.1, hp, R, S, [[dev(b) for b in s] for s in bits], wd,
                                 layout=layout, first_step_stage=how == "stage",
                                 deferred_pack=how == "deferred",
                                 fuse_handover=how != "separate")
    orc = [O.MatrixOracle(O.widen(x), x, 0.1, hp.lr, hp.beta1, hp.beta2, hp.eps, hp.weight_decay,
                          R, S) for x in w]
    for t in range(1, T + 1):
        kind = r.step()
        torch.cuda.synchronize()
        for q, o in enumerate(orc):
            want = o.step(bits[(t - 1) % 4][q])
            assert np.array_equal(host(wd[q]), o.W), (t, q)
            for got, exp in zip(r.state[q], (o.P, o.M, o.V)):
                assert same_bits(host(got), exp), (t, q)
            if kind.interval_end:
                assert same_bits(host(r.unpacked[q]), want["unpacked"]), (t, q)


@pytest.mark.parametrize("shape", [(33, 1003), (130, 965), (7, 9), (64, 2049)])
@pytest.mark.parametrize("how", ["stage", "plain", "deferred"])
def test_row_major_odd_rows_runner(shape, how):
    _odd_runner(zf.ROW_MAJOR, [shape], how)


@pytest.mark.parametrize("n", [1, 3, 5, 255, 349, 351, 849, 851, 999, 1001, 1027, 2047, 2049, 4099])
@pytest.mark.parametrize("how", ["stage", "plain", "separate", "deferred"])
def test_channel_major_odd_channels_runner(n, how):
    _odd_runner(zf.CHANNEL_MAJOR, [(n, 21), (64, 10), (1003, 5)], how)


# Channel-major scores of channels of any length: element by element below 850
# rows, else whole groups of eight and the rows after them, and both stores a refresh may ride on the pass.
@pytest.mark.parametrize("n", [1, 7, 8, 9, 511, 513, 849, 851, 999, 1001, 2048, 2055, 4099])
def test_channel_major_odd_scores(n):
    m, dev = 13, torch.device("cuda")
    g = gbits(n, m, n)
    want = (O.widen(g).astype(np.float64) ** 2).sum(0)
    for offset in (0, 1, 3):
        G = bf16_dev(np.ascontiguousarray(g.T), offset=offset)
        norms = torch.zeros(m, device=dev)
        out = torch.full((m, n), float("nan"), device=dev)
        stage = torch.zeros(m, n, dtype=torch.bfloat16, device=dev)
        w, acc = torch.zeros_like(stage), torch.zeros(m - 1, n, device=dev)
        st = [torch.zeros(1, n, device=dev) for _ in range(3)]
        plan = zf.Plan([zf.MatrixBuffers(
            grad=G, k=1, sel=zf.Selection(m, 1), weight=w, master=st[0], exp_avg=st[1],
            exp_avg_sq=st[2], acc=acc, norms=norms, unpacked=out, acc_first=stage,
            layout=zf.CHANNEL_MAJOR)])
        for call in (plan.colnorm, plan.colnorm_stage, lambda: plan.colnorm_handover(0.5)):
            norms.zero_()
            call()
            torch.cuda.synchronize()
            assert rel_close(f32_np(norms), want, 2.0 ** -23)[0], (n, offset)
        assert np.array_equal(bits_np(stage), g.T), (n, offset)
        assert same_bits(f32_np(out), O.widen(g).T * np.float32(0.5)), (n, offset)
        plan.close()


# Channel-major hand-over of kept gradients, with four and with eight of them in
# flight: intervals around both, short and long channels, on and off the aligned
# path, fixed and gated.  The additions in step order, each one fp32 operation.
@pytest.mark.parametrize("n", [64, 349, 351, 1023, 4096, 4099])
@pytest.mark.parametrize("steps", [2, 4, 5, 8, 9, 16])
def test_channel_major_handover_of_kept_gradients(n, steps):
    m, k, dev, hp = 21, 2, torch.device("cuda"), zf.AdamHparams(lr=1e-3)
    gen = torch.Generator(device=dev).manual_seed(n + steps)
    G = [torch.randn(m, n, generator=gen, device=dev).bfloat16() for _ in range(steps)]
    sel = zf.topk_select(torch.rand(m, generator=gen, device=dev), 0.1)
    out = torch.empty(m, n, device=dev)
    st = [torch.zeros(k, n, device=dev) for _ in range(3)]
    w = torch.zeros(m, n, dtype=torch.bfloat16, device=dev)
    plans = [zf.Plan([zf.MatrixBuffers(grad=g, k=k, sel=sel, weight=w, master=st[0], exp_avg=st[1],
                                       exp_avg_sq=st[2], unpacked=out, layout=zf.CHANNEL_MAJOR)])
             for g in G]

    def want(kept):
        a = G[-kept].float()
        for g in G[steps - kept + 1:]:
            a = a + g.float()
        a = a * np.float32(1.0 / kept).item()
        a[sel.sel_idx.long()] = 0.0
        return a

    out.fill_(float("nan"))
    plans[-1].update_handover_deferred(hp, 3, plans[:-1], float(np.float32(1.0 / steps)))
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int32), want(steps).view(torch.int32))
    for kept in {1, 2, steps}:
        out.fill_(float("nan"))
        plans[-1].handover_zen_deferred(plans[:-1], torch.tensor([kept, 1], dtype=torch.int32, device=dev))
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int32), want(kept).view(torch.int32)), kept
    for p in plans:
        p.close()

"""The work whose speed this repository answers for.

Each case is a piece of a training program that uses the library: the
per-matrix calls on one weight, or a SelectiveUpdateRunner stepping one
decoder layer (or a set of odd-sized weights) through whole refresh periods.
Shapes are the Llama-2 layer shapes of `workloads/`, the paper's ratio,
intervals and AdamW settings, plus generic small and odd sizes.

A case is a dict of plain values:
  kind      "calls"  -- the per-matrix entry points over a two-step interval:
                        scores, selection, Adam and packing of the first step,
                        Adam and packing of the second, hand-over
                        ("fused": update_fused / update_fused_handover instead
                        of the separate calls);
            "runner" -- SelectiveUpdateRunner.step, `steps` times;
  shapes    "n x m" of every weight (n outputs, m input channels);
  layout    "row" (PyTorch's [out, in]) or "channel" (its transpose);
  ratio     the selected share of the channels;
  refresh, accum, steps   the schedule (R, S, steps of one pass; a multiple
            of R, so that every pass starts with a refresh and ends with a
            hand-over);
  deferred  packing deferred to the interval's last step;
  tau       Zen-auto's threshold, 0 for the fixed schedule;
  offload   the offloaded optimizer (overlapped; a pass ends with sync());
  master    fp32 master weights given (else the bf16 weights are the start);
  decay     AdamW weight decay.
"""

import math

import torch

import paper_2505_12242_amd as zf

LAYER_7B = "4096x4096 4096x4096 4096x4096 4096x4096 11008x4096 11008x4096 4096x11008"
LAYER_13B = "5120x5120 5120x5120 5120x5120 5120x5120 13824x5120 13824x5120 5120x13824"
LAYER_70B = "8192x8192 1024x8192 1024x8192 8192x8192 28672x8192 28672x8192 8192x28672"
LAYER_SMALL = "1024x1024 1024x1024 1024x1024 1024x1024 2816x1024 2816x1024 1024x2816"

LR, BETA1, BETA2, EPS = 1e-5, 0.9, 0.999, 1e-8


def _case(kind, shapes, layout, ratio, refresh, accum, steps, deferred=False, tau=0.0,
          offload=False, master=False, decay=0.0, fused=False, name=None):
    c = {"kind": kind, "shapes": shapes, "layout": layout, "ratio": ratio, "refresh": refresh,
         "accum": accum, "steps": steps, "deferred": deferred, "tau": tau, "offload": offload,
         "master": master, "decay": decay, "fused": fused}
    return dict(c, name=name) if name is not None else c


def listed():
    return [
        # The smallest calls: one small projection, a handful of launches whose
        # latency is the cost.
        _case("calls", "512x512", "row", 0.10, 2, 2, 2, master=True, name="weight-512"),
        # One 4096 x 4096 weight through the five per-matrix entry points, a
        # fresh selection and a packed interval.
        _case("calls", "4096x4096", "row", 0.10, 2, 2, 2, master=True, name="weight-4096"),
        # A weight with odd sizes (an unpadded vocabulary, a pruned projection)
        # in the channel-major layout, through the fused calls.
        _case("calls", "5003x3001", "channel", 0.10, 2, 2, 2, master=True, fused=True,
              name="weight-odd-channel"),
        # A small model's layer, packing deferred: launches and the selection
        # weigh as much as the passes.
        _case("runner", LAYER_SMALL, "row", 0.10, 4, 4, 4, deferred=True,
              name="small-layer-row-deferred"),
        # One Llama-2-7B layer as the benchmark runs it: channel-major,
        # deferred packing, R = S = 4.
        _case("runner", LAYER_7B, "channel", 0.10, 4, 4, 4, deferred=True, name="7b-layer-channel"),
        # The same layer with PyTorch's own layout and the runner's defaults
        # (packing every step).
        _case("runner", LAYER_7B, "row", 0.10, 4, 4, 4, name="7b-layer-row"),
        # Zen-auto (the adaptive interval) decided on the device, both layouts.
        _case("runner", LAYER_7B, "channel", 0.10, 4, 4, 4, deferred=True, tau=1.0,
              name="7b-layer-zen-channel"),
        _case("runner", LAYER_7B, "row", 0.10, 4, 4, 4, tau=1.0, master=True,
              name="7b-layer-zen-row"),
        # The 13B sweep's end that refreshes every step and selects a quarter.
        _case("runner", LAYER_13B, "channel", 0.25, 1, 4, 2, decay=0.01, name="13b-layer-refresh1"),
        # The largest: one Llama-2-70B layer with an accumulation interval of 8.
        _case("runner", LAYER_70B, "channel", 0.10, 8, 8, 8, deferred=True, name="70b-layer-channel"),
        # Odd sizes in PyTorch's layout: rows that are not 16-byte aligned, two
        # intervals to a refresh.
        _case("runner", "3001x5003 5003x3001 2999x3001", "row", 0.10, 8, 4, 8, master=True,
              name="odd-row"),
        # The offloaded optimizer: the store in pinned host memory, the
        # deferred update on the host overlapped with the next interval.
        _case("runner", "4096x4096 4096x4096", "channel", 0.10, 4, 4, 8, offload=True,
              name="offload-channel"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi):
    """A size between lo and hi: any integer (odd ones among them), or one
    of the multiples of 64 that layers mostly have."""
    x = _log(rng, lo, hi)
    return x if rng.random() < 0.4 else max(64, 64 * round(x / 64))


def draw(rng):
    layout = rng.choice(["row", "channel"])
    ratio = rng.choice([0.01, 0.05, 0.10, 0.25])
    master = rng.random() < 0.5
    decay = rng.choice([0.0, 0.01])
    if rng.random() < 0.35:
        n, m = _size(rng, 256, 16384), _size(rng, 256, 12288)
        return _case("calls", f"{n}x{m}", layout, ratio, 2, 2, 2, master=master, decay=decay,
                     fused=rng.random() < 0.5)
    hidden = _size(rng, 512, 4096)
    ffn = int(hidden * rng.uniform(2.5, 3.5))
    if rng.random() < 0.6:
        ffn = max(64, 64 * round(ffn / 64))
    kv = hidden if rng.random() < 0.6 else max(64, hidden // 8)
    shapes = [(hidden, hidden), (kv, hidden), (kv, hidden), (hidden, hidden), (ffn, hidden),
              (ffn, hidden), (hidden, ffn)]
    shapes = " ".join(f"{n}x{m}" for n, m in shapes[:rng.randint(1, 7)])
    accum = rng.choice([2, 4, 8])
    refresh = min(8, accum * rng.choice([1, 1, 2])) if rng.random() < 0.85 else 1
    tau = rng.choice([0.0, 0.0, 1.0])
    deferred = rng.random() < 0.5 and refresh > 1 and not (tau and layout == "row")
    return _case("runner", shapes, layout, ratio, refresh, accum, max(refresh, 2),
                 deferred=deferred, tau=tau, master=master, decay=decay)


def _shapes(case):
    return [tuple(int(x) for x in s.split("x")) for s in case["shapes"].split()]


def _layout(case):
    return zf.ROW_MAJOR if case["layout"] == "row" else zf.CHANNEL_MAJOR


def _slots(case):
    """Gradient buffers: one for every step of a pass, at most those of an
    interval and its refresh period's reuse (step t reads slot t - 1 modulo
    their number)."""
    if case["kind"] == "calls":
        return 2
    return min(case["steps"], max(2, case["accum"]))


def _inputs(case, seed):
    """Gradients by slot, bf16 weights and fp32 masters, all stored in the
    case's layout: independent normal elements times a lognormal scale per
    input channel (a few channels carry most of the norm) that persists
    between steps up to 5% jitter."""
    dev = torch.device("cuda")
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed))
    row = case["layout"] == "row"
    slots = [[] for _ in range(_slots(case))]
    weights, masters = [], []
    for n, m in _shapes(case):
        shape = (n, m) if row else (m, n)
        base = torch.exp(1.5 * torch.randn(m, generator=g, device=dev)) * 1e-4
        for s in slots:
            scale = base * torch.exp(0.05 * torch.randn(m, generator=g, device=dev))
            x = torch.randn(shape, generator=g, device=dev)
            x *= scale[None, :] if row else scale[:, None]
            s.append(x.to(torch.bfloat16))
            del x
        p = torch.randn(shape, generator=g, device=dev) * 0.02
        weights.append(p.to(torch.bfloat16))
        masters.append(p if case["master"] else None)
        del p
    return slots, weights, masters


def _hp(case):
    return zf.AdamHparams(LR, BETA1, BETA2, EPS, case["decay"])


def prepare(case, seed):
    slots, weights, masters = _inputs(case, seed)
    layout = _layout(case)
    if case["kind"] == "runner":
        return {"case": case, "runner": zf.SelectiveUpdateRunner(
            _shapes(case), case["ratio"], _hp(case), case["refresh"], case["accum"], slots,
            weights, init_master=masters if case["master"] else None, layout=layout,
            zen_tau=case["tau"] or None, offload=case["offload"],
            deferred_pack=case["deferred"])}
    (n, m), = _shapes(case)
    k = zf.k_from_ratio(case["ratio"], m)
    f32 = torch.float32
    return {
        "case": case, "hp": _hp(case), "layout": layout, "g": [s[0] for s in slots],
        "w": weights[0], "sel": zf.Selection(m, k), "norms": torch.empty(m, dtype=f32, device="cuda"),
        "ws": torch.empty(max(8, zf.colnorm_workspace_bytes(n, m, layout)), dtype=torch.uint8,
                          device="cuda"),
        "p": [zf.alloc_stored(layout, n, k, f32) for _ in range(3)],
        "acc": zf.alloc_stored(layout, n, m - k, f32), "out": zf.alloc_stored(layout, n, m, f32),
        # the first step starts every selected column from the fp32 master, or
        # from the bf16 weights as they are then
        "src": zf.StateSource(init_master=masters[0]),
    }


def run(state):
    case = state["case"]
    if case["kind"] == "runner":
        r = state["runner"]
        for _ in range(case["steps"]):
            r.step()
        if case["offload"]:
            r.sync()
            return {"weight": r.weights, "state": [list(s) for s in r.state],
                    "store": [list(s) for s in r.store],
                    "sel": [s.sel_idx for s in r.selection]}
        out = {"weight": r.weights, "state": [list(s) for s in r.state], "out": r.unpacked,
               "norms": r.norms, "sel": [s.sel_idx for s in r.selection]}
        if case["tau"]:
            out["sel_sq"], out["acc_sq"] = r.sel_sq, r.acc_sq
        return out
    s = state
    L, sel, hp, w, src, ratio = s["layout"], s["sel"], s["hp"], s["w"], s["src"], case["ratio"]
    g1, g2 = s["g"]
    P, M, V = s["p"]
    zf.colnorm(g1, out=s["norms"], workspace=s["ws"], layout=L)
    zf.topk_select(s["norms"], ratio, out=sel)
    if case["fused"]:
        zf.update_fused(g1, sel, P, M, V, w, hp, 1, s["acc"], 1, 2, mode=zf.STATES_INIT, src=src,
                        layout=L)
        zf.update_fused_handover(g2, sel, P, M, V, w, hp, 2, s["acc"], 2, 2, 0.5, out=s["out"],
                                 layout=L)
    else:
        zf.adam_selected(g1, sel, P, M, V, w, hp, 1, mode=zf.STATES_INIT, src=src, layout=L)
        zf.pack_accumulate(g1, sel, s["acc"], 1, 2, layout=L)
        zf.adam_selected(g2, sel, P, M, V, w, hp, 2, layout=L)
        zf.pack_accumulate(g2, sel, s["acc"], 2, 2, layout=L)
        zf.unpack(s["acc"], sel, 0.5, out=s["out"], layout=L)
    return {"norms": s["norms"], "sel": [sel.sel_idx, sel.unsel_idx, sel.mask, sel.prefix],
            "state": [P, M, V], "weight": w, "acc": s["acc"], "out": s["out"]}


def work(case):
    """Each gradient read once by the step it belongs to (and once more by a
    refresh's scores), the selected channels' states read and written and
    their weights written by every step, the hand-over written once per
    interval.  Zen-auto's and the packing's running sums are not counted: they
    are neither inputs nor outputs.  The offloaded optimizer reads and writes
    the unselected channels' states once per interval."""
    total = flops = 0.0
    R, S, T = case["refresh"], case["accum"], case["steps"]
    for n, m in _shapes(case):
        k = zf.k_from_ratio(case["ratio"], m)
        sel, uns = float(n * k), float(n * (m - k))
        refreshes = sum((t - 1) % R == 0 for t in range(1, T + 1))
        ends = sum(t % R == 0 or t % S == 0 for t in range(1, T + 1))
        total += refreshes * (2.0 * n * m + 8.0 * m) + T * (28.0 * sel + 2.0 * uns)
        total += ends * (26.0 * uns if case["offload"] else 4.0 * n * m)
        if case["kind"] == "calls":
            total += 4.0 * uns  # the packed buffer is an output of its own
        flops += refreshes * 2.0 * n * m + T * (15.0 * sel + uns) + ends * uns
    return {"bytes": total, "flops": flops}


def tolerance(case):
    """fp32 element sequences and fp64 sums rounded once.  Against exact() the
    fp32 outputs are 2e-8 to 1.1e-7 off; a bf16 weight that an ulp of its fp32
    master tips over is off by one bf16 step (2^-7 of the value at most),
    which makes the weights up to 5e-6 off."""
    return {"rel": 2e-5, "max": 8e-3, "differ": 0.0}


# ---------------------------------------------------------------------------
# The same work in plain torch, fp64
# ---------------------------------------------------------------------------

def _select(score, k):
    """The k columns with the largest score, equal ones to the lower index."""
    order = torch.sort(score, descending=True, stable=True).indices
    idx = torch.sort(order[:k]).values
    mask = torch.zeros(score.numel(), dtype=torch.bool, device=score.device)
    mask[idx] = True
    return idx, torch.nonzero(~mask).flatten()


def _adam(g, p, m, v, t, decay):
    m = BETA1 * m + (1 - BETA1) * g
    v = BETA2 * v + (1 - BETA2) * g * g
    u = (m / (1 - BETA1 ** t)) / (torch.sqrt(v / (1 - BETA2 ** t)) + EPS)
    return p - LR * decay * p - LR * u, m, v


class _Matrix:
    """One weight in fp64, stored channel by channel ([m, n])."""

    def __init__(self, case, q, slots, weights, masters):
        self.row = case["layout"] == "row"
        self.case = case
        self.slots = [s[q] for s in slots]
        p = masters[q] if masters[q] is not None else weights[q]
        self.w = self.cm(weights[q]).double()
        self.start = self.cm(p)
        self.m, self.n = self.start.shape
        self.k = zf.k_from_ratio(case["ratio"], self.m)
        self.sel = self.uns = self.p = self.mo = self.v = None
        self.sum = None
        self.out = None
        if case["offload"]:
            z = torch.zeros(self.m, self.n, dtype=torch.float64, device="cuda")
            self.store = [self.start.double(), z, z.clone()]

    def cm(self, t):
        return t.t() if self.row else t

    def stored(self, t):
        return t.t().contiguous() if self.row else t

    def grad(self, t):
        return self.cm(self.slots[(t - 1) % len(self.slots)]).double()

    def refresh(self, g):
        self.norms = g.square().sum(1)
        old = (self.sel, self.p, self.mo, self.v)
        self.sel, self.uns = _select(self.norms.float(), self.k)
        if self.case["offload"]:
            self.p, self.mo, self.v = (x[self.sel] for x in self.store)
        else:
            base = self.start if self.case["master"] else self.w
            self.p = base[self.sel].double()
            self.mo = torch.zeros_like(self.p)
            self.v = torch.zeros_like(self.p)
        if old[0] is None:
            return
        # a column that stays keeps its states; one that leaves goes to the
        # store (if there is one)
        at = torch.full((self.m,), -1, dtype=torch.int64, device="cuda")
        at[old[0]] = torch.arange(self.k, device="cuda")
        src = at[self.sel]
        stay = src >= 0
        for new, was in zip((self.p, self.mo, self.v), old[1:]):
            new[stay] = was[src[stay]]
        if self.case["offload"]:
            at[self.sel] = -1
            left = torch.nonzero(at >= 0).flatten()
            for full, was in zip(self.store, old[1:]):
                full[left] = was[at[left]]

    def update(self, g, t):
        self.p, self.mo, self.v = _adam(g[self.sel], self.p, self.mo, self.v, t, self.case["decay"])
        self.w[self.sel] = self.p.to(torch.bfloat16).double()

    def accumulate(self, g, first):
        self.sum = g[self.uns] if first else self.sum + g[self.uns]

    def hand_over(self, steps, th):
        if not self.case["offload"]:
            self.out = torch.zeros(self.m, self.n, dtype=torch.float64, device="cuda")
            self.out[self.uns] = self.sum / steps
            return
        new = _adam(self.sum / steps, *(x[self.uns] for x in self.store), th, self.case["decay"])
        for full, part in zip(self.store, new):
            full[self.uns] = part
        self.w[self.uns] = new[0].to(torch.bfloat16).double()

    def state(self):
        return [self.stored(x) for x in (self.p, self.mo, self.v)]


def exact(case, seed):
    slots, weights, masters = _inputs(case, seed)
    mats = [_Matrix(case, q, slots, weights, masters) for q in range(len(weights))]
    R, S = case["refresh"], case["accum"]
    length, ended, th = 0, True, 0
    for t in range(1, case["steps"] + 1):
        refresh = (t - 1) % R == 0
        length = 1 if refresh or ended else length + 1
        root_sel, root_acc = [], []
        for x in mats:
            g = x.grad(t)
            if refresh:
                x.refresh(g)
            x.update(g, t)
            x.accumulate(g, length == 1)
            if case["tau"]:
                x.sel_sq, x.acc_sq = g[x.sel].square().sum(1), x.sum.square().sum(1)
                root_sel.append(x.sel_sq.sqrt())
                root_acc.append(x.acc_sq.sqrt())
        ended = t % R == 0 or (length >= S if case["tau"] else t % S == 0)
        if case["tau"]:
            a, b = torch.cat(root_acc), torch.cat(root_sel)
            ended = ended or bool(a.mean() >= case["tau"] * b.mean())
        if ended:
            th += 1
            for x in mats:
                x.hand_over(length, th)
    if case["kind"] == "calls":
        x, = mats
        return {"norms": x.norms, "sel": [None] * 4, "state": x.state(), "weight": x.stored(x.w),
                # the fused hand-over leaves the first step's values packed
                "acc": x.stored(mats[0].grad(1)[x.uns] if case["fused"] else x.sum),
                "out": x.stored(x.out)}
    got = {"weight": [x.stored(x.w) for x in mats], "state": [x.state() for x in mats],
           "sel": [None] * len(mats)}
    if case["offload"]:
        # a selected column's part of the store holds what it held when the
        # column entered the selection
        got["store"] = [[x.stored(y) for y in x.store] for x in mats]
        return got
    got["out"], got["norms"] = [x.stored(x.out) for x in mats], [x.norms for x in mats]
    if case["tau"]:
        got["sel_sq"], got["acc_sq"] = [x.sel_sq for x in mats], [x.acc_sq for x in mats]
    return got

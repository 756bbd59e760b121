"""Which kernels a call launches, and what it refuses, without a GPU.

The library's host side is run in a process of its own in which the HIP
runtime's launches and copies are replaced by ones that only take notes
(tests/native/hip_record.cpp).  Fake device addresses are never read."""
import ctypes
import json
import os
import shutil
import subprocess
import sys

import pytest

from tests.conftest import ROOT

RM, CM = 0, 1
INPLACE, REMAP, INIT = 0, 1, 2
EINVAL = 1


# ---------------------------------------------------------------------------
# the recording process
# ---------------------------------------------------------------------------

class Recorder:
    def __init__(self):
        from paper_2505_12242_amd import _lib
        self.L = _lib
        self.rec = ctypes.CDLL(os.environ["ZF_RECORDER"])
        self.buf = ctypes.create_string_buffer(1 << 16)
        self.hp = _lib.ZfAdamHparams(1e-5, 0.9, 0.999, 1e-8, 0.0)
        self.top = 0x100000000000
        self.state = self.addr(8192, 0)
        self.names = {}

    def addr(self, nbytes, off):
        """A fresh fake address, `off` bytes past a 4 KiB boundary."""
        p = self.top + off
        self.top += (nbytes + off + 8192) & ~4095
        return p

    def matrix(self, n, m, layout, off16=0, off32=0, zen=False, grad=True, ld=None, acc=True,
               stage=False, ratio=0.1):
        """off16 / off32: bytes the bf16 gradient / the fp32 buffers start past
        a 16-byte boundary; ld: the weight's row stride in elements."""
        k = self.L.LIB.zf_k_from_ratio(ratio, m)
        x = self.L.ZfMatrix()
        x.n, x.m, x.k, x.layout = n, m, k, layout
        rows, cols = (n, m) if layout == RM else (m, n)

        def store(r, c, size, off=0, stride=None):
            """(address, stride): rows padded to 16 bytes unless off is given."""
            per = 16 // size
            s = stride or (c if off or layout == CM else max(per, -(-c // per) * per))
            return self.addr(max(r, 1) * s * size, off), s

        def part(count):  # n x count in the layout
            return (n, count) if layout == RM else (count, n)

        if grad:
            x.grad, x.ld_grad = store(rows, cols, 2, off16)
        else:
            x.grad, x.ld_grad = None, cols
        x.weight, x.ld_weight = store(rows, cols, 2, stride=ld)
        for name in ("master", "exp_avg", "exp_avg_sq"):
            p, x.ld_state = store(*part(k), 4, off32)
            setattr(x, name, p)
        if acc:
            x.acc, x.ld_acc = store(*part(m - k), 4, off32)
        x.unpacked, x.ld_unpacked = store(rows, cols, 4, off32)
        x.norms_sq = self.addr(4 * m, 0)
        x.sel = self.L.ZfSelection(self.addr(4 * m, 0), self.addr(4 * m, 0), self.addr(m, 0),
                                   self.addr(m, 0))
        if zen:
            x.sel_sq, x.acc_sq = self.addr(4 * m, 0), self.addr(4 * m, 0)
        if stage:
            x.acc_first, x.ld_acc_first = store(rows, cols, 2)
        return x

    def plan(self, mats):
        arr = (self.L.ZfMatrix * len(mats))(*mats)
        nbytes, h = ctypes.c_size_t(), ctypes.c_void_p()
        st = self.L.LIB.zf_plan_query(arr, len(mats), ctypes.byref(nbytes))
        assert st == 0, st
        st = self.L.LIB.zf_plan_create(arr, len(mats), self.addr(nbytes.value, 0), nbytes.value,
                                       None, ctypes.byref(h))
        assert st == 0, st
        return h

    def call(self, fn, *args):
        """[status, [[kernel, grid, block], ...]]"""
        self.rec.rec_take(self.buf, len(self.buf))
        st = getattr(self.L.LIB, fn)(*args)
        self.rec.rec_take(self.buf, len(self.buf))
        out = []
        for ln in self.buf.value.decode().splitlines():
            name, grid, block = ln.rsplit(" ", 2)
            out.append([self.demangle(name), int(grid), int(block)])
        return [st, out]

    def demangle(self, name):
        if name not in self.names:
            s = subprocess.run(["c++filt", name], capture_output=True, text=True).stdout.strip()
            s = s.replace("(anonymous namespace)::", "").replace("void ", "").replace("zf::", "")
            self.names[name] = s.split("(")[0]
        return self.names[name]

    # the calls -------------------------------------------------------------
    def update(self, p, mode=INPLACE, sii=3, adam=1, pack=1):
        return self.call("zf_plan_update", p, ctypes.byref(self.hp), 5, mode, sii, 8, adam, pack,
                         None)

    def zen(self, p, mode=INPLACE, force=0):
        return self.call("zf_plan_update_zen_device", p, ctypes.byref(self.hp), 5, mode, 8, force,
                         1.0, self.state, self.state + 4096, None)

    def fused(self, x, mode=INPLACE):
        return self.call("zf_update_fused", x.grad, x.n, x.m, x.ld_grad, x.layout,
                         ctypes.byref(x.sel), x.k, x.master, x.exp_avg, x.exp_avg_sq, x.ld_state,
                         x.weight, x.ld_weight, ctypes.byref(self.hp), 5, mode, None, x.acc,
                         x.ld_acc, 2, 4, None)

    def adam(self, x, mode=INPLACE):
        return self.call("zf_adam_selected", x.grad, x.n, x.m, x.ld_grad, x.layout,
                         ctypes.byref(x.sel), x.k, x.master, x.exp_avg, x.exp_avg_sq, x.ld_state,
                         x.weight, x.ld_weight, ctypes.byref(self.hp), 5, mode, None, None)

    def deferred(self, p, earlier):
        hs = (ctypes.c_void_p * len(earlier))(*[e.value for e in earlier])
        return self.call("zf_plan_update_handover_deferred", p, ctypes.byref(self.hp), 5, hs,
                         len(earlier), 0.25, None)


def scenarios(r):
    out = {}
    # deferred hand-over, an earlier step without a gradient
    for layout in (RM, CM):
        for off in (0, 2):
            for ratio in (0.1, 1.0):
                a = [r.matrix(64, 72, layout, off16=off, ratio=ratio)]
                e = [r.matrix(64, 72, layout, off16=off, ratio=ratio)]
                none = [r.matrix(64, 72, layout, off16=off, ratio=ratio, grad=False)]
                if layout == CM and off:  # the same access path as the plan's
                    none[0].weight += 2
                p = r.plan(a)
                out[f"no-grad {layout} {off} {ratio}"] = [r.deferred(p, [r.plan(e)]),
                                                          r.deferred(p, [r.plan(none)])]
    # row-major routes by alignment, width and size
    for name, shapes, kw in ROW_MAJOR_SETS:
        mats = [r.matrix(n, m, RM, zen=True, **kw) for n, m in shapes]
        p, e = r.plan(mats), r.plan([r.matrix(n, m, RM, **kw) for n, m in shapes])
        out["rm " + name] = {
            "fused": r.update(p), "init": r.update(p, INIT), "adam": r.update(p, pack=0),
            "pack": r.update(p, adam=0), "deferred": r.deferred(e, [e]), "zen": r.zen(p),
            "zen-init": r.zen(p, INIT), "zen-end": r.zen(p, force=2),
            "call-fused": r.fused(mats[0]), "call-adam": r.adam(mats[0])}
    # channel-major hand-over of kept gradients: how many in flight
    for n, m, off in ((1024, 40, 0), (4096, 40, 0), (1023, 40, 2), (4095, 40, 2)):
        x = [r.matrix(n, m, CM, off16=off, zen=True)]
        p = r.plan(x)
        for steps in (2, 4, 5, 8):
            hs = (ctypes.c_void_p * 16)(*[p.value] * (steps - 1))
            out[f"kept {n} {steps}"] = [
                r.deferred(p, [p] * (steps - 1)),
                r.call("zf_plan_handover_zen_deferred", p, hs, steps - 1, r.state, None)]
    # column tiles of the row-major 16-byte update (one row: one row block)
    out["tiles"] = {str(m): r.update(r.plan([r.matrix(1, m, RM)]), adam=0) for m in TILE_COLUMNS}
    # second stage of the row-major column sums
    for n, m in ((128, 4096), (144, 4096), (4096, 4096), (1, (1 << 30) - 1), (0, 64)):
        ws = r.L.LIB.zf_colnorm_workspace_bytes(n, m, RM)
        out[f"scores {n} {m}"] = [r.call("zf_colnorm", r.addr(2 * n * m, 0), n, m, m, RM,
                                         r.addr(4 * m, 0), r.addr(ws, 0), ws, None)]
    for name, shapes in (("few", [(128, 72)] * 3), ("many", [(144, 72), (4096, 72)]),
                         ("huge", [(4096, 72)] + [(1, (1 << 26) - 8)] * 9)):
        p = r.plan([r.matrix(n, m, RM, zen=True) for n, m in shapes])
        out["scores " + name] = [r.call("zf_plan_colnorm", p, None), r.zen(p)]
    return out


TILE_COLUMNS = [1, 8, 63, 64, 65, 960, 961, 1000, 1001, 1024, 1920, 1921, 2000, 2001, 4096, 5120,
                8192, 11008, 13824, 28672, 32000, 70001]

# name, shapes, and how their buffers lie (off16 / off32: bytes past a 16-byte
# boundary, rows then unpadded)
ROW_MAJOR_SETS = [
    ("aligned small", [(64, 72)], {}),
    ("aligned narrow", [(50000, 32)], {}),
    ("odd rows, small", [(1024, 1023)] * 8, {"off16": 2}),
    ("odd rows, five small", [(1024, 1024)] * 4 + [(1024, 1023)], {"off16": 2}),
    ("odd states, small", [(1024, 1024)], {"off32": 4}),
    ("odd rows, narrow", [(1 << 20, 33)], {"off16": 2}),
    ("odd rows, tiles of 512", [(65600, 1023)], {"off16": 2}),
    ("odd rows, 2^22 wide", [(1049, 4001)], {"off16": 2}),
    ("odd rows, 2^24 wide", [(4194, 4001)], {"off16": 2}),
    ("odd rows, 2^25 wide", [(8387, 4001)], {"off16": 2}),
    ("odd rows, 2^25 wide over 8", [(1049, 4001)] * 8, {"off16": 2}),
    ("odd rows, 2^26 wide", [(16774, 4001)], {"off16": 2}),
    # a weight whose row stride is too long for the statistics' row blocks
    ("long rows", [(64, 72)], {"ld": 1 << 26}),
]

if __name__ == "__main__":
    print("RESULT " + json.dumps(scenarios(Recorder())))
    sys.exit(0)


# ---------------------------------------------------------------------------
# the tests
# ---------------------------------------------------------------------------

@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None or shutil.which("c++filt") is None:
        pytest.skip("g++ and c++filt needed")
    so = str(tmp_path_factory.mktemp("rec") / "librec.so")
    subprocess.run([gxx, "-O1", "-std=c++17", "-shared", "-fPIC", "-o", so,
                    os.path.join(ROOT, "tests", "native", "hip_record.cpp"), "-ldl"], check=True)
    pre = os.environ.get("LD_PRELOAD", "")
    env = dict(os.environ, LD_PRELOAD=so + (":" + pre if pre else ""), ZF_RECORDER=so)
    run = subprocess.run([sys.executable, "-m", "tests.test_host_routes"], cwd=ROOT, env=env,
                         capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stdout + run.stderr
    line = [x for x in run.stdout.splitlines() if x.startswith("RESULT ")][-1]
    return json.loads(line[len("RESULT "):])


@pytest.mark.parametrize("off", [0, 2])
@pytest.mark.parametrize("ratio", [0.1, 1.0])
def test_deferred_handover_needs_the_earlier_gradients(routes, off, ratio):
    """Row-major, the hand-over reads whole rows of every earlier gradient,
    the selected columns too: a plan without one is refused whatever k.
    Channel-major reads the unselected channels only: with k = m there are
    none."""
    with_grad, without = routes[f"no-grad {RM} {off} {ratio}"]
    assert with_grad[0] == 0 and len(with_grad[1]) == 2
    assert without == [EINVAL, []]
    with_grad, without = routes[f"no-grad {CM} {off} {ratio}"]
    assert with_grad[0] == 0 and len(with_grad[1]) == 1
    assert without[0] == (0 if ratio == 1.0 else EINVAL)


COL, VEC = "update_kernel", "rv_update_kernel"
# the passes in which each set takes the 16-byte kernel
ROW_MAJOR_VEC = {
    "aligned small": {"fused", "adam", "pack", "deferred", "zen", "call-fused", "call-adam"},
    "aligned narrow": {"fused", "adam", "pack", "deferred", "zen", "call-fused", "call-adam"},
    "odd rows, small": {"deferred"},  # (8 M elements: the hand-over alone)
    "odd rows, five small": {"deferred"},
    "odd states, small": set(),
    "odd rows, narrow": set(),
    "odd rows, tiles of 512": {"deferred"},
    "odd rows, 2^22 wide": {"deferred"},
    "odd rows, 2^24 wide": {"deferred", "zen"},
    "odd rows, 2^25 wide": {"fused", "deferred", "zen", "call-fused"},
    "odd rows, 2^25 wide over 8": {"fused", "deferred", "zen"},
    "odd rows, 2^26 wide": {"fused", "adam", "pack", "deferred", "zen", "call-fused", "call-adam"},
    # (its plan with the Zen-auto statistics has blocks of 16 rows or more;
    # without them, and in the calls, 4 rows fit)
    "long rows": {"deferred", "call-fused", "call-adam"},
}


@pytest.mark.parametrize("name", list(ROW_MAJOR_VEC))
def test_row_major_routes(routes, name):
    """In place, packing alone and the hand-over: the 16-byte kernel where every
    buffer has 16-byte rows, or where the set is wide and large; a refresh: the
    per-column kernel; long rows: the per-column kernels."""
    got, vec = routes["rm " + name], ROW_MAJOR_VEC[name]

    def kernels(what):
        status, launches = got[what]
        assert status == 0, what
        return [x[0].split("<")[0] for x in launches]

    for what in ("fused", "adam", "pack", "call-fused", "call-adam"):
        assert kernels(what) == [VEC if what in vec else COL], what
    assert kernels("init") == [COL]
    adam = VEC if "adam" in vec or name == "long rows" else COL
    assert kernels("deferred") == [adam, VEC if "deferred" in vec else "rm_handover_deferred_kernel"]
    tail = ["rm_zen_finalize_kernel", "zen_total_kernel"]
    partial = ["rm_zen_partial_kernel"]
    zen = "zen" in vec
    assert kernels("zen") == ([VEC] if zen else [COL] + partial) + tail
    assert kernels("zen-end") == ([VEC] if zen else [COL] + partial) + tail
    assert kernels("zen-init") == ([COL, VEC] if zen else [COL] + partial) + tail


@pytest.mark.parametrize("n", [1023, 1024, 4095, 4096])
@pytest.mark.parametrize("steps", [2, 4, 5, 8])
def test_channel_major_gradients_in_flight(routes, n, steps):
    """Eight kept gradients in flight on long channels (in the gated hand-over
    from five steps on), four otherwise."""
    (st, fixed), (st2, gated) = routes[f"kept {n} {steps}"]
    rag = "true" if n % 8 else "false"
    assert st == 0 and st2 == 0
    assert [x[0] for x in fixed] == [
        f"cm_handover_deferred_kernel<{rag}, {8 if n > 2048 else 4}>"]
    assert [x[0] for x in gated] == [
        f"cm_unpack_zen_kernel<true, {rag}, {8 if n > 2048 and steps > 4 else 4}>"]


@pytest.mark.parametrize("name,waves", [("128 4096", 1), ("144 4096", 8), ("4096 4096", 8),
                                        (f"1 {(1 << 30) - 1}", 1), ("0 64", 1), ("few", 1),
                                        ("many", 8), ("huge", 1)])
def test_row_major_sums_second_stage(routes, name, waves):
    """One wave a block up to eight partials a column, and where eight would not
    fit one launch, whose work-items are a 32-bit count."""
    calls = routes["scores " + name]
    for status, launches in calls:
        assert status == 0
        assert all(grid * block < 1 << 32 for _, grid, block in launches)
        assert [block for k, _, block in launches if "finalize" in k] == [64 * waves]


@pytest.mark.parametrize("m", TILE_COLUMNS)
def test_row_major_column_tiles(routes, m):
    """One block a tile of the width that test_rv_geometry.py checks."""
    from tests.test_rv_geometry import rv_max_cols, rv_width
    status, launches = routes["tiles"][str(m)]
    assert status == 0 and len(launches) == 1 and launches[0][0].startswith("rv_update_kernel")
    assert launches[0][1] == -(-m // rv_width(m, rv_max_cols()))

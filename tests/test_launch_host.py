"""Host code that prepares and issues the launches, on the CPU: libdugks.so runs
over a stand-in for the HIP runtime (hip_stub.c), which hands every launch with
its arguments to the test.  The stand-in's symbols must come before the real
ones, so each case runs in a process of its own."""
import collections
import ctypes
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
NQUEUE = 8


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("stub") / "hip_stub.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-w", "-o", so,
                    os.path.join(HERE, "hip_stub.c")], check=True)
    return so


def run(stub, case, *args):
    r = subprocess.run([sys.executable, os.path.abspath(__file__), stub, case, *map(str, args)],
                       cwd=os.path.dirname(HERE), capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]


# ------------------------------------------------------------ in the process
class Dim3(ctypes.Structure):
    _fields_ = [(c, ctypes.c_uint32) for c in "xyz"]


class ItemPieces(ctypes.Structure):   # dugks_noalloc.hip
    _fields_ = [("qstart", ctypes.c_int32 * 9), ("n", ctypes.c_int32),
                ("start", ctypes.c_int32 * 264), ("grid", ctypes.c_int32 * 263),
                ("first", ctypes.c_int32 * 263)]


Event = collections.namedtuple("Event", "what obj blocks threads args")
HOOK = ctypes.CFUNCTYPE(None, ctypes.c_char_p, ctypes.c_void_p, Dim3, Dim3,
                        ctypes.POINTER(ctypes.c_void_p))


class Trace(list):
    """The calls since the last clear(); `on` may look at each as it is made."""

    def __init__(self, so):
        super().__init__()
        self.on = None
        self.error = None             # the first exception of `on` (ctypes drops them)

        def hook(what, obj, grid, block, args):
            e = Event(what.decode(), obj, grid.x * grid.y * grid.z,
                      block.x * block.y * block.z, args)
            self.append(e)
            try:
                if self.on:
                    self.on(e)
            except Exception as x:
                self.error = self.error or x

        self.hook = HOOK(hook)
        self.lib = ctypes.CDLL(so, mode=ctypes.RTLD_GLOBAL)
        self.lib.stub_set_hook(self.hook)

    def kernels(self, name):
        return [e for e in self if name in e.what]


def plan(C, nx, ny, precision=0, recon=1, flags=0, scheme=0, rows=0, vel=0):
    return C.dugks_plan_create(C.make_params(nx, ny, 0.02, 4.0, 0.5, recon, precision=precision,
                                             vel_kind=vel, flags=flags, scheme=scheme,
                                             tile_rows=rows))


LISTS = {"one 512": [512], "one 1000": [1000], "one 2048": [2048], "uneven": [512, 32, 40, 64],
         "large and small": [1600] + [64] * 40, "three": [1000, 999, 700], "tiny": [64, 40, 33],
         "mix": [32 + 37 * k % 480 for k in range(256)]}


def many_queues(C, trace, sizes, precision, flags, scheme):
    """dugks_step_many_noalloc gives the 8 XCDs equal work, whatever the grids
    (but whole grids where no XCD has more blocks than its 32 compute units); every
    tile of every grid is in the list once, taller marching tiles first within a
    queue."""
    pieces = ItemPieces()

    def on(e):
        if "noalloc_items_kernel" in e.what:
            ctypes.memmove(ctypes.byref(pieces), e.args[0], ctypes.sizeof(pieces))

    trace.on = on
    sizes = LISTS[sizes]
    plans = [plan(C, n, n, precision, 1, flags, scheme, 24 if n == 700 else 0) for n in sizes]
    C.dugks_step_many_noalloc(plans, [256] * len(plans), [0] * len(plans), 1, 0)
    total = pieces.qstart[NQUEUE]
    seen = collections.Counter()
    for p in range(pieces.n):
        for i in range(pieces.start[p], pieces.start[p + 1]):
            seen[pieces.grid[p], pieces.first[p] + i - pieces.start[p]] += 1
    assert len(seen) == total and set(seen.values()) == {1}
    tiles = [1 + max(t for g, t in seen if g == j) for j in range(len(sizes))]
    assert sum(tiles) == total
    block = trace.kernels("batch_tile_kernel")
    counts = [pieces.qstart[q + 1] - pieces.qstart[q] for q in range(NQUEUE)]
    if block:
        assert max(counts) <= 32 or max(counts) - min(counts) <= 1, counts
        assert all(e.blocks == NQUEUE * max(counts) for e in block)
        return
    # marching: a tile costs its rows (whole groups of 8) and 5 more; each cut is
    # less than a tile short of an eighth of all
    segs = [t // -(-n // 58) for n, t in zip(sizes, tiles)]
    cost = [min(n, 8 * -(-(-(-n // s)) // 8)) + 5 for n, s in zip(sizes, segs)]
    share = [0] * NQUEUE
    for p in range(pieces.n):
        q = max(k for k in range(NQUEUE) if pieces.qstart[k] <= pieces.start[p])
        share[q] += (pieces.start[p + 1] - pieces.start[p]) * cost[pieces.grid[p]]
    assert max(share) - min(share) < 2 * max(cost), share
    for p in range(pieces.n - 1):
        if pieces.start[p + 1] not in list(pieces.qstart):
            assert cost[pieces.grid[p]] >= cost[pieces.grid[p + 1]]


class BatchCtl(ctypes.Structure):     # dugks_kernels.h
    _fields_ = [("items", ctypes.POINTER(ctypes.c_int32 * 2)), ("nitems", ctypes.c_int32),
                ("nq", ctypes.c_int32), ("qstart", ctypes.c_int32 * 9)]


def batch_queues(C, trace, precision, flags, scheme):
    """A batch of which an eighth of the grids goes on after the others: each
    XCD's queue holds an eighth of the tiles that are left."""
    n, keep = 1024, 128
    plans = [plan(C, 256, 256, precision, 1, flags, scheme)] * n
    b = C.dugks_batch_create(n, precision, 1, flags | (C.BATCH_T3S3 if scheme else 0))
    for k, p in enumerate(plans):
        C.dugks_batch_set(b, k, p, 256, 0, 50 if k < keep else 5)
    C.dugks_batch_commit(b, 0)
    left = [0] * NQUEUE

    def on(e):
        if "batch_step_kernel" in e.what:
            ctl = ctypes.cast(ctypes.cast(e.args[2], ctypes.POINTER(ctypes.c_void_p))[0],
                              ctypes.POINTER(BatchCtl))[0]
            assert ctl.nq == NQUEUE and len({tuple(ctl.items[i]) for i in range(ctl.nitems)}) \
                == ctl.nitems == 5 * 16 * n
            for q in range(NQUEUE):
                left[q] = sum(ctl.items[i][0] < keep
                              for i in range(ctl.qstart[q], ctl.qstart[q + 1]))

    trace.on = on
    C.dugks_batch_step(b, 1, 0, 0)
    # a grid's bands differ by one tile
    assert sum(left) == 5 * 16 * keep and max(left) - min(left) <= keep, left


def graph_lifetime(C, trace):
    """An executable graph the batch replaces (its list has outgrown it, or the
    steps per graph changed) is not destroyed while a replay may be running: not
    before an event recorded after its last replay has been waited for or found
    passed (the stand-in's events never pass by themselves).  Never more than a
    few of them are kept, and destroying the batch leaves none."""
    sizes = [16, 64, 128, 256, 512]
    plans = [plan(C, n, n) for n in sizes]
    b = C.dugks_batch_create(len(sizes), 0, 1, 0)
    live, replayed, recorded, over = set(), {}, {}, set()
    clock = [0]
    most = [0]

    def on(e):
        clock[0] += 1
        if e.what == "instantiate":
            live.add(e.obj)
            most[0] = max(most[0], len(live))
        elif e.what == "graph_launch":
            assert e.obj in live
            replayed[e.obj] = clock[0]
        elif e.what == "event_record":
            recorded[e.obj] = clock[0]
        elif e.what == "event_sync":
            over.add(recorded.get(e.obj, 0))
        elif e.what == "device_sync":
            over.add(clock[0])
        elif e.what == "exec_destroy":
            assert any(t > replayed[e.obj] for t in over), "destroyed while it may be running"
            live.remove(e.obj)

    trace.on = on
    for k, p in enumerate(plans):      # the list grows, with a round in flight
        C.dugks_batch_set(b, k, p, 256, 0, 1 << 20)
        C.dugks_batch_commit(b, 0)
        C.dugks_batch_step(b, 16, 16, 0)
    for k in range(60):
        C.dugks_batch_step(b, 20, 4 + k % 3, 0)
    assert most[0] <= 24
    C.dugks_batch_destroy(b)
    assert not live


# (nx, ny, precision, recon, flags, scheme, tile_rows): rows of a marching tile, or 0
# for the tile kernel; both sides of each line (default and requested heights)
KERNELS = [
    # corrected FP64: one round of 512 blocks of 8 rows
    (448, 448, 0, 1, 2, 0, 0, 0), (512, 512, 0, 1, 2, 0, 0, 8), (768, 768, 0, 0, 2, 0, 0, 8),
    (512, 512, 0, 0, 2, 1, 0, 8), (768, 768, 0, 2, 2, 0, 0, 0),
    # corrected upwind-5
    (576, 576, 1, 3, 2, 0, 0, 0), (704, 704, 1, 3, 2, 0, 0, 8), (900, 900, 1, 3, 2, 0, 0, 8),
    (704, 704, 1, 3, 0, 0, 0, 0), (768, 768, 1, 3, 0, 0, 0, 8), (980, 980, 1, 3, 0, 0, 0, 16),
    (832, 832, 0, 3, 2, 0, 0, 0),
    (940, 940, 0, 3, 2, 0, 0, 16), (1000, 1000, 0, 3, 2, 0, 0, 0), (1000, 1300, 0, 3, 0, 0, 0, 24),
    (1100, 1100, 0, 3, 0, 0, 0, 0),
    # 8 rows asked for on large grids: marched at that height, as a height of 16 is
    (2048, 2048, 1, 1, 0, 0, 8, 8), (2048, 2048, 1, 1, 2, 0, 8, 8), (2048, 2048, 0, 1, 0, 0, 8, 8),
    (2048, 2048, 0, 1, 0, 1, 8, 8), (2500, 2500, 1, 3, 0, 0, 8, 8), (768, 768, 1, 3, 0, 0, 8, 8), (2048, 2048, 1, 1, 0, 0, 6, 6),
    (2048, 2048, 1, 1, 2, 0, 1, 8), (2048, 2048, 0, 1, 0, 0, 16, 16),
    # where the tile kernel beats that
    (2048, 2048, 0, 2, 0, 0, 8, 0), (2500, 2500, 0, 3, 2, 0, 8, 0), (1024, 1024, 0, 1, 0, 0, 8, 0),
    (2048, 2048, 1, 1, 0, 0, 2, 0), (150, 400, 0, 1, 0, 0, 8, 0),
    # more than 2^32 threads in 4-row tiles
    (60000, 60000, 1, 1, 0, 0, 3, 3),
    # the tilings of test_gpu_march_heights.py
    (150, 401, 0, 1, 0, 0, 9, 9), (150, 401, 1, 1, 0, 0, 12, 12), (800, 905, 1, 1, 2, 0, 8, 8),
    (75, 402, 0, 2, 0, 0, 9, 9, 4), (700, 563, 0, 1, 0, 1, 5, 5), (1003, 903, 0, 1, 2, 0, 1, 8),
    (1003, 903, 1, 1, 2, 0, 1, 8), (800, 803, 1, 3, 0, 0, 7, 7), (262, 221, 0, 0, 0, 0, 8, 0),
    (262, 222, 0, 1, 0, 0, 8, 0, 4), (301, 229, 0, 3, 0, 0, 8, 0), (301, 229, 1, 3, 0, 0, 8, 0),
    # default heights: FP32 with velocity arrays has 3 wavefronts per SIMD to fill
    (1900, 1900, 1, 2, 0, 0, 0, 22, 4), (1900, 1900, 1, 1, 0, 0, 0, 22, 4),
    (1024, 8192, 1, 2, 0, 0, 0, 16, 4), (3000, 3000, 1, 1, 0, 0, 0, 16, 4), (1900, 1900, 1, 1, 0, 0, 0, 34, 0),
]


def kernels(C, trace):
    for nx, ny, precision, recon, flags, scheme, asked, rows, *vel in KERNELS:
        p = plan(C, nx, ny, precision, recon, flags, scheme, asked, *vel)
        trace.clear()
        C.dugks_step(p, 256, 0, 1, 0)
        case = (nx, ny, precision, recon, flags, scheme, asked, rows)
        assert all(e.blocks * e.threads < 1 << 32 for e in trace), case
        march = trace.kernels("11step_kernel")
        assert bool(march) == (rows > 0) and bool(trace.kernels("tile_kernel")) == (rows == 0), case
        if rows:   # whole segments per XCD from 32 on, else whole tiles; not for upwind-5
            strips, segs = -(-nx // 58), -(-ny // rows)
            least = 8 * -(-segs // 8) * strips if segs >= 32 and recon != 3 else strips * segs
            assert all(least <= e.blocks < least + 8 * strips + 8 for e in march), case


def batch_of(C, sizes, precision=1, flags=2):
    b = C.dugks_batch_create(len(sizes), precision, 1, flags)
    for k, n in enumerate(sizes):
        C.dugks_batch_set(b, k, plan(C, n, n, precision, 1, flags), 256, 0, 1 << 20)
    C.dugks_batch_commit(b, 0)
    return b


def listed(C, trace, b):
    """(kernel, tiles in the list) of the batch's next step."""
    got = []

    def on(e):
        for name, k in (("batch_step_kernel", 2), ("batch_tile_kernel", 2)):
            if name in e.what:
                ctl = ctypes.cast(ctypes.cast(e.args[k], ctypes.POINTER(ctypes.c_void_p))[0],
                                  ctypes.POINTER(BatchCtl))[0]
                got.append((name, ctl.nitems))

    before, trace.on = trace.on, on
    C.dugks_batch_step(b, 1, 0, 0)
    trace.on = before
    return got[0]


def batch_tuning(C, trace):
    """The tuner keeps what measured fastest, the batch's own choice among it, and
    a tuner that fails leaves the batch's choice as it was."""
    fastest = [None]
    state = {}

    def on(e):   # the time of a candidate by the tiles of its list
        if "batch_step_kernel" in e.what or "batch_tile_kernel" in e.what:
            ctl = ctypes.cast(ctypes.cast(e.args[2], ctypes.POINTER(ctypes.c_void_p))[0],
                              ctypes.POINTER(BatchCtl))[0]
            state["last"] = ("batch_tile_kernel" in e.what, ctl.nitems)
        elif e.what == "elapsed":
            ctypes.cast(e.obj, ctypes.POINTER(ctypes.c_float))[0] = \
                1.0 if state["last"] == fastest[0] else 2.0

    trace.on = on
    # one grid of 1000^2, corrected FP32: marched 8 rows by default, 18 x 125 tiles
    b = batch_of(C, [1000])
    assert listed(C, trace, b) == ("batch_step_kernel", 18 * 125)
    fastest[0] = (False, 18 * 125)
    assert C.dugks_batch_tune(b, 1, 0) == 8 == C.dugks_batch_tile_rows(b)
    assert listed(C, trace, b) == ("batch_step_kernel", 18 * 125)
    C.dugks_batch_set_tile_rows(b, 8)
    C.dugks_batch_commit(b, 0)
    assert listed(C, trace, b) == ("batch_step_kernel", 18 * 125)
    fastest[0] = (False, 18 * 21)          # 48 rows
    assert C.dugks_batch_tune(b, 1, 0) == 48
    assert listed(C, trace, b) == ("batch_step_kernel", 18 * 21)
    # few grids: block tiles stay while they are few, then the best marching height
    b = batch_of(C, [64, 64, 64])
    fastest[0] = (True, 3 * 2 * 8)
    assert 16 <= C.dugks_batch_tune(b, 1, 0) <= 256
    assert listed(C, trace, b) == ("batch_tile_kernel", 3 * 2 * 8)
    C.dugks_batch_set(b, 0, plan(C, 2000, 2000, 1, 1, 2), 256, 0, 1 << 20)
    C.dugks_batch_commit(b, 0)
    assert listed(C, trace, b)[0] == "batch_step_kernel"
    # a device error on the way
    b = batch_of(C, [64, 64, 64])
    rc = ctypes.c_int.in_dll(trace.lib, "stub_event_sync_rc")
    rc.value = 1
    try:
        C.dugks_batch_tune(b, 1, 0)
        raise AssertionError("no error")
    except RuntimeError:
        pass
    rc.value = 0
    C.dugks_batch_commit(b, 0)
    assert listed(C, trace, b) == ("batch_tile_kernel", 3 * 2 * 8)
    # 8 rows asked for on a list too large for block tiles
    b = batch_of(C, [512] * 40)
    C.dugks_batch_set_tile_rows(b, 8)
    C.dugks_batch_commit(b, 0)
    assert listed(C, trace, b) == ("batch_step_kernel", 40 * 9 * 64)


def many_limit(C, trace):
    """dugks_step_many_noalloc: 115680 tiles of the heights the plans ask for."""
    def status(nx, ny, rows, flags=0):
        try:
            C.dugks_step_many_noalloc([plan(C, nx, ny, 1, 1, flags, 0, rows)], [256], [0], 1, 0)
        except C.DugksError as e:
            return e.code
        return C.OK

    strips = 142                        # 8192 columns
    assert status(8192, 115680 // strips * 8, 8) == C.OK
    assert status(8192, 115680 // strips * 8 + 8, 8) == C.EINVAL
    assert status(8192, 115680 // strips * 12, 12) == C.OK
    assert status(8192, 115680 // strips * 12 + 1, 12) == C.EINVAL
    assert status(8192, 115680 // strips * 8, 1, C.FLAG_MASS_FIX) == C.OK   # whole groups of 8
    assert status(8192, 8192, 0) == C.OK
    assert status(512, 512, 1) == C.OK


# --------------------------------------------------------------------- tests
@pytest.mark.parametrize("precision,flags,scheme", [(0, 0, 0), (1, 2, 0), (0, 0, 1), (1, 0, 0)])
@pytest.mark.parametrize("sizes", sorted(LISTS))
def test_allocation_free_step_spreads_over_the_xcds(stub, sizes, precision, flags, scheme):
    run(stub, "many_queues", sizes, precision, flags, scheme)


@pytest.mark.parametrize("precision,flags,scheme", [(0, 0, 0), (1, 2, 0), (0, 0, 1)])
def test_batch_spreads_what_goes_on_over_the_xcds(stub, precision, flags, scheme):
    run(stub, "batch_queues", precision, flags, scheme)


def test_replaced_graphs_outlive_their_replays(stub):
    run(stub, "graph_lifetime")


def test_kernel_and_height_of_a_step(stub):
    run(stub, "kernels")


def test_batch_tuner_keeps_the_fastest(stub):
    run(stub, "batch_tuning")


def test_allocation_free_step_limit(stub):
    run(stub, "many_limit")


if __name__ == "__main__":
    sys.path.insert(0, os.getcwd())
    the_trace = Trace(sys.argv[1])
    from paper_2007_07760_amd import _lib
    globals()[sys.argv[2]](_lib, the_trace,
                           *[int(a) if a.lstrip("-").isdigit() else a for a in sys.argv[3:]])
    if the_trace.error:
        raise the_trace.error

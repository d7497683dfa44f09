"""The library's host code (events, workspace, stream order, size limits) against a stand-in
HIP runtime: no GPU."""
import pytest

from tests import fake_hip


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    folder = tmp_path_factory.mktemp("fakehip")
    return lambda code: fake_hip.run(folder, code)


def test_the_stand_in_runs_every_path(run):
    """A sum with wave columns, workgroup columns and row windows: the kernels of each are
    launched and every call succeeds."""
    out = run("""
        BINS[3], BINS[G1], BINS[WIN], WINDOWS.value, TOTAL.value = 70, 5, 2, 9, 40
        s = Sum(1 << 20, 77, 6)
        st = s.all(stream(0))
        out = [st, s.nnz.value, sorted({x[0] for x in log()})]
    """)
    assert out[0] == [0, 0, 0] and out[1] == 40
    for k in ("k_bounds", "k_wave_sym_fused", "k_wave_pipe", "k_bitmap_wg", "k_win_records"):
        assert any(k in x for x in out[2]), k


# ---- launches ----

ROW = {threads: (2**32 - 1) // threads for threads in (64, 256, 512, 1024)}


@pytest.mark.parametrize("what, opts, bins, windows, kernel, blocks", [
    # row windows, of which a workgroup takes one
    ("windows", dict(), {"WIN": 2}, ROW[512] + 1, "k_bitmap_wg", 2 * (ROW[512] + 1)),
    ("windows", dict(window_cap=8192), {"WIN": 2}, ROW[1024] + 1, "k_bitmap_wg", 2 * (ROW[1024] + 1)),
    ("windows", dict(accum_mode=1), {"WIN": 2}, 2 * ROW[512] + 1, "k_hash_wg", 2 * (2 * ROW[512] + 1)),
    # workgroup columns
    ("columns", dict(), {"G1": ROW[256] + 1}, 0, "k_bitmap_wg", 2 * (ROW[256] + 1)),
    ("columns", dict(), {"G3": ROW[1024] + 1}, 0, "k_bitmap_wg", 2 * (ROW[1024] + 1)),
    ("columns", dict(accum_mode=1), {"G1": ROW[256] + 1}, 0, "k_hash_wg", 2 * (ROW[256] + 1)),
    # columns cut into windows, of which the planning kernels take one a workgroup
    ("columns", dict(), {"WIN": ROW[256] + 1}, ROW[256] + 1, "k_win_fill", ROW[256] + 1),
    ("columns", dict(flags=16), {"WIN": ROW[256] + 1}, ROW[256] + 1, "k_uwin_chfill", ROW[256] + 1),
    # a wavefront a column, four of them a workgroup
    ("waves", dict(accum_mode=1), {"W3": ROW[64] + 1}, 0, "k_num_wave", (ROW[64] + 4) // 4),
])
def test_launches_of_more_blocks_than_a_grid_row(run, what, opts, bins, windows, kernel, blocks):
    """As many units as make 2^32 work-items and more of a launch: every launch stays below that,
    and together they have a block for every unit."""
    n = sum(bins.values())
    out = run(f"""
        F.fake_limit(1 << 40)
        W3 = 3
        for b, c in {bins!r}.items():
            BINS[dict(W3=3, G1=G1, G3=G3, WIN=WIN)[b]] = c
        WINDOWS.value, TOTAL.value = {windows}, 40
        st = Sum(1 << 30, {n}, {65 if what == "waves" else 2}, **{opts!r}).all(stream(0))
        out = [st, [x[0] for x in log() if x[0] == "refused"], F.fake_blocks({kernel!r}.encode())]
    """)
    assert out[0] == [0, 0, 0] and out[1] == []
    assert blocks <= out[2] <= blocks + 2 * 4096 * 3, out[2] - blocks


@pytest.mark.parametrize("unsorted", [False, True])
def test_passes_over_more_elements_than_a_grid_row(run, unsorted):
    """More chunks of the window columns' entries than a grid row has blocks, and (sorted inputs)
    2^32 boundary positions and more."""
    out = run(f"""
        F.fake_limit(1 << 40)
        BINS[WIN], WINDOWS.value, TOTAL.value = 2, {1 << 20 if unsorted else 1 << 25}, {ROW[256] + 1}
        st = Sum(1 << 30, 2, {2 if unsorted else 128}, flags={16 if unsorted else 0}).all(stream(0))
        out = [st, [x[0] for x in log() if x[0] == "refused"], F.fake_blocks(b"k_uwin_pass"),
               F.fake_blocks(b"k_win_locate"), F.fake_blocks(b"k_win_bpos_t")]
    """)
    assert out[0] == [0, 0, 0] and out[1] == []
    if unsorted:
        assert out[2] >= 2 * (ROW[256] + 1)
    else:
        assert out[3] >= ROW[256] + 1 and out[4] * 256 >= ((1 << 25) + 2) * 128


@pytest.mark.parametrize("most", [1000, 2**22])
def test_a_batch_for_many_requests(run, most):
    """A batch made for more requests than a grid row has blocks of its colptr pass."""
    out = run(f"""
        h, ptrs = ctypes.c_void_p(), (ctypes.c_void_p * 2)(ADDR, ADDR)
        a = ctypes.addressof(ptrs)
        q = B.Request(100, 5, 2, a, a, a, ADDR, ADDR, ADDR, 10)
        st = [L.spkadd_batch_create(ctypes.byref(h), 0, {most}, 1000, 1000, None)]
        st.append(L.spkadd_batch_run(h, ctypes.byref(q), 1, 0, stream(0)))
        out = [st, [x[0] for x in log() if x[0] == "refused"], F.fake_blocks(b"k_batch_scan")]
        L.spkadd_batch_destroy(h)
    """)
    assert out[0] == [0, 0] and out[1] == [] and most <= out[2] <= most + 1


# ---- events ----

def test_events_stay_on_their_device(run):
    """Sums on two devices in turn, whose workspace blocks and summaries take recycled events:
    none is recorded on a stream of another device, no call fails, and freeing a plan while
    another device is current does not mix them either."""
    out = run("""
        BINS[3], BINS[G1], BINS[WIN], WINDOWS.value, TOTAL.value = 70, 5, 2, 9, 40
        st = []
        for turn in range(4):
            for dev in (0, 1):
                F.hipSetDevice(dev)
                st += Sum(1 << 20, 77, 6).all(stream(dev, turn))
                st += Sum(1 << 20, 77, 6, flags=2).all(stream(dev, turn))
        F.hipSetDevice(0)
        s = Sum(1 << 20, 77, 6)
        st += [s.plan(stream(0)), s.symbolic(stream(0)), s.numeric(stream(0))]
        F.hipSetDevice(1)
        st.append(s.free())
        st += Sum(1 << 20, 77, 6).all(stream(1))
        out = [st, F.fake_foreign_records()]
    """)
    assert set(out[0]) == {0} and out[1] == 0


def test_a_release_without_its_event_leaves_no_status(run):
    """A block whose event cannot be recorded is released all the same, and the status of the
    failed record is not reported by the calls that follow."""
    out = run("""
        BINS[3], BINS[WIN], WINDOWS.value, TOTAL.value = 70, 2, 9, 40
        s = Sum(1 << 20, 77, 6)
        st = [s.plan(stream(0)), s.symbolic(stream(0)), s.numeric(stream(0))]
        F.fake_fail_records(100)
        st.append(s.free())
        out = [st, F.fake_last_error()]
        F.fake_fail_records(0)
        st += Sum(1 << 20, 77, 6).all(stream(0))
    """)
    assert set(out[0]) == {0} and out[1] == 0


def test_events_are_bounded(run):
    """Many plans at once, then none: what the pool keeps is bounded, and sums that follow each
    other make no new events."""
    out = run("""
        BINS[3], TOTAL.value = 70, 40
        plans = [Sum(1000, 70, 2, flags=2) for _ in range(600)]  # (traced: several events each)
        st = [p.plan(stream(0, i % 5)) for i, p in enumerate(plans)] + [p.free() for p in plans]
        kept = F.fake_events()
        for _ in range(3): st += Sum(1000, 70, 2).all(stream(0))
        made = F.fake_events_made()
        for _ in range(50): st += Sum(1000, 70, 2).all(stream(0))
        out = [st, kept, F.fake_events_made() - made]
    """)
    assert set(out[0]) == {0}
    assert out[1] <= 600 + 2 * 256  # (one of every cached block, and the pools')
    assert out[2] == 0


# ---- stream order ----

@pytest.mark.parametrize("windows", [0, 9])
@pytest.mark.parametrize("kind", ["deferred", "validated", "many inputs", "load factor"])
def test_symbolic_on_another_stream_follows_the_plan(run, kind, windows):
    """The symbolic pass on a second stream waits, before its first launch, for an event recorded
    after the plan's last launch on the first; where the plan itself waited for its bin counts
    and has no row windows, it builds the column lists (all that may still be missing) again."""
    out = run(f"""
        kind = {kind!r}
        BINS[3], BINS[WIN], WINDOWS.value, TOTAL.value = 70, min({windows}, 2), {windows}, 40
        s = Sum(1 << 20, 77, 200 if kind == "many inputs" else 6, flags=1 if kind == "validated" else 0,
                load_factor_num=0.25 if kind == "load factor" else 0.0)
        a, b = stream(0, 1), stream(0, 2)
        st = [s.plan(a), s.symbolic(b), s.numeric(b), s.free()]
        out = [st, log(), a.value, b.value]
    """)
    st, log, a, b = out
    assert set(st) == {0}
    on = lambda s: [i for i, x in enumerate(log) if x[0] not in ("malloc", "free") and int(x[1], 16) == s]
    first = on(b)[0]
    launched = [i for i in on(a) if log[i][0].startswith("_Z")]
    if kind != "deferred" and not windows:
        assert "k_bin_scatter" in log[first][0] and "k_bin_scatter" in log[launched[-1]][0]
        return
    assert log[first][0] == "wait" and launched[-1] < first
    recorded = [i for i in on(a) if log[i][0] == "record" and log[i][2] == log[first][2]]
    assert recorded and launched[-1] < recorded[-1] < first


# ---- the copy of the column pointers ----

TABLE = """
    BINS[3], BINS[G1], BINS[WIN], WINDOWS.value, TOTAL.value = 199000, 900, 100, 120000, 40
    s = Sum(1 << 20, 200000, 64)
"""


def test_a_sum_that_fits_without_the_copy_succeeds(run):
    """Device memory for everything but the copy of the column pointers: the sum gives the copy
    up when a later allocation fails, or does not make it, and no launch reads it afterwards."""
    peak, tables = run(TABLE + """
    st = s.all(stream(0))
    assert st == [0, 0, 0]
    out = [F.fake_peak(), F.fake_tables()]
    """)
    table = 1 << (200001 * 64 * 4 - 1).bit_length()
    assert tables > 0 and peak > 2 * table
    for limit in (peak - 4096, peak - table // 2, peak - table, table // 2):
        got = run(TABLE + f"""
    F.fake_limit({limit})
    st = s.all(stream(0))
    out = [st, F.fake_stale_tables(), s.message]
    """)
        assert got[1] == 0
        if limit >= peak - table:
            assert got[0] == [0, 0, 0], (limit, got)
        else:  # (the row windows alone need more)
            assert got[0] == [0, 2], got


def test_no_copy_above_its_limit(run):
    """More column pointers than the copy may hold (1 GiB): the kernels read the inputs' arrays;
    at the limit no more than 1 GiB is taken for it."""
    out = run("""
        BINS[3], TOTAL.value = 100, 40
        big, most = Sum(1000, (1 << 28) // 64, 64), Sum(1000, (1 << 28) // 64 - 1, 64)
        st = big.all(stream(0))
        out = [F.fake_tables(), F.fake_peak()]
        F.fake_peak_reset()
        st += most.all(stream(0))
        out += [F.fake_tables(), F.fake_peak() - out[1], st]
    """)
    assert set(out[4]) == {0}
    assert out[0] == 0 and out[2] > 0 and out[3] <= 1 << 30


@pytest.mark.parametrize("k,n,copied", [(5, 1 << 20, False), (6, 3071, False), (6, 3072, True), (128, 3071, False),
                                        (128, 3072, True), (4, 1000, False)])
def test_which_sums_copy_their_column_pointers(run, k, n, copied):
    """Few inputs, or arrays of a few pages, are read where they are."""
    out = run(f"""
        BINS[3], TOTAL.value = 100, 40
        out = [Sum(1000, {n}, {k}).all(stream(0)), F.fake_tables()]
    """)
    assert out[0] == [0, 0, 0] and (out[1] > 0) == copied


# ---- the no-allocation call's static array ----

def test_noalloc_takes_as_many_columns_as_before(run):
    """The largest sum without row windows that fitted the 64 MiB with fourteen bins fits with the
    bins there are now; one of 3% more columns does not, and says so."""
    out = run("""
        SCRATCH, TILE, THREADS = 64 << 20, None, 256
        def need(n, k, bins, tile):
            r = lambda x: (x + 255) // 256 * 256
            blocks = (n + THREADS - 1) // THREADS
            return (r(24 * k) + 3 * r(4 * n) + r(n) + r(4 * blocks * bins) + r(4 * (2 * bins + 1)) + r(96) +
                    r(4 * (n + 1)) + r(8 * ((n + tile - 1) // tile + 1)) + 4096)
        out = []
        BINS[3], TOTAL.value = 100, 40
        for k in (1, 4, 300):
            lo, hi = 1, 1 << 23
            while lo < hi:
                mid = (lo + hi + 1) // 2
                if need(mid, k, 14, 4096) <= SCRATCH: lo = mid
                else: hi = mid - 1
            out.append([lo, Sum(1000, lo, k).noalloc(stream(0)), Sum(1000, lo + lo // 32, k).noalloc(stream(0))])
    """)
    for n, fits, more in out:
        assert n > 3500000 and (fits, more) == (0, 6)


# ---- on-chip memory ----

@pytest.mark.parametrize("accum_mode", [0, 1])
@pytest.mark.parametrize("dtype", [0, 1])
def test_the_largest_number_of_inputs_is_refused_or_runs(run, dtype, accum_mode):
    """Around the number of inputs whose segment table just fits a workgroup's LDS (with the
    kernels' own arrays), a sum runs or is refused as unsupported: no launch fails."""
    out = run(f"""
        out = []
        for b in ([G1, G1 + 1, G3, WIN] if {accum_mode} == 0 else [G1, G1 + 1, WIN]):
            for i in range(WIN + 1): BINS[i] = 0
            BINS[b], WINDOWS.value, TOTAL.value = 5, 9 if b == WIN else 0, 40
            status = lambda k: Sum(1 << 20, 70, k, {dtype}, accum_mode={accum_mode}).all(stream(0))
            lo, hi = 1, 20000
            while lo < hi:
                mid = (lo + hi + 1) // 2
                if status(mid) == [0, 0, 0]: lo = mid
                else: hi = mid - 1
            out.append([b, lo, sorted({{status(k)[-1] for k in range(lo - 3, lo + 24)}})])
    """)
    for b, most, statuses in out:
        assert most >= 3719 and statuses == [0, 6], (b, most, statuses)


# ---- the tuner ----

@pytest.mark.parametrize("k", [6, 130])
def test_the_tuner_tries_load_factors_only_where_tables_are_used(run, k):
    """On bitmaps alone a load factor changes nothing: it is tried only with hash tables chosen
    before it, or with more inputs than the bitmaps of a wavefront take."""
    out = run(f"""
        BINS[3], TOTAL.value = 70, 1
        best, rep, trials = B.Opts(), B.TuneReport(), (B.TuneTrial * 200)()
        ptrs = (ctypes.c_void_p * {k})(*[ADDR] * {k})
        st = B._tune_fns().spkadd_tune(200000, 70, {k}, ptrs, ptrs, ptrs, 0, None, 1, ctypes.byref(best),
                                       ctypes.byref(rep), trials, 200, stream(0))
        out = [st, [(t.opts.accum_mode, round(t.opts.load_factor_sym, 2)) for t in trials[:rep.trials]]]
    """)
    assert out[0] == 0 and len(out[1]) >= 10
    assert all(f == 0.0 or a == 1 or k > 128 for a, f in out[1])
    assert k <= 128 or {0.35, 0.5, 0.7} <= {f for a, f in out[1]}

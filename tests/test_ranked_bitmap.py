"""The ranked bitmap of the wave kernels (matrices too tall for a bitmap of all their
rows) and two inputs per lane (64 < k <= 128), against the CPU oracle: rows bit-exact,
integer values bit-exact, real values within max(k, t) * u * sum|a|."""
import numpy as np
import pytest
import torch  # (before the library, which then shares its HIP runtime)

import oracle
import workloads
from tests.gpu_util import assert_matches, note, run_gpu

pytestmark = pytest.mark.gpu


def _opts(**kw):
    from paper_2112_10223_amd import binding
    return binding.make_opts(**kw)


def tall_batch(m, k, sizes, dtype, integers, seed):
    """Columns of about the given input entries, drawn from a pool of rows (so that inputs
    share rows) that holds the first and last rows of the matrix and of 64-row and
    4096-row blocks."""
    rng = np.random.default_rng(seed)
    edges = np.array([0, 1, 31, 32, 63, 64, 65, 4095, 4096, m - 1, m - 2, m - 64, m - 65, m // 2], dtype=np.int64)
    edges = edges[(edges >= 0) & (edges < m)]
    rows, cps = [[] for _ in range(k)], np.zeros((k, len(sizes) + 1), np.int32)
    for j, u in enumerate(sizes):
        pool = np.unique(np.concatenate([edges, rng.integers(0, m, size=max(2, int(0.8 * u)))]))
        if u == 0:
            pool = pool[:0]
        cnt = rng.multinomial(u, np.ones(k) / k)
        for i in range(k):
            r = np.sort(rng.choice(pool, size=min(int(cnt[i]), pool.shape[0]), replace=False)).astype(np.int32)
            rows[i].append(r)
            cps[i, j + 1] = cps[i, j] + r.shape[0]
    rows = [np.concatenate(r) for r in rows]
    if integers:
        vals = [rng.integers(-3, 4, size=r.shape[0]).astype(dtype) for r in rows]
    else:
        vals = [rng.uniform(-1, 1, size=r.shape[0]).astype(dtype) for r in rows]
    return workloads.CSCBatch(m, len(sizes), cps, rows, vals)


SIZES = [0, 1, 2, 63, 64, 65, 128, 129, 190, 250, 257, 320, 321, 384, 500, 512, 513, 640, 641, 768, 900, 1023, 1024, 7,
         0, 30]


@pytest.mark.parametrize("m", [70000, 1 << 19, (1 << 19) + 1, 1 << 21, (1 << 21) + 1, 1 << 27, (1 << 27) + 1,
                               (1 << 31) - 2])
@pytest.mark.parametrize("k", [1, 7, 64, 65, 128])
def test_levels(m, k):
    dtype = np.float64 if (m + k) % 2 else np.float32
    integers = k in (7, 65)
    note(f"ranked bitmap m={m} k={k} {dtype.__name__} integers={integers}")
    b = tall_batch(m, k, SIZES, dtype, integers, seed=m % 1000 + k)
    got = run_gpu(b, _opts(), stats=True)
    assert got[3]["n_wave_cols"] > 0
    assert_matches(b, got, oracle.spkadd(b), exact_values=integers)


@pytest.mark.parametrize("k", [65, 100, 127, 128, 129])
@pytest.mark.parametrize("accum_mode", [0, 1, 2])
def test_many_inputs(k, accum_mode):
    """Bitmap, ranked bitmap and hash tables at the edges of two inputs per lane (k = 129
    and hash tables above 64 take the unpipelined kernels)."""
    for m in (3000, 60000, 200000):
        note(f"many inputs k={k} m={m} accum_mode={accum_mode}")
        b = tall_batch(m, k, SIZES, np.float32, True, seed=k)
        assert_matches(b, run_gpu(b, _opts(accum_mode=accum_mode)), oracle.spkadd(b), exact_values=True)


def test_more_columns_than_resident_wavefronts():
    """Several units per wavefront (odd counts, replayed steps), one and two inputs per lane."""
    for k, m, n in ((9, 300001, 20001), (70, 90001, 9001)):
        note(f"ranked bitmap n={n} k={k}")
        b = workloads.er(m, n, k, 3.0, seed=k, values="int32f")
        assert_matches(b, run_gpu(b), oracle.spkadd(b), exact_values=True)


def test_batched_requests_with_few_entries():
    """Batched runs whose columns are too sparse for the bitmap, fused and one launch per
    slot, requests of several heights in one run."""
    from tests.gpu_util import to_device
    from paper_2112_10223_amd import binding
    reqs = [workloads.er(m, n, k, d, seed=m, values="int32f")
            for m, n, k, d in ((65536, 300, 7, 3.0), (1 << 20, 500, 40, 9.0), (5000001, 200, 64, 14.0), (300, 50, 2, 1.0),
                               ((1 << 21) + 1, 77, 20, 40.0))]
    for fused in (0, -1):
        note(f"batched ranked bitmap batch_fused_cols={fused}")
        bt = binding.Batch(binding.SPKADD_F32, 8, 4000, 400, _opts(batch_fused_cols=fused))
        args = []
        for b in reqs:
            cps, ris, vas = to_device(b)
            args.append({"m": b.m, "colptrs": cps, "rowidxs": ris, "values": vas, "cap_c": b.nnz_in,
                         "colptr_c": torch.zeros(b.n + 1, dtype=torch.int32, device="cuda:0"),
                         "rowidx_c": torch.zeros(b.nnz_in, dtype=torch.int32, device="cuda:0"),
                         "values_c": torch.zeros(b.nnz_in, dtype=torch.float32, device="cuda:0")})
        for _ in range(2):
            bt.run(args)
            nnz, status = bt.results()
        for b, q, z, st in zip(reqs, args, nnz, status):
            assert st == binding.SPKADD_REQ_OK
            got = (q["colptr_c"].cpu().numpy().astype(np.int64), q["rowidx_c"][:z].cpu().numpy(),
                   q["values_c"][:z].cpu().numpy())
            assert_matches(b, got, oracle.spkadd(b), exact_values=True)
        bt.close()


WG_SIZES = [1025, 1500, 2047, 2048, 2049, 3072, 3073, 4095, 4096, 4097, 5000, 6143, 6144, 6145, 8191, 8192, 8193, 12000,
            30000, 0, 3]


@pytest.mark.parametrize("m", [9000, 131072, 131073, 1 << 20, 40960 * 32 + 1, 163840 * 32 + 1, 1 << 27, (1 << 31) - 2])
@pytest.mark.parametrize("k", [1, 6, 64, 130])
def test_workgroup_levels(m, k):
    """Workgroup columns of all three sizes and row windows: one bit per row, one and two
    levels of ranked blocks; 64 columns and more take the large capacities."""
    dtype = np.float64 if (m // 7 + k) % 2 else np.float32
    integers = k in (6, 64)
    note(f"workgroup bitmap levels m={m} k={k} {dtype.__name__} integers={integers}")
    b = tall_batch(m, k, (WG_SIZES * 4)[:70], dtype, integers, seed=m % 1000 + k)
    got = run_gpu(b, _opts(), stats=True)
    assert got[3]["n_wg_cols"] > 0 and (m < 10000 or got[3]["n_window_cols"] > 0)
    assert_matches(b, got, oracle.spkadd(b), exact_values=integers)


@pytest.mark.parametrize("window_cap", [64, 1000, 4096, 5000, 8192])
def test_window_capacities(window_cap):
    """Windows in 512 and 1024 threads, windows of more entries than registers (dense rows),
    every column forced to windows."""
    for m, k, sizes in ((3000, 20, [40000, 9000, 100, 2500]), (1 << 21, 9, [40000, 9000, 100, 2500])):
        note(f"window_cap={window_cap} m={m}")
        b = tall_batch(m, k, sizes * 2, np.float32, True, seed=window_cap + k)
        ref = oracle.spkadd(b)
        for force in (-1, 1, 2):
            assert_matches(b, run_gpu(b, _opts(window_cap=window_cap, force_bin=force)), ref, exact_values=True)


@pytest.mark.parametrize("m,k", [(500, 24), (70000, 7), (70000, 100), ((1 << 21) + 1, 64), ((1 << 27) + 1, 3), (40, 128)])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_ordered_in_the_wave_kernels(m, k, dtype):
    """Values summed in input order by the wave kernels (both bitmaps, one and two inputs
    per lane, rows that most inputs share): bit-identical to the ordered oracle."""
    from paper_2112_10223_amd import binding
    note(f"ordered wave kernels m={m} k={k} {dtype.__name__}")
    b = tall_batch(m, k, SIZES + [1100, 3000], dtype, False, seed=m % 1000 + k)
    got = run_gpu(b, _opts(flags=binding.SPKADD_FLAG_ORDERED))
    ref = oracle.spkadd_ordered(b)
    assert np.array_equal(got[0], ref.colptr) and np.array_equal(got[1], ref.rowidx)
    assert np.array_equal(got[2], ref.val.astype(dtype))


def test_every_top_block_of_the_tallest_matrix():
    """A workgroup column with a row in each of the 64 top blocks of a 2^31 - 2 row matrix
    (small capacities: five levels of ranked blocks)."""
    note("workgroup bitmap, every top block")
    m = (1 << 31) - 2
    col = np.minimum(np.arange(64, dtype=np.int64) * (1 << 25) + np.arange(64) * 33, m - 1).astype(np.int32)
    rows = [np.concatenate([col[0::2], col[:3]]), np.concatenate([col[1::2], col[1:2]])]
    cps = np.array([[0, 32, 35], [0, 32, 33]], dtype=np.int32)
    vals = [np.arange(1, r.shape[0] + 1).astype(np.float32) for r in rows]
    b = workloads.CSCBatch(m, 2, cps, rows, vals)
    assert_matches(b, run_gpu(b, _opts(force_bin=1, window_cap=64)), oracle.spkadd(b), exact_values=True)

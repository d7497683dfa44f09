"""Sums whose kernels read the copy of the column pointers, and those just too small for it
(fewer than 6 inputs or 3,072 columns), against the CPU oracle."""
import numpy as np
import pytest
import torch  # (before the library, which then shares its HIP runtime)

import oracle
from tests.gpu_util import assert_matches, note, run_gpu
from tests.test_ranked_bitmap import tall_batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3071, 3072, 3073])
@pytest.mark.parametrize("k", [5, 6, 7, 16, 64, 65, 127, 129])
def test_both_sides_of_the_rule(n, k):
    """Columns of every kind (empty, wavefront, workgroup, row windows) at k around a multiple of
    the copy's 16-byte rows and of a lane's inputs."""
    from paper_2112_10223_amd import binding
    dtype = np.float64 if (n + k) % 2 else np.float32
    note(f"column table n={n} k={k} {dtype.__name__}")
    rng = np.random.default_rng(n + k)
    sizes = rng.integers(0, 12, size=n)
    at = rng.choice(n, size=12, replace=False)
    sizes[at] = [64, 65, 300, 640, 1000, 1024, 1025, 2049, 4097, 7000, 9000, 20000]
    sizes[-1], sizes[0] = 5, 700  # (the last column's end is the table's last row)
    b = tall_batch(1 << 20, k, sizes.tolist(), dtype, True, seed=k)
    ref = oracle.spkadd(b)
    got = run_gpu(b, stats=True)
    assert min(got[3]["n_wave_cols"], got[3]["n_wg_cols"], got[3]["n_window_cols"]) > 0
    assert_matches(b, got, ref, exact_values=True)
    for kw in ({"flags": binding.SPKADD_FLAG_ORDERED}, {"flags": binding.SPKADD_FLAG_UNSORTED_IN}, {"accum_mode": 1},
               {"force_bin": 1}):
        assert_matches(b, run_gpu(b, binding.make_opts(**kw)), ref, exact_values=True)


def test_a_refilled_plan():
    """Numeric passes over new values on a kept plan whose symbolic pass is done."""
    from paper_2112_10223_amd import binding
    from tests.gpu_util import to_device
    note("column table, refilled plan")
    rng = np.random.default_rng(7)
    b = tall_batch(60000, 24, rng.integers(0, 60, size=4000).tolist(), np.float32, True, seed=3)
    cps, ris, vas = to_device(b)
    plan = binding.spkadd_plan(b.m, b.n, cps, ris, binding.SPKADD_F32)
    try:
        c = torch.empty(b.n + 1, dtype=torch.int32, device="cuda:0")
        nnz = binding.spkadd_symbolic(plan, c)
        r = torch.empty(nnz, dtype=torch.int32, device="cuda:0")
        v = torch.empty(nnz, dtype=torch.float32, device="cuda:0")
        for scale in (1.0, -2.0):
            b2 = b.__class__(b.m, b.n, b.colptr, b.rowidx, [x * np.float32(scale) for x in b.vals])
            new = [torch.from_numpy(x).to("cuda:0") for x in b2.vals]
            binding.spkadd_numeric(plan, new, r, v)
            torch.cuda.synchronize()
            assert_matches(b2, (c.cpu().numpy().astype(np.int64), r.cpu().numpy(), v.cpu().numpy()), oracle.spkadd(b2),
                           exact_values=True)
    finally:
        plan.free()

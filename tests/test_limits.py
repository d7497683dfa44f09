"""The most inputs that fit a workgroup's LDS, and the largest window capacity, against the
CPU oracle."""
import numpy as np
import pytest
import torch  # (before the library, which then shares its HIP runtime)

import oracle
from tests.gpu_util import assert_matches, note, run_gpu, to_device
from tests.test_ranked_bitmap import tall_batch

pytestmark = pytest.mark.gpu

# (the most inputs with columns of one workgroup of 1024 threads; up to 3,721 ran at all times)
MOST = {np.float32: 4767, np.float64: 4373}


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("less", [0, 1, 300, -60])
def test_many_inputs_in_workgroup_columns(dtype, less):
    """Columns of one workgroup (all three sizes) and row windows of thousands of inputs, most of
    them empty in a column; a few inputs more are refused.  (Short columns are sent to workgroups
    too: wavefronts hold tables for 660 to 1,840 inputs.)"""
    from paper_2112_10223_amd import binding
    opts = binding.make_opts(force_bin=binding.SPKADD_BIN_WG)
    k = MOST[dtype] - less
    note(f"{k} inputs {dtype.__name__}")
    sizes = ([1100, 3000, 5000, 6100, 20000] + [3] * 10) * 5
    b = tall_batch(1 << 20, k, sizes[:70], dtype, True, seed=k)
    if less < 0:
        cps, ris, vas = to_device(b)
        with pytest.raises(binding.SpkaddError) as ei:
            binding.spkadd_plan(b.m, b.n, cps, ris, binding.SPKADD_F64 if dtype == np.float64 else binding.SPKADD_F32,
                                opts)
        assert ei.value.status == binding.SPKADD_ERR_UNSUPPORTED
        return
    got = run_gpu(b, opts, stats=True)
    assert got[3]["n_wg_cols"] > 0 and got[3]["n_window_cols"] > 0
    assert_matches(b, got, oracle.spkadd(b), exact_values=True)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("m", [9000, 1 << 21])
def test_largest_window_capacity(m, dtype):
    """window_cap = 8192: workgroup columns and windows of as many entries, one bit per row and
    ranked."""
    from paper_2112_10223_amd import binding
    note(f"window_cap=8192 m={m} {dtype.__name__}")
    b = tall_batch(m, 9, [8192, 8191, 8193, 40000, 5000, 100] * 2, dtype, True, seed=m % 97)
    ref = oracle.spkadd(b)
    for force in (-1, 1, 2):
        assert_matches(b, run_gpu(b, binding.make_opts(window_cap=8192, force_bin=force)), ref, exact_values=True)

"""SPKADD_FLAG_ORDERED in the wave kernels: rows that no plan can hold, and terms whose bits
a sum has to keep."""
import numpy as np
import pytest
import torch  # (before the library, which then shares its HIP runtime)

import workloads
from tests.gpu_util import note, to_device

pytestmark = pytest.mark.gpu


def _planned(b, dtype):
    """An ordered plan of b with its symbolic pass done, its inputs and its output arrays (all of
    which the numeric pass may read: the caller keeps every one of them)."""
    from paper_2112_10223_amd import binding
    cps, ris, vas = to_device(b)
    plan = binding.spkadd_plan(b.m, b.n, cps, ris, binding.SPKADD_F64 if dtype == np.float64 else binding.SPKADD_F32,
                               binding.make_opts(flags=binding.SPKADD_FLAG_ORDERED))
    c = torch.empty(b.n + 1, dtype=torch.int32, device="cuda:0")
    nnz = binding.spkadd_symbolic(plan, c)
    r = torch.empty(nnz, dtype=torch.int32, device="cuda:0")
    return plan, cps, ris, vas, c, r, torch.empty(nnz, dtype=vas[0].dtype, device="cuda:0")


@pytest.mark.parametrize("m", [5000, 60000, 1 << 20, (1 << 27) + 1])
@pytest.mark.parametrize("k", [6, 100])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_rows_outside_the_matrix_are_reported(m, k, dtype):
    """Rows overwritten between the passes by some below 0, at m and far above, one and all of a
    column's: every numeric pass ends and the error is reported (plain and ranked bitmap, one
    and two inputs per lane)."""
    from paper_2112_10223_amd import binding
    b = workloads.er(m, 400, k, 500.0 / k, seed=k, values="f64" if dtype == np.float64 else "f32")
    bad = np.array([-1, m, m + 1, m + 8191, 8192 * ((m + 8191) // 8192), (1 << 31) - 1, -(1 << 31)], dtype=np.int64)
    for every in (97, 1):
        note(f"ordered, rows outside the matrix m={m} k={k} {dtype.__name__} every={every}")
        plan, cps, ris, vas, c, r, v = _planned(b, dtype)
        try:
            for i, x in enumerate(ris):
                at = torch.arange(i % 7, x.numel(), every, device="cuda:0")
                x[at] = torch.from_numpy(bad[(np.arange(at.numel()) + i) % bad.shape[0]].astype(np.int32)).to("cuda:0")
            binding.spkadd_numeric(plan, vas, r, v)
            torch.cuda.synchronize()
            with pytest.raises(binding.SpkaddError) as ei:
                binding.spkadd_get_stats(plan)
            assert ei.value.status == binding.SPKADD_ERR_INVALID
        finally:
            plan.free()


@pytest.mark.parametrize("m", [3000, 1 << 20])
@pytest.mark.parametrize("k", [5, 100])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_special_values_keep_their_bits(m, k, dtype):
    """Zeros of both signs, subnormal numbers, infinities, quiet and signalling NaN: a single term
    comes out as it is stored, two equal zeros as that zero, a sum with a NaN as a NaN."""
    from paper_2112_10223_amd import binding
    note(f"ordered, special values m={m} k={k} {dtype.__name__}")
    bits, sign, exp, quiet = (np.uint32, 31, 0xFF << 23, 1 << 22) if dtype == np.float32 else \
        (np.uint64, 63, 0x7FF << 52, 1 << 51)
    special = np.array([0, 1 << sign, 1, (1 << sign) | 5, exp, exp | (1 << sign), exp | quiet | 9, exp | 1,
                        exp | (1 << sign) | 77], dtype=bits)
    ns = special.shape[0]
    # column 0: every special value alone in a row of its own; column 1: each in the first and
    # in the last input; column 2: each added to 1 from another input; the rest empty
    rows, vals, cps = [], [], np.zeros((k, 4), np.int32)
    for i in range(k):
        alone = np.arange(i, ns, k, dtype=np.int32) * 7
        twice = np.arange(ns, dtype=np.int32) * (m // ns) if i in (0, k - 1) else np.zeros(0, np.int32)
        one = np.arange(ns, dtype=np.int32) * 3 if i in (1, 2) else np.zeros(0, np.int32)
        rows.append(np.concatenate([alone, twice, one]))
        v = [special[alone // 7], special[: twice.shape[0]]]
        v.append(special[: one.shape[0]] if i == 1 else np.full(one.shape[0], dtype(1.0)).view(bits))
        vals.append(np.concatenate(v).view(dtype))
        cps[i] = np.cumsum([0, alone.shape[0], twice.shape[0], one.shape[0]])
    b = workloads.CSCBatch(m, 3, cps, rows, vals)
    plan, dcps, ris, vas, c, r, v = _planned(b, dtype)
    try:
        binding.spkadd_numeric(plan, vas, r, v)
        torch.cuda.synchronize()
        binding.spkadd_get_stats(plan)
    finally:
        plan.free()
    assert c.cpu().tolist() == [0, ns, 2 * ns, 3 * ns]
    got = v.cpu().numpy()
    assert np.array_equal(got[:ns].view(bits), special)
    with np.errstate(all="ignore"):
        for part, want in ((got[ns:2 * ns], special.view(dtype) * 2), (got[2 * ns:], special.view(dtype) + dtype(1.0))):
            nan = np.isnan(want)
            assert np.array_equal(np.isnan(part), nan)
            assert np.array_equal(part[~nan].view(bits), want[~nan].view(bits))


@pytest.mark.parametrize("m", [1 << 17, (1 << 17) + 1, 1 << 22, (1 << 31) - 2])
@pytest.mark.parametrize("k,sizes", [(1, [20000]), (9, [6000, 40, 30000]), (40, [5000] * 70)])
def test_row_windows_of_tall_matrices(m, k, sizes):
    """Few long columns, which get more row windows than their entries ask for, and more columns:
    bit-identical to the ordered oracle."""
    import oracle
    from paper_2112_10223_amd import binding
    from tests.gpu_util import run_gpu
    from tests.test_ranked_bitmap import tall_batch
    note(f"ordered row windows m={m} k={k} columns={len(sizes)}")
    b = tall_batch(m, k, sizes, np.float32 if k == 9 else np.float64, False, seed=m % 1000 + k)
    got = run_gpu(b, binding.make_opts(flags=binding.SPKADD_FLAG_ORDERED), stats=True)
    ref = oracle.spkadd_ordered(b)
    assert got[3]["n_window_cols"] > 0
    assert np.array_equal(got[0], ref.colptr) and np.array_equal(got[1], ref.rowidx)
    assert np.array_equal(got[2], ref.val.astype(got[2].dtype))

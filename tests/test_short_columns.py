"""Columns of few entries of very tall matrices: the symbolic pass counts them in hash tables
beside the levels of the ranked bitmap, and unsorted output takes tables in the numeric pass,
against the CPU oracle."""
import numpy as np
import pytest
import torch  # (before the library, which then shares its HIP runtime)

import oracle
import workloads
from tests.gpu_util import assert_matches, note, run_gpu
from tests.test_ranked_bitmap import tall_batch

pytestmark = pytest.mark.gpu


def _sorted_columns(got):
    """The same result with every column's rows ascending."""
    colptr, rows, vals = got[:3]
    col = np.repeat(np.arange(colptr.shape[0] - 1), np.diff(colptr))
    at = np.lexsort((rows, col))
    return colptr, rows[at], vals[at]


# (m of two, three and four levels; each number of entries on both sides of 10, 20, 17, 32 and 29)
@pytest.mark.parametrize("m", [1 << 19, 1 << 20, 1 << 21, 1 << 24, 1 << 27, (1 << 31) - 2])
@pytest.mark.parametrize("k", [1, 3, 40, 64, 65, 100])
def test_around_the_short_columns(m, k):
    from paper_2112_10223_amd import binding
    dtype = np.float64 if (m.bit_length() + k) % 2 else np.float32
    note(f"short columns m={m} k={k} {dtype.__name__}")
    sizes = list(range(0, 66)) * 6 + [100, 300, 700] + [2, 5, 9] * 200
    b = tall_batch(m, k, sizes, dtype, True, seed=m % 1000 + k)
    ref = oracle.spkadd(b)
    assert_matches(b, run_gpu(b), ref, exact_values=True)
    for kw in ({"flags": binding.SPKADD_FLAG_UNSORTED_OUT}, {"flags": binding.SPKADD_FLAG_UNSORTED_OUT, "wave_merge": 1},
               {"flags": binding.SPKADD_FLAG_UNSORTED_OUT, "load_factor_sym": 0.05}):
        assert_matches(b, _sorted_columns(run_gpu(b, binding.make_opts(**kw))), ref, exact_values=True)
    for kw in ({"flags": binding.SPKADD_FLAG_UNSORTED_IN}, {"flags": binding.SPKADD_FLAG_ORDERED},
               {"load_factor_sym": 0.05}):
        assert_matches(b, run_gpu(b, binding.make_opts(**kw)), ref, exact_values=True)


def test_batched_short_columns():
    """Batched requests of very tall matrices with few entries per column, both kinds of launch."""
    from paper_2112_10223_amd import binding
    from tests.gpu_util import to_device
    reqs = [workloads.er(m, 500, k, d, seed=m % 997 + k, values="int32f")
            for m, k, d in ((1 << 20, 3, 2.0), (1 << 21, 8, 2.0), (1 << 24, 4, 5.0), ((1 << 27) + 3, 10, 3.0))]
    for fused in (0, -1):
        note(f"batched short columns batch_fused_cols={fused}")
        bt = binding.Batch(binding.SPKADD_F32, 8, 4000, 400, binding.make_opts(batch_fused_cols=fused))
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

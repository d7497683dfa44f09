"""Workgroup columns whose rows fill every top block of the tallest matrix: the ranked
levels then number 2^31 bits, one more than a signed integer counts."""
import numpy as np
import pytest
import torch  # (before the library, which then shares its HIP runtime)

import oracle
import workloads
from tests.gpu_util import assert_matches, note, run_gpu

M = (1 << 31) - 2


def top_level(cap, span):
    """(shift, blocks) of the top level for units of at most cap entries: lds_layout_bitmap_wg's
    bits (at most 20 per entry over blocks of 32 rows) and bitmap_wg_unit's loop."""
    low, top = (32 * cap + 1023) & ~1023, (20 * cap + 1023) & ~1023
    blocks = (span + 31) // 32
    if blocks <= top:
        top = (blocks + 1023) & ~1023 if span > low else 0
    sh = 0
    if span > low:
        sh = 5
        while (span - 1) >> sh >= top:
            sh += 5
    return sh, ((span - 1) >> sh) + 1


CAPS = {"G1": 2048, "G2": 3072}


def test_the_columns_below_number_2_31_bits():
    for cap in CAPS.values():
        sh, blocks = top_level(cap, M)
        assert blocks <= 2048 <= cap and blocks << sh == 1 << 31


def _column(rng, extra):
    """Sorted rows: one in each block of 2^20 (first, last and other rows of the blocks) and
    some of them again or near, dealt to inputs so that a few rows meet."""
    block = np.arange(2048, dtype=np.int64) << 20
    at = rng.integers(0, 1 << 20, size=2048)
    at[::7], at[3::7] = 0, (1 << 20) - 1
    rows = np.minimum(block + at, M - 1)
    return rows, rng.choice(np.minimum(rows + rng.integers(0, 2, size=2048) * 33, M - 1), size=extra, replace=False)


@pytest.mark.gpu
@pytest.mark.parametrize("bin,n,dtype", [("G1", 3, np.float32), ("G1", 70, np.float64), ("G2", 3, np.float32),
                                         ("G2", 70, np.float64)])
def test_every_top_block(bin, n, dtype):
    """Columns of 2,048 rows, one in each of the 2,048 top blocks (one workgroup of 256 threads)
    and of 3,072 (512 threads; fp32 with fewer than 64 columns, fp64 with more)."""
    note(f"every top block {bin} n={n} {dtype.__name__}")
    rng = np.random.default_rng(n)
    k = 4
    parts = [[] for _ in range(k)]
    cps = np.zeros((k, n + 1), np.int32)
    for j in range(n):
        if j % 17 == 0:
            own, more = _column(rng, CAPS[bin] - 2048)
            deal = rng.integers(0, k - 1, size=own.shape[0])
            rows = [own[deal == i] for i in range(k - 1)] + [np.sort(np.unique(more))]
        else:
            rows = [np.array([j, M - 1 - j], dtype=np.int64)] + [np.zeros(0, np.int64)] * (k - 1)
        for i in range(k):
            parts[i].append(rows[i].astype(np.int32))
            cps[i, j + 1] = cps[i, j] + rows[i].shape[0]
    rows = [np.concatenate(p) for p in parts]
    vals = [rng.integers(-3, 4, size=r.shape[0]).astype(dtype) for r in rows]
    b = workloads.CSCBatch(M, n, cps, rows, vals)
    got = run_gpu(b, stats=True)
    assert got[3]["n_wg_cols"] == (n + 16) // 17
    assert_matches(b, got, oracle.spkadd(b), exact_values=True)

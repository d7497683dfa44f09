"""Sums of more columns than a launch has workgroups for (2^32 work-items): the planning passes
number their blocks over several grid rows, the columns and windows take several launches."""
import pytest
import torch

from tests.gpu_util import note

pytestmark = pytest.mark.gpu

ROW = {threads: (2**32 - 1) // threads for threads in (64, 256)}


@pytest.mark.parametrize("n, k, opts", [
    (ROW[256] + 70, 2, dict(force_bin=2)),               # a window a column
    (ROW[256] + 1, 2, dict(force_bin=2, accum_mode=1)),
    (ROW[256] + 300, 2, dict(force_bin=2, flags=16)),    # (inputs that may be unsorted)
    (ROW[256] + 2, 2, dict(force_bin=1)),                # a workgroup a column
    (ROW[256] + 257, 2, dict(force_bin=1, accum_mode=1)),
    (ROW[64] + 5, 65, dict(accum_mode=1)),               # a wavefront a column
])
def test_many_columns(n, k, opts):
    """Two inputs of one entry a column, in the same row in even columns (the other inputs are
    empty)."""
    from paper_2112_10223_amd import binding as B
    note(f"n={n} k={k} {opts}")
    dev, m = "cuda:0", 64
    j = torch.arange(n, dtype=torch.int32, device=dev)
    colptr, none = torch.arange(n + 1, dtype=torch.int32, device=dev), torch.zeros(n + 1, dtype=torch.int32, device=dev)
    r0, r1 = j % 63, j % 63 + j % 2
    v0, v1 = (j % 1001).float(), (j % 13).float()
    cps = B.PtrArray([colptr] + [none] * (k - 2) + [colptr])
    ris, vas = B.PtrArray([r0] + [r0] * (k - 2) + [r1]), B.PtrArray([v0] + [v0] * (k - 2) + [v1])
    c = torch.empty(n + 1, dtype=torch.int32, device=dev)
    p = B.spkadd_plan(m, n, cps, ris, B.SPKADD_F32, B.make_opts(**opts))
    nnz = B.spkadd_symbolic(p, c)
    r, v = torch.empty(nnz, dtype=torch.int32, device=dev), torch.empty(nnz, device=dev)
    B.spkadd_numeric(p, vas, r, v)
    stats = B.spkadd_get_stats(p)
    assert stats["n_window_cols" if opts.get("force_bin") == 2 else "n_wg_cols" if opts.get("force_bin") else "n_wave_cols"] == n
    p.free()
    odd = j % 2 == 1
    assert nnz == n + n // 2
    assert torch.equal(c[1:] - c[:-1], (1 + j % 2).to(torch.int32)) and int(c[0]) == 0
    at = c[:-1].long()
    assert torch.equal(r[at], r0) and torch.equal(v[at], torch.where(odd, v0, v0 + v1))
    assert torch.equal(r[at[odd] + 1], r1[odd]) and torch.equal(v[at[odd] + 1], v1[odd])

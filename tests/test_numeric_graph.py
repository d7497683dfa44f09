"""spkadd_numeric of a kept plan captured into a HIP graph: every replay, with eager sums and
synchronizations between, gives the eager pass's result for the values then in the inputs."""
import numpy as np
import pytest
import torch  # (before the library, which then shares its HIP runtime)

import oracle
import workloads
from tests.gpu_util import assert_matches, note, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["wave", "ranked", "long", "ordered", "unsorted_out", "unsorted_in"])
def test_captured_numeric_replays(kind):
    from paper_2112_10223_amd import binding
    from tests.test_ranked_bitmap import tall_batch
    note(f"captured numeric {kind}")
    flags = {"ordered": binding.SPKADD_FLAG_ORDERED, "unsorted_out": binding.SPKADD_FLAG_UNSORTED_OUT,
             "unsorted_in": binding.SPKADD_FLAG_UNSORTED_IN}.get(kind, 0)
    if kind == "wave":
        b = workloads.er(3000, 4000, 7, 9.0, seed=3, values="int32f")
    elif kind in ("ranked", "unsorted_out"):
        b = workloads.er((1 << 21) + 5, 3000, 5, 3.0, seed=4, values="int32f")
    else:
        b = tall_batch(1 << 20, 6, [30, 700, 1500, 5000, 9000, 20000] * 12, np.float32, True, seed=5)
    cps, ris, vas = to_device(b)
    plan = binding.spkadd_plan(b.m, b.n, cps, ris, binding.SPKADD_F32, binding.make_opts(flags=flags))
    c = torch.empty(b.n + 1, dtype=torch.int32, device="cuda:0")
    nnz = binding.spkadd_symbolic(plan, c)
    r = torch.zeros(nnz, dtype=torch.int32, device="cuda:0")
    v = torch.zeros(nnz, dtype=torch.float32, device="cuda:0")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, capture_error_mode="relaxed"):
        binding.spkadd_numeric(plan, vas, r, v)
    for scale in (1.0, -3.0, 2.0):
        b2 = workloads.CSCBatch(b.m, b.n, b.colptr, b.rowidx, [x * np.float32(scale) for x in b.vals])
        for t, x in zip(vas, b2.vals):
            t.copy_(torch.from_numpy(x))
        r.zero_()
        v.zero_()
        graph.replay()
        torch.cuda.synchronize()
        binding.spkadd(b.m, cps, ris, vas)  # (eager work between the replays)
        torch.cuda.synchronize()
        rows, vals = r.cpu().numpy(), v.cpu().numpy()
        if kind == "unsorted_out":
            ptr = c.cpu().numpy()
            at = np.lexsort((rows, np.repeat(np.arange(b.n), np.diff(ptr))))
            rows, vals = rows[at], vals[at]
        assert_matches(b2, (c.cpu().numpy().astype(np.int64), rows, vals), oracle.spkadd(b2), exact_values=True)
    del graph
    plan.free()

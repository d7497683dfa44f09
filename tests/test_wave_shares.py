"""Launches of the wave kernels around the sizes where the number of resident wavefronts
changes (one and two units per wavefront of a full chip), against the CPU oracle."""
import pytest
import torch  # (before the library, which then shares its HIP runtime)

import oracle
import workloads
from tests.gpu_util import assert_matches, note, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [4096, 4097, 8192, 8193, 16384, 16385, 24577])
@pytest.mark.parametrize("k,d", [(3, 4.0), (12, 8.0)])
def test_around_the_resident_wavefronts(n, k, d):
    note(f"wave shares n={n} k={k} d={d}")
    b = workloads.er(5000, n, k, d, seed=n + k, values="int32f")
    assert_matches(b, run_gpu(b), oracle.spkadd(b), exact_values=True)

"""Host-side checks of bench.py: the sources a traffic summary belongs to, and the columns of
one workgroup as the library's statistics give them."""
import os
import re
import sys

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2112_10223_amd", "csrc")
sys.path.insert(0, ROOT)


def test_every_included_header_is_a_source():
    """A kernel's sources hold every header of csrc/ that one of them includes."""
    import bench
    for kernel in ("num_wave_e10", "num_window"):
        files = bench.kernel_sources(kernel)
        for fn in files:
            text = open(os.path.join(CSRC, fn)).read()
            for inc in re.findall(r'#include "([^"]+)"', text):
                assert inc in files or not os.path.exists(os.path.join(CSRC, inc)), (kernel, fn, inc)
        assert "wave_device.h" in files and "internal.h" in files
        assert bench.source_sha(kernel) != bench.source_sha("num_wave" if kernel == "num_window" else "num_window")


def test_longest_workgroup_column():
    import bench
    u = np.array([0, 10, 1024, 4096, 4097, 8192, 8193, 20000, 7000])
    assert bench.longest_workgroup_column(u, 4096, 2) == 8192  # (the window columns hold 8193 and 20000)
    assert bench.longest_workgroup_column(u, 4096, 5) == 4096  # (no column above the window capacity)
    assert bench.longest_workgroup_column(u, 3072, 9) == 3072
    names = bench.kernel_of_column(u, 4096, g3_max=8192)
    assert names.tolist()[3:] == ["num_wg512", "num_wg1024", "num_wg1024", "num_window", "num_window", "num_wg1024"]

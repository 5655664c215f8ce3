"""bench.py accepts committed counter summaries only for the kernel sources they were taken with: its list has to hold
every file that the kernels are compiled from."""
import os

import bench


def test_every_kernel_source_is_in_the_hash():
    files = {f for f in os.listdir(bench.CSRC) if f.endswith((".hip", ".h"))}
    assert set(bench.KERNEL_SOURCES) == files - {"api.hip"}
    assert len(bench.KERNEL_SOURCES) == len(set(bench.KERNEL_SOURCES))

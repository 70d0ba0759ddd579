"""The counters that the benchmark takes from committed profiles are tied to the
kernel by a hash of its sources: the hash covers every file it is compiled from."""
import os

import bench
from paper_2509_22684_amd import build


def test_kernel_hash_covers_the_kernels_sources():
    deps = build._deps(os.path.join(build.CSRC, "ntt_mfma_bls.hip"))
    assert sorted(bench.KERNEL_SOURCES) == sorted(os.path.relpath(d, build.ROOT) for d in deps)

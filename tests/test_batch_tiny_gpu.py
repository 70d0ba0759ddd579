"""Batches of many tiny transforms of one plan: one grouped launch of the register
kernels, nothing left to the persistent kernel, bit for bit against the oracle."""
import numpy as np
import pytest

import seeded_inputs as si
from oracle import coracle
from tests.gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("log2n", [2, 5, 6])
def test_64_tiny_transforms_are_one_launch(cuda, log2n):
    import torch

    from paper_2509_22684_amd import Batch, Plan

    field = "bls12_381_fr"
    xs = [si.uniform_field_vector(field, 1 << log2n, si.stream_seed(96, log2n, k)) for k in range(64)]
    bufs = [to_dev(x, cuda) for x in xs]
    batch = Batch([Plan(field, log2n)] * 64, bufs)
    assert batch.items == 0
    batch.launch_eager()
    torch.cuda.synchronize()
    assert batch.status() == 0
    for k, (buf, x) in enumerate(zip(bufs, xs)):
        assert np.array_equal(to_host(buf), coracle.transform(field, "forward", x)), f"2^{log2n} job {k}"

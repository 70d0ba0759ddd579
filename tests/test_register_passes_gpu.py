"""Whole transforms of 2^8 to 2^10 points in launches that fill the chip, which
the register kernels take over from the matrix cores."""
import numpy as np
import pytest

import seeded_inputs as si
from oracle import coracle
from tests.gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("field", ["bls12_381_fr", "bn254_fr", "bls12_377_fr"])
@pytest.mark.parametrize("log2n,log2total", [(8, 21), (9, 21), (10, 20), (10, 19)])
def test_many_whole_transforms(cuda, field, log2n, log2total):
    """2^log2total elements and one job more in one launch (2^19 of 2^10 points
    are still the matrix cores'), eight inputs in turn, against the oracle."""
    import torch

    from paper_2509_22684_amd import Plan, ntt_batch_create_jobs, ntt_batch_destroy, ntt_batch_launch_eager, ntt_batch_status

    n, count = 1 << log2n, (1 << (log2total - log2n)) + 1
    xs = [si.uniform_field_vector(field, n, si.stream_seed(97, log2n, k)) for k in range(7)]
    xs.append(si.boundary_field_vector(field, n, si.stream_seed(98, log2n, 0)))
    plan = Plan(field, log2n, log2_tile=10)
    src = [to_dev(x, cuda) for x in xs]
    out = torch.empty((count, n, 8), dtype=torch.int32, device=cuda)
    for kind in ("forward", "coset_inverse"):
        out.fill_(-1)
        h = ntt_batch_create_jobs([dict(plan=plan, op=kind, out=out[k], work=None, **{"in": src[k % 8]}) for k in range(count)], direct=True)
        ntt_batch_launch_eager(h)
        torch.cuda.synchronize()
        assert ntt_batch_status(h) == 0
        ntt_batch_destroy(h)
        want = [to_dev(coracle.transform(field, kind, x), cuda) for x in xs]
        for k in range(8):
            assert bool((out[k::8] == want[k]).all()), f"{field} 2^{log2n} {kind} input {k}"

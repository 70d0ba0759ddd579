"""GPU parity of matrix-core passes that only launches over several vectors reach:
radix 2^8 with two elements per lane (two 2^17 or four 2^16 transforms, and the
quotient at 2^17; no single transform of 2^18 to 2^20 has such a pass) and radix
2^9 with four (three 2^18 vectors)."""
import numpy as np
import pytest

import seeded_inputs as si
from oracle import coracle
from tests.gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu

FIELDS = ["bls12_381_fr", "bn254_fr", "bls12_377_fr"]


def _vector(field, log2n, seed):
    """Uniform elements, a third of them at the edges of the range."""
    x = si.uniform_field_vector(field, 1 << log2n, si.stream_seed(101, log2n, seed))
    edge = si.boundary_field_vector(field, 1 << 12, si.stream_seed(102, log2n, seed))
    x[1::3] = np.resize(edge, (len(x[1::3]), x.shape[1]))
    return x


@pytest.mark.parametrize("field", FIELDS)
@pytest.mark.parametrize("log2n,count,twiddles", [(16, 4, 1), (17, 2, 1), (17, 2, 2), (18, 3, 1)])
def test_grouped_passes(cuda, field, log2n, count, twiddles):
    import torch

    from paper_2509_22684_amd import Plan, ntt_batch_create_jobs, ntt_batch_destroy, ntt_batch_launch_eager, ntt_batch_status

    plan = Plan(field, log2n, log2_pass_radix=9, twiddle_mode=twiddles)
    xs = [_vector(field, log2n, k) for k in range(count)]
    src = [to_dev(x, cuda) for x in xs]
    for kind in ("forward", "coset_inverse"):
        out = [torch.full_like(s, -1) for s in src]
        h = ntt_batch_create_jobs([dict(plan=plan, op=kind, out=o, work=torch.empty_like(s), **{"in": s})
                                   for s, o in zip(src, out)], direct=True)
        ntt_batch_launch_eager(h)
        torch.cuda.synchronize()
        assert ntt_batch_status(h) == 0
        ntt_batch_destroy(h)
        for k in range(count):
            assert np.array_equal(to_host(out[k]), coracle.transform(field, kind, xs[k])), f"{field} 2^{log2n} {kind} job {k}"


@pytest.mark.parametrize("field", FIELDS)
def test_quotient_2_17(cuda, field):
    from paper_2509_22684_amd import Plan

    xs = [_vector(field, 17, 10 + v) for v in range(3)]
    got = Plan(field, 17).quotient(*(to_dev(x, cuda) for x in xs))
    assert np.array_equal(to_host(got), coracle.quotient(field, *xs))

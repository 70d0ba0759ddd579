"""GPU parity of the matrix-core passes at every radix and tile class.

One element per lane below 2^18 elements in a launch, two up to 2^20, four
from 2^21: each radix 2^3 .. 2^9 in each class (2^9 in the largest class
through a grouped launch), on vectors concentrated at the edges of the range,
bit for bit against the oracle.
"""
import numpy as np
import pytest

import seeded_inputs as si
from oracle import coracle
from tests.gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu

FIELDS = ["bls12_381_fr", "bn254_fr", "bls12_377_fr"]


@pytest.mark.parametrize("field", FIELDS)
@pytest.mark.parametrize("log2n,radix", [(9, 5), (13, 4), (13, 7), (16, 8), (17, 9),
                                         (18, 4), (18, 5), (18, 6), (18, 9), (19, 7), (20, 8),
                                         (21, 4), (21, 5), (21, 6), (21, 7), (22, 8)])
def test_every_radix_in_every_tile_class(cuda, field, log2n, radix):
    from paper_2509_22684_amd import Plan

    x = si.boundary_field_vector(field, 1 << 12, si.stream_seed(91, log2n, radix))
    x = np.tile(x, (max(1, (1 << log2n) >> 12), 1))[: 1 << log2n]
    x[1::3] = si.uniform_field_vector(field, 1 << log2n, si.stream_seed(92, log2n, radix))[1::3]
    plan = Plan(field, log2n, log2_tile=8 if log2n == 9 else 10, log2_pass_radix=radix)
    d = to_dev(x, cuda)
    kinds = ["forward", "coset_inverse"] if log2n > 13 else ["forward", "inverse", "coset_forward", "coset_inverse"]
    for kind in kinds:
        want = coracle.transform(field, kind, x)
        assert np.array_equal(to_host(getattr(plan, kind)(d)), want), f"{field} 2^{log2n} radix 2^{radix} {kind}"


@pytest.mark.parametrize("field", FIELDS)
def test_two_level_twiddles(cuda, field):
    from paper_2509_22684_amd import Plan

    for log2n in (12, 18, 21):
        x = si.uniform_field_vector(field, 1 << log2n, si.stream_seed(93, log2n, 0))
        got = to_host(Plan(field, log2n, twiddle_mode=2).forward(to_dev(x, cuda)))
        assert np.array_equal(got, coracle.transform(field, "forward", x)), f"{field} 2^{log2n}"


def test_grouped_launches_in_the_largest_class(cuda):
    """Sixteen 2^17 transforms as direct pass launches (radix 2^9 and 2^8)."""
    import torch

    from paper_2509_22684_amd import Plan, ntt_batch_create_jobs, ntt_batch_destroy, ntt_batch_launch_eager, ntt_batch_status

    field, log2n = "bn254_fr", 17
    plan = Plan(field, log2n)
    jobs, xs = [], []
    for k in range(16):
        xs.append(si.uniform_field_vector(field, 1 << log2n, si.stream_seed(94, log2n, k)))
        src = to_dev(xs[-1], cuda)
        jobs.append(dict(plan=plan, op="forward", out=torch.empty_like(src), work=torch.empty_like(src), **{"in": src}))
    h = ntt_batch_create_jobs(jobs, direct=True)
    ntt_batch_launch_eager(h)
    torch.cuda.synchronize()
    assert ntt_batch_status(h) == 0
    for k, job in enumerate(jobs):
        assert np.array_equal(to_host(job["out"]), coracle.transform(field, "forward", xs[k])), f"job {k}"
    ntt_batch_destroy(h)


@pytest.mark.parametrize("field", FIELDS)
@pytest.mark.parametrize("log2n,radix,twiddles", [(12, 6, 1), (12, 7, 2), (14, 7, 1), (16, 8, 1), (18, 9, 1), (18, 6, 1),
                                                  (19, 7, 2), (20, 8, 1), (22, 8, 1), (23, 8, 1), (24, 6, 1), (15, 8, 1)])
def test_quotient_bridges(cuda, field, log2n, radix, twiddles):
    """The chain with its transforms bridged, at each bridged radix, tile class
    and number of passes (four at (24, 6)), and one plan without a bridge,
    against the chain's stages run one by one."""
    import torch

    from paper_2509_22684_amd import Plan, quotient_pointwise

    plan = Plan(field, log2n, log2_tile=10, log2_pass_radix=radix, twiddle_mode=twiddles)
    xs = []
    for v in range(3):
        x = si.boundary_field_vector(field, 1 << 12, si.stream_seed(95, log2n, v))
        xs.append(to_dev(np.tile(x, ((1 << log2n) >> 12, 1)), cuda))
        # whole-vector structure, so that no column repeats another
        xs[v] = plan.coset_forward(xs[v])
    h = plan.quotient(*xs)
    a, b, c = (plan.coset_forward(plan.inverse(x)) for x in xs)
    e = torch.empty_like(a)
    quotient_pointwise(plan.handle, a, b, c, e)
    want = plan.coset_inverse(e)
    assert torch.equal(h, want), f"{field} 2^{log2n} radix 2^{radix}"

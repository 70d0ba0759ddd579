"""Pass splits that only plan options reach: 2^9 points with the one-pass limit
below them, and four passes of 2^20 points or more."""
import numpy as np
import pytest

import seeded_inputs as si
from oracle import coracle
from tests.gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("field", ["bls12_381_fr", "bn254_fr", "bls12_377_fr"])
@pytest.mark.parametrize("twiddles", [1, 2])
def test_two_passes_past_the_tile(cuda, field, twiddles):
    from paper_2509_22684_amd import Plan
    from paper_2509_22684_amd._lib import ntt_workspace_bytes

    plan = Plan(field, 9, log2_tile=8, twiddle_mode=twiddles)
    assert plan.passes == 2 and ntt_workspace_bytes(plan.handle) == 32 << 9
    x = si.boundary_field_vector(field, 1 << 9, si.stream_seed(99, 9, twiddles))
    d = to_dev(x, cuda)
    for kind in ("forward", "inverse", "coset_forward", "coset_inverse"):
        assert np.array_equal(to_host(getattr(plan, kind)(d)), coracle.transform(field, kind, x)), f"{field} {kind}"


@pytest.mark.parametrize("field", ["bls12_381_fr", "bn254_fr", "bls12_377_fr"])
@pytest.mark.parametrize("log2n,radix,twiddles", [(20, 6, 1), (20, 6, 2), (22, 7, 1)])
def test_four_passes(cuda, field, log2n, radix, twiddles):
    """6-4-4-6 and 6-6-4-6: a transform against the oracle, the bridged quotient
    against its stages."""
    import torch

    from paper_2509_22684_amd import Plan, quotient_pointwise

    plan = Plan(field, log2n, log2_pass_radix=radix, twiddle_mode=twiddles)
    assert plan.passes == 4
    xs = [si.uniform_field_vector(field, 1 << log2n, si.stream_seed(103, log2n, v)) for v in range(3)]
    xs[0][1::3] = np.resize(si.boundary_field_vector(field, 1 << 12, si.stream_seed(104, log2n, 0)), xs[0][1::3].shape)
    d = [to_dev(x, cuda) for x in xs]
    for kind in ("forward", "coset_inverse"):
        assert np.array_equal(to_host(getattr(plan, kind)(d[0])), coracle.transform(field, kind, xs[0])), f"{field} {kind}"
    a, b, c = (plan.coset_forward(plan.inverse(x)) for x in d)
    e = torch.empty_like(a)
    quotient_pointwise(plan.handle, a, b, c, e)
    assert torch.equal(plan.quotient(*d), plan.coset_inverse(e)), field

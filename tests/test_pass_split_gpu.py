"""2^9 points with the one-pass limit below them: two passes, against the oracle."""
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

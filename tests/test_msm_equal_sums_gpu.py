"""MSM where whole sums meet their equals and their opposites: the doubling and
the cancelling case of the addition that four lanes share, in each step that
uses it (runs' heads per bucket, the large-bucket lists, the bucket tree, the
final sum), with bases that repeat."""
import pytest

import seeded_inputs as si
from oracle import msm_ref as M
from oracle import ref
from tests.gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu

FR = ref.BLS12_381_FR


def _run(points, scal, cuda, window_bits):
    from paper_2509_22684_amd import MsmBases

    bases = MsmBases(to_dev(M.points_to_device_layout(points), cuda), window_bits)
    res = bases.msm(to_dev(si.ints_to_limbs(FR.to_mont(scal)), cuda))
    words = to_host(res)[:48]
    return M.xyzz_to_affine(*(M.fq_from_limbs(words[12 * k:12 * (k + 1)].reshape(1, 12))[0] for k in range(4)))


@pytest.fixture(scope="module")
def points():
    return M.subgroup_point(13), M.subgroup_point(17)


@pytest.mark.parametrize("n,window_bits", [(64, 8), (136, 8), (144, 8), (1024, 8), (5000, 8), (1024, 1)])
def test_copies_of_one_base(cuda, points, n, window_bits):
    """n copies, all scalars 1: every run of the one bucket has the same sum.  At
    c = 8 runs are 8 entries to begin with (136: 17 runs, whose heads one quad adds
    in turn; 144: 18, which go to the list), 16 at 1024 (64 equal heads) and 32 at
    5000."""
    P, _ = points
    assert _run([P] * n, [1] * n, cuda, window_bits) == M.mul(n, P)


@pytest.mark.parametrize("n,window_bits", [(257, 1), (2047, 8), (65535 // 19, 14)])
def test_opposite_runs_cancel(cuda, points, n, window_bits):
    """n copies of P in one histogram group (so in sorted order), n of -P in the
    next: runs of P meet runs of -P, and the sum passes through infinity.  Then
    one more base, which alone is left."""
    P, Q = points
    assert 65535 // (-(-255 // window_bits)) == n
    assert _run([P] * n + [M.neg(P)] * n, [1] * (2 * n), cuda, window_bits) is None
    assert _run([P] * n + [M.neg(P)] * n + [Q], [1] * (2 * n + 1), cuda, window_bits) == Q


@pytest.mark.parametrize("window_bits", [2, 8, 9, 16])
def test_equal_and_opposite_buckets(cuda, points, window_bits):
    """Every bucket P (the tree doubles at every level); neighbours P and -P (each
    node of the first level is infinity)."""
    P, _ = points
    top = min(1 << window_bits, 256)
    scal = list(range(top))
    assert _run([P] * top, scal, cuda, window_bits) == M.mul(sum(scal), P)
    signs = [P if k % 2 == 0 else M.neg(P) for k in range(top)]
    assert _run(signs, scal, cuda, window_bits) == M.mul(FR.p - top // 2, P)


@pytest.mark.parametrize("b", [1, 2, 4, 8, 15])
def test_equal_and_opposite_terms_of_the_final_sum(cuda, points, b):
    """2^b P from bucket 2^b and from bucket 1: equal terms 2^b G_b and G_0, then
    opposite ones."""
    P, Q = points
    R = M.mul(1 << b, P)
    assert _run([P, R], [1 << b, 1], cuda, 16) == M.mul(2 << b, P)
    assert _run([P, M.neg(R)], [1 << b, 1], cuda, 16) is None
    assert _run([P, M.neg(R), Q], [1 << b, 1, 1], cuda, 16) == Q

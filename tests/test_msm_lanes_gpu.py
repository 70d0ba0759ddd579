"""MSM over windows that are small for the number of points: few buckets of many
entries each, where every bucket's sum goes through the large-bucket lists."""
import random

import pytest

import seeded_inputs as si
from oracle import msm_ref as M
from oracle import ref
from tests.gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu

FR = ref.BLS12_381_FR


def run_msm(points, scal, cuda, window_bits):
    from paper_2509_22684_amd import MsmBases

    bases = MsmBases(to_dev(M.points_to_device_layout(points), cuda), window_bits)
    res = bases.msm(to_dev(si.ints_to_limbs(FR.to_mont(scal)), cuda))
    words = to_host(res)[:48]
    X, Y, ZZ, ZZZ = (M.fq_from_limbs(words[12 * k:12 * (k + 1)].reshape(1, 12))[0] for k in range(4))
    return M.xyzz_to_affine(X, Y, ZZ, ZZZ), bases


@pytest.fixture(scope="module")
def multiples_g():
    G = M.subgroup_point(11)
    return G, M.multiples(G, 1 << 14)


@pytest.mark.parametrize("n,window_bits", [(700, 1), (4096, 1), (4096, 3), (511, 6), (1 << 14, 5), (1 << 14, 8)])
def test_small_windows_keep_the_lanes_busy(cuda, multiples_g, n, window_bits):
    """The closed form, and a workspace with the accumulators (two points of 224
    bytes a lane) of at least a lane for every 32 digits, up to 2^15 lanes."""
    G, mults = multiples_g
    rng = random.Random(100 * n + window_bits)
    scal = [rng.randrange(FR.p) for _ in range(n)]
    got, bases = run_msm(mults[:n], scal, cuda, window_bits)
    assert bases.window_bits == window_bits
    assert got == M.mul(sum(s * (i + 1) for i, s in enumerate(scal)) % FR.p, G)
    lanes = min(1 << 15, -(-255 // window_bits) * n // 32)
    ws = bases.workspace()
    assert ws.numel() * ws.element_size() >= 2 * 224 * lanes

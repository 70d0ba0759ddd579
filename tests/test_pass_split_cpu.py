"""The pass split behind the plan options, through the table sizes it leads to
(host only)."""
import pytest

from paper_2509_22684_amd import _lib


def table_bytes(radices):
    """w_R per radix, an inter-pass table for each pass after the first, three
    coset tables, 32 bytes an entry."""
    n = 1 << sum(radices)
    inter = sum(1 << sum(radices[:k + 1]) for k in range(1, len(radices)))
    return 32 * (sum(1 << r for r in set(radices)) + inter + 3 * n)


@pytest.mark.parametrize("log2n,opts,radices", [
    (9, dict(log2_tile=8), [5, 4]),  # log2_tile is the largest transform in one pass
    (9, dict(log2_tile=8, log2_pass_radix=9), [5, 4]),
    (9, dict(log2_tile=10), [9]),
    (8, dict(log2_tile=8), [8]),
    (10, dict(log2_tile=8), [5, 5]),
    (11, dict(log2_tile=10), [6, 5]),
    (11, dict(log2_tile=11), [11]),
    (20, dict(log2_pass_radix=8), [7, 6, 7]),
    (20, dict(log2_pass_radix=6), [6, 4, 4, 6]),
    (21, dict(log2_pass_radix=6), [6, 5, 4, 6]),
    (22, dict(log2_pass_radix=6), [6, 6, 4, 6]),
    (22, dict(log2_pass_radix=7), [6, 6, 4, 6]),
    (23, dict(log2_pass_radix=7), [6, 6, 5, 6]),
    (20, dict(log2_pass_radix=5), [5, 5, 5, 5]),
    (20, dict(log2_pass_radix=6, flags=2), [5, 5, 5, 5]),
])
def test_split(log2n, opts, radices):
    _lib.ntt_tuning_clear()
    assert _lib.ntt_plan_table_bytes("bls12_381_fr", log2n, twiddle_mode=1, **opts) == table_bytes(radices)

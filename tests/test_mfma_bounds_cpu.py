"""Bounds the matrix-core rounds rely on, from the moduli alone.

Each round sums products of signed byte digits: data digits in [-128, 127]
times the digits of w_16^k 2^(8 b) mod p.  Two neighbouring columns are joined
as c_0 + 2^8 c_1 in 32 bits, so 257 times the largest column must stay below
2^31, and the digits themselves must not carry out of the 32nd byte.
"""
import pytest

import seeded_inputs as si
from oracle import ref


def balanced(v):
    out, carry = [], 0
    for i in range(32):
        d = ((v >> (8 * i)) & 255) + carry
        carry = d >= 128
        out.append(d - 256 * carry)
    assert not carry, "carry out of the last digit"
    return out


@pytest.mark.parametrize("field", sorted(si.MODULI))
def test_column_sums_fit(field):
    p, g = si.MODULI[field], ref.FIELDS[field].generator
    w = pow(g, (p - 1) // 16, p)
    mats = [[balanced(pow(w, k, p) * (1 << (8 * b)) % p) for b in range(32)] for k in range(16)]
    row = [[sum(abs(m[b][c]) for b in range(32)) for c in range(32)] for m in mats]
    for rho in (4, 8, 16):
        worst = max(sum(row[i * j * (16 // rho) % 16][c] for j in range(rho)) for i in range(rho) for c in range(32))
        assert 257 * 128 * worst < 1 << 31
    # a pair's sum fits eight limbs and its difference 32 signed digits, with
    # operands below p (BLS12-381 Fr, made canonical first) or 2p (the others)
    top = p if p >> 254 else 2 * p
    assert 2 * top <= 1 << 256
    assert top <= int("7f" * 32, 16)
    assert 1.3 * p < 1 << 256

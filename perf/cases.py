"""Performance cases: the work that a prover asks of this library, through its
public entry points, from a single small transform to the 2^24 quotient chain.

Every case is a dict of plain values.  `listed()` gives the fixed ones,
`draw(rng)` one more of the same ranges, `prepare` what a program holds before
the call (inputs, plan, bases, batch), `run` one pass, `work` the bytes and
operations a pass cannot do without, and `exact` the expected output from
Python integers.
"""
from __future__ import annotations

import functools

import numpy as np
import torch

from paper_2509_22684_amd import MsmBases, Plan
from paper_2509_22684_amd import _lib as zk

# field: (modulus, smallest generator of the multiplicative group)
FIELDS = {
    "bls12_381_fr": (0x73EDA753299D7D483339D80809A1D80553BDA402FFFE5BFEFFFFFFFF00000001, 7),
    "bn254_fr": (0x30644E72E131A029B85045B68181585D2833E84879B9709143E1F593F0000001, 5),
    "bls12_377_fr": (0x12AB655E9A2CA55660B44D1E5C37B00159AA76FED00000010A11800000000001, 22),
}
OPS = ("forward", "inverse", "coset_forward", "coset_inverse")

# BLS12-381 G1, y^2 = x^3 + 4: base field, subgroup order, cofactor, from the curve's seed
_X0 = -0xD201000000010000
_R = _X0 ** 4 - _X0 ** 2 + 1
_Q = (_X0 - 1) ** 2 * _R // 3 + _X0
_H = (_X0 - 1) ** 2 // 3


def listed() -> list:
    return [
        # The smallest call a program makes often: one transform that fits one tile, where
        # the launch and the kernel's latency are all there is.
        {"name": "forward_2e10_bn254", "path": "ntt", "op": "forward", "field": "bn254_fr", "log2n": 10},
        # The small transform of the benchmark (n = 2^12), two passes over few workgroups.
        {"name": "forward_2e12_bls381", "path": "ntt", "op": "forward", "field": "bls12_381_fr", "log2n": 12},
        # A coset transform of a small circuit, an odd power of two.
        {"name": "coset_forward_2e15_bls377", "path": "ntt", "op": "coset_forward", "field": "bls12_377_fr",
         "log2n": 15},
        # An interpolation of a medium circuit: passes of different radix (2^9 and 2^8).
        {"name": "inverse_2e17_bn254", "path": "ntt", "op": "inverse", "field": "bn254_fr", "log2n": 17},
        # The benchmark's medium transform (n = 2^20): one round of workgroups a pass.
        {"name": "forward_2e20_bls381", "path": "ntt", "op": "forward", "field": "bls12_381_fr", "log2n": 20},
        # A large coset interpolation, several rounds of workgroups, uneven passes (8, 7, 7).
        {"name": "coset_inverse_2e22_bls381", "path": "ntt", "op": "coset_inverse", "field": "bls12_381_fr",
         "log2n": 22},
        # The smallest quotient job of the serving mix: seven dependent transforms.
        {"name": "quotient_2e14_bls381", "path": "quotient", "field": "bls12_381_fr", "log2n": 14},
        # A medium quotient job of the serving mix over the other curve.
        {"name": "quotient_2e19_bn254", "path": "quotient", "field": "bn254_fr", "log2n": 19},
        # The headline workload: the Groth16 quotient chain at n = 2^24.
        {"name": "quotient_2e24_bls381", "path": "quotient", "field": "bls12_381_fr", "log2n": 24},
        # Many small transforms of uneven sizes over two fields in one graph launch (log2 n in 10..18).
        {"name": "batch_64_mixed", "path": "batch", "jobs": 64, "lo": 10, "hi": 18, "bn_every": 4},
        # The prover's largest MSM: a quotient's coefficients (uniform scalars) over 2^20 bases.
        {"name": "msm_2e20_uniform", "path": "msm", "n": 1 << 20, "small_share": 0.0},
        # A witness MSM of a ragged size: most scalars of a witness are 0 or 1.
        {"name": "msm_50000_witness", "path": "msm", "n": 50000, "small_share": 0.6},
    ]


def draw(rng) -> dict:
    path = rng.choice(("ntt", "ntt", "ntt", "quotient", "batch", "msm"))
    field = rng.choice(sorted(FIELDS))
    if path == "ntt":
        return {"path": path, "op": rng.choice(OPS), "field": field, "log2n": rng.randint(8, 24)}
    if path == "quotient":
        return {"path": path, "field": field, "log2n": rng.randint(8, 22)}
    if path == "batch":
        lo = rng.randint(6, 12)
        return {"path": path, "jobs": rng.randint(5, 72), "lo": lo, "hi": lo + rng.randint(2, 6),
                "bn_every": rng.randint(2, 6)}
    return {"path": path, "n": int(2.0 ** rng.uniform(8.0, 19.5)) | 1,
            "small_share": rng.choice((0.0, round(rng.uniform(0.3, 0.9), 3)))}


# ---------------------------------------------------------------------------
# Inputs

def _dev() -> torch.device:
    return torch.device("cuda", torch.cuda.current_device())


def _vector(field: str, n: int, gen: torch.Generator) -> torch.Tensor:
    """n random canonical elements: seven uniform limbs under a top limb below the modulus's."""
    x = torch.randint(-(1 << 31), 1 << 31, (n, 8), dtype=torch.int32, device=gen.device, generator=gen)
    x[:, 7] = torch.randint(0, FIELDS[field][0] >> 224, (n,), dtype=torch.int32, device=gen.device, generator=gen)
    return x


def _generator(seed: int) -> torch.Generator:
    return torch.Generator(device=_dev()).manual_seed(seed)


def _batch_jobs(case: dict, seed: int) -> list:
    """(field, log2n) of the batch's jobs; the sizes are the case's, whatever the seed."""
    span = case["hi"] - case["lo"] + 1
    return [("bn254_fr" if k % case["bn_every"] == case["bn_every"] - 1 else "bls12_381_fr",
             case["lo"] + (5 * k + k // span) % span) for k in range(case["jobs"])]


def _scalars(case: dict, seed: int, gen: torch.Generator) -> torch.Tensor:
    """Montgomery scalars over BLS12-381 Fr; a share of them 0 or 1, as in a witness."""
    x = _vector("bls12_381_fr", case["n"], gen)
    if case["small_share"] > 0.0:
        u = torch.rand(case["n"], device=gen.device, generator=gen)
        one = _limbs([(1 << 256) % FIELDS["bls12_381_fr"][0]], 8).to(gen.device)
        x[u < case["small_share"]] = 0
        x[u < 0.5 * case["small_share"]] = one[0]
    return x


def prepare(case: dict, seed: int) -> dict:
    gen = _generator(seed)
    path = case["path"]
    if path == "ntt":
        plan = Plan(case["field"], case["log2n"])
        x = _vector(case["field"], plan.n, gen)
        plan.workspace(x)
        return {"path": path, "op": getattr(plan, case["op"]), "x": x, "out": torch.empty_like(x)}
    if path == "quotient":
        plan = Plan(case["field"], case["log2n"])
        A, B, C = (_vector(case["field"], plan.n, gen) for _ in range(3))
        return {"path": path, "plan": plan, "A": A, "B": B, "C": C, "H": torch.empty_like(A)}
    if path == "batch":
        plans, jobs, outs = {}, [], []
        for field, log2n in _batch_jobs(case, seed):
            if (field, log2n) not in plans:
                plans[field, log2n] = Plan(field, log2n)
            plan = plans[field, log2n]
            x = _vector(field, plan.n, gen)
            nb = zk.ntt_workspace_bytes(plan.handle)
            work = torch.empty(nb // 4, dtype=torch.int32, device=gen.device) if nb else None
            outs.append(torch.empty_like(x))
            jobs.append({"plan": plan, "op": "forward", "in": x, "out": outs[-1], "work": work})
        return {"path": path, "plans": plans, "jobs": jobs, "outs": outs,
                "batch": _BatchHandle(zk.ntt_batch_create_jobs(jobs, graph=True))}
    points = torch.from_numpy(_points(case["n"]).view(np.int32)).to(gen.device)
    bases = MsmBases(points)
    bases.workspace()
    return {"path": path, "bases": bases, "scalars": _scalars(case, seed, gen)}


class _BatchHandle:
    """Owns a batch made from general jobs."""

    def __init__(self, handle: int):
        self.handle = handle

    def __del__(self):
        try:
            zk.ntt_batch_destroy(self.handle)
        except Exception:
            pass


def run(state: dict):
    path = state["path"]
    if path == "ntt":
        return state["op"](state["x"], state["out"])
    if path == "quotient":
        return state["plan"].quotient(state["A"], state["B"], state["C"], state["H"])
    if path == "batch":
        zk.ntt_batch_launch(state["batch"].handle)
        return state["outs"]
    # The library returns XYZZ coordinates, one of many for the point; a prover
    # takes them to the host and divides once, for the proof's affine point.
    v = state["bases"].msm(state["scalars"]).cpu().numpy().view(np.uint32)[:48]
    X, Y, ZZ, ZZZ = (int.from_bytes(v[12 * k:12 * k + 12].tobytes(), "little") for k in range(4))
    if ZZ == 0:
        return torch.zeros(24, dtype=torch.int32)
    inv = pow(ZZ * ZZZ, -1, _Q)
    return _limbs([X * inv * ZZZ % _Q, Y * inv * ZZ % _Q], 12).reshape(24)


def work(case: dict) -> dict:
    """Operations are 32 x 32-bit multiply-adds times two: 2 s^2 + s of them in
    a Montgomery product of s limbs, one product per radix-2 butterfly, ten per
    mixed point addition.  Bytes: 32 an element, each vector once."""
    def transform(n):
        lg = n.bit_length() - 1
        return n // 2 * lg * 136 * 2

    path = case["path"]
    if path == "ntt":
        n = 1 << case["log2n"]
        return {"bytes": 64 * n, "flops": transform(n)}
    if path == "quotient":
        n = 1 << case["log2n"]
        return {"bytes": 4 * 32 * n, "flops": 7 * transform(n) + 2 * n * 136 * 2}
    if path == "batch":
        sizes = [1 << lg for _, lg in _batch_jobs(case, 0)]
        return {"bytes": 64 * sum(sizes), "flops": sum(transform(n) for n in sizes)}
    n = case["n"]
    c = max(4, min(16, n.bit_length() - 3))
    adds = n * (1.0 - case["small_share"]) * ((255 + c - 1) // c) + n * 0.5 * case["small_share"]
    return {"bytes": (32 + 96) * n + 192, "flops": int(adds) * 10 * 300 * 2}


# ---------------------------------------------------------------------------
# Expected outputs, from Python integers

def _ints(x) -> list:
    b = np.ascontiguousarray(x.cpu().numpy()).tobytes()
    w = 4 * x.shape[1]
    return [int.from_bytes(b[k:k + w], "little") for k in range(0, len(b), w)]


def _limbs(vals: list, words: int) -> torch.Tensor:
    b = b"".join(v.to_bytes(4 * words, "little") for v in vals)
    return torch.from_numpy(np.frombuffer(b, dtype=np.int32).copy().reshape(len(vals), words))


def _dft(a: list, w: int, p: int) -> list:
    n = len(a)
    if n == 1:
        return a
    even, odd = _dft(a[0::2], w * w % p, p), _dft(a[1::2], w * w % p, p)
    t, x = [], 1
    for o in odd:
        t.append(o * x % p)
        x = x * w % p
    return [(e + u) % p for e, u in zip(even, t)] + [(e - u) % p for e, u in zip(even, t)]


def _transform(op: str, field: str, a: list) -> list:
    p, g = FIELDS[field]
    n = len(a)
    w = pow(g, (p - 1) // n, p)
    if op in ("inverse", "coset_inverse"):
        w = pow(w, -1, p)
    if op == "coset_forward":
        a = [x * s % p for x, s in zip(a, _powers(g, n, p))]
    out = _dft(a, w, p)
    if op in ("inverse", "coset_inverse"):
        ninv = pow(n, -1, p)
        out = [x * ninv % p for x in out]
    if op == "coset_inverse":
        out = [x * s % p for x, s in zip(out, _powers(pow(g, -1, p), n, p))]
    return out


def _powers(g: int, n: int, p: int) -> list:
    out, x = [], 1
    for _ in range(n):
        out.append(x)
        x = x * g % p
    return out


def exact(case: dict, seed: int):
    """The output of `run` on these inputs; None where plain integers take too long."""
    path = case["path"]
    if path == "ntt":
        if case["log2n"] > 17:
            return None
        x = _ints(_vector(case["field"], 1 << case["log2n"], _generator(seed)))
        return _limbs(_transform(case["op"], case["field"], x), 8)  # linear: Montgomery form in and out
    if path == "quotient":
        if case["log2n"] > 14:
            return None
        field = case["field"]
        p, g = FIELDS[field]
        n = 1 << case["log2n"]
        gen = _generator(seed)
        a, b, c = ([v * pow(1 << 256, -1, p) % p for v in _ints(_vector(field, n, gen))] for _ in range(3))
        ea, eb, ec = (_transform("coset_forward", field, _transform("inverse", field, v)) for v in (a, b, c))
        z = pow(pow(g, n, p) - 1, -1, p)
        h = _transform("coset_inverse", field, [(x * y - u) * z % p for x, y, u in zip(ea, eb, ec)])
        return _limbs([v * (1 << 256) % p for v in h], 8)
    if path == "batch":
        jobs = _batch_jobs(case, seed)
        if sum(1 << lg for _, lg in jobs) > 1 << 18:
            return None
        gen = _generator(seed)
        return [_limbs(_transform("forward", f, _ints(_vector(f, 1 << lg, gen))), 8) for f, lg in jobs]
    r = FIELDS["bls12_381_fr"][0]
    s = _ints(_scalars(case, seed, _generator(seed)))
    k = sum(v * m for v, m in zip(s, map(_multiple, range(len(s))))) * pow(1 << 256, -1, r) % r
    P = _mul(k, _base_point())
    return _limbs(list(P), 12).reshape(24) if P else torch.zeros(24, dtype=torch.int32)


# ---------------------------------------------------------------------------
# MSM bases: a fixed key of distinct subgroup points, P_i = _multiple(i) G

_ROW = 1024


def _multiple(i: int) -> int:
    return (i % _ROW + 1) + ((i // _ROW + 1) << 40)


def _add(P, T):
    if P is None or T is None:
        return P or T
    (x1, y1), (x2, y2) = P, T
    if x1 == x2:
        if (y1 + y2) % _Q == 0:
            return None
        lam = 3 * x1 * x1 * pow(2 * y1, -1, _Q) % _Q
    else:
        lam = (y2 - y1) * pow(x2 - x1, -1, _Q) % _Q
    x3 = (lam * lam - x1 - x2) % _Q
    return x3, (lam * (x1 - x3) - y1) % _Q


def _mul(k: int, P):
    acc = None
    for bit in bin(k)[2:]:
        acc = _add(acc, acc)
        if bit == "1":
            acc = _add(acc, P)
    return acc


@functools.lru_cache(maxsize=None)
def _base_point():
    """A point of the order-r subgroup: the first x from 5 up on the curve, times the cofactor."""
    x = 5
    while pow(x ** 3 + 4, (_Q - 1) // 2, _Q) != 1:
        x += 1
    return _mul(_H, (x, pow(x ** 3 + 4, (_Q + 1) // 4, _Q)))


@functools.lru_cache(maxsize=None)
def _row(b: int) -> np.ndarray:
    """Device limbs of P_i for i in row b: T_a + (b + 1) 2^40 G with T_a = (a + 1) G, one shared inversion."""
    first, step = _first_row()
    x2, y2 = _mul((b + 1) << 40, step)
    pre, acc = [], 1
    for x1, _ in first:
        pre.append(acc)
        acc = acc * (x2 - x1) % _Q
    inv = pow(acc, -1, _Q)
    out = [b""] * _ROW
    for a in range(_ROW - 1, -1, -1):
        x1, y1 = first[a]
        lam = (y2 - y1) * (inv * pre[a] % _Q) % _Q
        inv = inv * (x2 - x1) % _Q
        x3 = (lam * lam - x1 - x2) % _Q
        y3 = (lam * (x1 - x3) - y1) % _Q
        out[a] = ((x3 << 384) % _Q).to_bytes(48, "little") + ((y3 << 384) % _Q).to_bytes(48, "little")
    return np.frombuffer(b"".join(out), dtype=np.uint32).reshape(_ROW, 24)


@functools.lru_cache(maxsize=None)
def _first_row():
    G = _base_point()
    pts = [G]
    while len(pts) < _ROW:
        pts.append(_add(pts[-1], G))
    return pts, G


def _points(n: int) -> np.ndarray:
    rows = [_row(b) for b in range((n + _ROW - 1) // _ROW)]
    return np.ascontiguousarray(np.concatenate(rows)[:n])

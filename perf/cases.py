"""Timing cases of the packed bit-matrix products.

Every case is a plain dict; ``prepare`` makes what a program holds before the call (seeded
operands in HBM, or in page-locked host memory for the out-of-core product, a workspace, a
batched plan), ``run`` is one pass through the public entry points, ``work`` is the traffic
and the bit operations that the product cannot do without, and ``exact`` is the same product
from plain torch float64 matrices.

Bits are drawn as the rest of the repository draws them: GF(2) operands Bernoulli(1/2),
Boolean operands Bernoulli(2^-e) with 2^-e near 1/sqrt(k), so that about 63% of C is set.
As bench.py does, a program loads the shipped autotune table once.
"""
import math
import os

import torch

import paper_1909_01554_amd as bmm

_TABLE = os.path.join(os.path.dirname(os.path.abspath(bmm.__file__)), "tune_gfx950.txt")
_LEAF = {"auto": bmm.LEAF_AUTO, "valu": bmm.LEAF_VALU, "int8": bmm.LEAF_MFMA_I8,
         "fp4": bmm.LEAF_MFMA_F4}
_loaded = False


def _square(kind, semiring, n, **kw):
    return _sized(kind, semiring, n, n, n, **kw)


def _sized(kind, semiring, m, k, n, leaf="auto", b_transposed=False, accumulate=False):
    return {"kind": kind, "semiring": semiring, "m": m, "k": k, "n": n, "leaf": leaf,
            "b_transposed": b_transposed, "accumulate": accumulate}


def listed():
    cases = [
        # the smallest call: one 256-bit block product, launches and latency
        ("gf2_256", _square("cubic", "gf2", 256)),
        # the small plain-method workload (bench.py --mode small)
        ("gf2_2048", _square("cubic", "gf2", 2048)),
        # sizes that divide nothing, B given transposed, a step C |= AB of a closure
        ("bool_ragged_accumulate", _sized("cubic", "bool", 5001, 7003, 3333, b_transposed=True,
                                          accumulate=True)),
        # an ordinary Boolean product on the automatic leaf
        ("bool_16384", _square("cubic", "bool", 16384)),
        # a few hundred words encoded by a large generator matrix: few rows, long k
        ("gf2_encode_256", _sized("cubic", "gf2", 256, 32768, 65536)),
        # the recursion at an ordinary and at a large size, everything automatic
        ("strassen_16384", _square("strassen", "gf2", 16384)),
        ("strassen_65536", _square("strassen", "gf2", 65536)),
        # the leaf that the headline names, in the recursion and in the cubic product
        ("strassen_int8_32768", _square("strassen", "gf2", 32768, leaf="int8")),
        ("bool_int8_32768", _square("cubic", "bool", 32768, leaf="int8")),
        # the other leaf that the headline names
        ("bool_valu_16384", _square("cubic", "bool", 16384, leaf="valu")),
        # uneven independent products through a kept plan (bench.py --mode batched, fewer)
        ("batched_256", {"kind": "batched", "count": 256, "lo": 256, "hi": 8192,
                         "sizes_seed": 3}),
        # host-resident operands streamed through HBM (bench.py --mode ooc, smaller)
        ("ooc_32768", {"kind": "ooc", "semiring": "gf2", "n": 32768, "block": 16384}),
    ]
    out = []
    for name, case in cases:
        case["name"] = name
        out.append(case)
    return out


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: cubic products of any size (odd ones included) on every leaf, the
    recursion on sizes it divides, batches and the out-of-core product."""
    r = rng.random()
    if r < 0.6:
        leaf = rng.choice(["auto", "auto", "auto", "auto", "int8", "valu"])
        top = 20000 if leaf == "auto" else 12000
        m, k, n = (_log_uniform(rng, 200, top) for _ in range(3))
        if rng.random() < 0.15:  # few rows against a large right-hand matrix
            m, k, n = _log_uniform(rng, 64, 600), k * 2, n * 3
        if rng.random() < 0.4:  # whole words
            m, k, n = (max(64, v // 64 * 64) for v in (m, k, n))
        semiring = rng.choice(["gf2", "bool"])
        # accumulation is drawn for OR only: it settles, so a pass can be repeated
        acc = semiring == "bool" and rng.random() < 0.3
        return _sized("cubic", semiring, m, k, n, leaf, rng.random() < 0.3, acc)
    if r < 0.85:
        unit = rng.choice([512, 1024, 2048])
        m, k, n = (unit * rng.randint(max(1, 4096 // unit), 32768 // unit) for _ in range(3))
        return _sized("strassen", "gf2", m, k, n, rng.choice(["auto", "auto", "int8"]),
                      rng.random() < 0.3)
    if r < 0.95:
        return {"kind": "batched", "count": _log_uniform(rng, 16, 300), "lo": 256,
                "hi": rng.choice([1024, 2048, 4096, 8192]),
                "sizes_seed": rng.randrange(1 << 30)}
    return {"kind": "ooc", "semiring": rng.choice(["gf2", "bool"]),
            "n": 64 * rng.randint(64, 400), "block": 64 * rng.choice([64, 128, 256])}


# ---- inputs ----

def _words(bits):
    return (bits + 63) // 64


def _density(semiring, k):
    """Exponent e of the bits' probability 2^-e."""
    return 1 if semiring == "gf2" else max(1, round(math.log2(k) / 2))


def _bits(gen, rows, cols, e):
    """rows x cols packed bits, each set with probability 2^-e; padding bits are zero."""
    x = None
    for _ in range(e):
        w = torch.randint(-(1 << 63), (1 << 63) - 1, (rows, _words(cols)), dtype=torch.int64,
                          device="cuda", generator=gen)
        x = w if x is None else x.bitwise_and_(w)
    if cols % 64:
        x[:, -1] &= (1 << (cols % 64)) - 1
    return x


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _operands(case, gen):
    """A, B (or B^T, which has the same distribution) and, when accumulating, C."""
    m, k, n, e = case["m"], case["k"], case["n"], _density(case["semiring"], case["k"])
    A = _bits(gen, m, k, e)
    B = _bits(gen, n, k, e) if case["b_transposed"] else _bits(gen, k, n, e)
    if case["accumulate"]:
        C = _bits(gen, m, n, 3)
    else:
        C = torch.zeros((m, _words(n)), dtype=torch.int64, device="cuda")
    return A, B, C


def _batch_sizes(case):
    import random
    rng = random.Random(case["sizes_seed"])
    return [tuple(max(64, _log_uniform(rng, case["lo"], case["hi"]) // 64 * 64)
                  for _ in range(3)) for _ in range(case["count"])]


def _batch_operands(case, gen):
    out = []
    for i, (m, k, n) in enumerate(_batch_sizes(case)):
        semiring = "gf2" if i % 2 == 0 else "bool"
        p = {"semiring": semiring, "m": m, "k": k, "n": n, "b_transposed": True,
             "accumulate": False}
        A, B, _ = _operands(p, gen)
        out.append((p, A, B))
    return out


def _ooc_operands(case, gen):
    n, e = case["n"], _density(case["semiring"], case["n"])
    return _bits(gen, n, n, e), _bits(gen, n, n, e)


def _semiring(case):
    return bmm.GF2 if case["semiring"] == "gf2" else bmm.BOOLEAN


def prepare(case, seed):
    global _loaded
    if not _loaded:
        bmm.bmm_autotune_load(_TABLE)
        _loaded = True
    gen = _generator(seed)
    if case["kind"] == "batched":
        problems = []
        # the results lie one after another in one buffer
        out = torch.zeros(sum(m * _words(n) for m, _, n in _batch_sizes(case)),
                          dtype=torch.int64, device="cuda")
        at = 0
        for p, A, B in _batch_operands(case, gen):
            m, n = p["m"], p["n"]
            C = out[at:at + m * _words(n)].view(m, _words(n))
            at += m * _words(n)
            problems.append({"semiring": _semiring(p), "m": m, "k": p["k"], "n": n, "A": A,
                             "B": B, "C": C, "b_transposed": True})
        return {"case": case, "plan": bmm.BatchedPlan(problems), "out": out}
    if case["kind"] == "ooc":
        host = []
        for x in _ooc_operands(case, gen):
            h = torch.empty(x.shape, dtype=torch.int64, pin_memory=True)
            h.copy_(x)
            host.append(h)
        C = torch.zeros((case["n"], _words(case["n"])), dtype=torch.int64, pin_memory=True)
        return {"case": case, "A": host[0], "B": host[1], "C": C}
    A, B, C = _operands(case, gen)
    state = {"case": case, "A": A, "B": B, "C": C,
             "options": bmm.Options(leaf=_LEAF[case["leaf"]])}
    if case["kind"] == "strassen":
        nbytes, _, _ = bmm.bmm_gf2_strassen_workspace(
            case["m"], case["k"], case["n"], -1, state["options"],
            b_transposed=case["b_transposed"])
        state["workspace"] = torch.empty(nbytes // 8 + 1, dtype=torch.int64, device="cuda")
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "batched":
        state["plan"].launch()
        return state["out"]
    if case["kind"] == "ooc":
        n = case["n"]
        bmm.bmm_ooc(_semiring(case), state["A"], state["B"], state["C"], n, n, n,
                    block=case["block"])
        return state["C"]
    m, k, n = case["m"], case["k"], case["n"]
    if case["kind"] == "strassen":
        bmm.bmm_gf2_strassen(state["A"], state["B"], state["C"], m, k, n, state["workspace"],
                             options=state["options"], b_transposed=case["b_transposed"])
    else:
        product = bmm.bmm_gf2 if case["semiring"] == "gf2" else bmm.bmm_boolean
        product(state["A"], state["B"], state["C"], m, k, n, options=state["options"],
                b_transposed=case["b_transposed"], accumulate=case["accumulate"])
    return state["C"]


# ---- the work of a pass ----

def _product_work(m, k, n, accumulate=False):
    nbytes = 8 * (m * _words(k) + k * _words(n) + (2 if accumulate else 1) * m * _words(n))
    return nbytes, 2 * m * k * n


def work(case):
    """One pass: operands read once and C written once (read too when accumulating), and
    2 m k n bit operations, an AND and an addition per term of the cubic sum.  The recursion
    takes 7/8 of them per level, counted down to leaves of 2048 bits."""
    if case["kind"] == "batched":
        parts = [_product_work(*s) for s in _batch_sizes(case)]
        return {"bytes": sum(b for b, _ in parts), "flops": sum(f for _, f in parts)}
    if case["kind"] == "ooc":
        nbytes, flops = _product_work(case["n"], case["n"], case["n"])
        return {"bytes": nbytes, "flops": flops}
    m, k, n = case["m"], case["k"], case["n"]
    nbytes, flops = _product_work(m, k, n, case["accumulate"])
    if case["kind"] == "strassen":
        u = 1
        while (m % (2 * u) == 0 and k % (128 * u) == 0 and n % (128 * u) == 0
               and min(m, k, n) // (2 * u) >= 2048):
            u *= 2
            flops = flops * 7 // 8
    return {"bytes": nbytes, "flops": flops}


# ---- the product in float64 ----

def _unpack(x, cols):
    shifts = torch.arange(64, device=x.device)
    return ((x.unsqueeze(-1) >> shifts) & 1).reshape(x.shape[0], -1)[:, :cols].double()


def _pack(bits):
    rows, cols = bits.shape
    pad = _words(cols) * 64 - cols
    bits = torch.nn.functional.pad(bits.long(), (0, pad)).reshape(rows, -1, 64)
    return (bits << torch.arange(64, device=bits.device)).sum(-1)


def _product(case, A, B, C):
    """The packed product from float64 matrices, 1024 rows of C at a time: the counts are
    whole numbers below 2^53, so their parity and their being zero are exact."""
    k, n = case["k"], case["n"]
    if case["b_transposed"]:
        right = torch.cat([_unpack(B[i:i + 1024], k) for i in range(0, B.shape[0], 1024)]).t()
    else:
        right = torch.cat([_unpack(B[i:i + 1024], n) for i in range(0, B.shape[0], 1024)])
    out = []
    for i in range(0, case["m"], 1024):
        counts = _unpack(A[i:i + 1024], k) @ right
        out.append(_pack(counts % 2 == 1 if case["semiring"] == "gf2" else counts > 0))
    got = torch.cat(out)
    return got | C if case["accumulate"] else got


def exact(case, seed):
    gen = _generator(seed)
    if case["kind"] == "batched":
        if sum(2 * m * k * n for m, k, n in _batch_sizes(case)) > 1 << 44:
            return None
        return torch.cat([_product(p, A, B, None).flatten()
                          for p, A, B in _batch_operands(case, gen)])
    if case["kind"] == "ooc":
        n = case["n"]
        if n > 20000:
            return None
        A, B = _ooc_operands(case, gen)
        p = {"m": n, "k": n, "n": n, "semiring": case["semiring"], "b_transposed": False,
             "accumulate": False}
        return _product(p, A, B, None).cpu()
    m, k, n = case["m"], case["k"], case["n"]
    if max(m * k, k * n, m * n) > 1 << 29 or 2 * m * k * n > 1 << 44:
        return None
    A, B, C = _operands(case, gen)
    return _product(case, A, B, C)

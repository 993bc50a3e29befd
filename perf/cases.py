"""The calls that a program using this library makes, as cases to be timed.

A case names one public call (``op``), the ring and prime chains of its
context, and the call's sizes.  Contexts are built once per parameter set and
shared, as a program keeps them; ciphertexts, plaintexts and keys are uniform
residues (every kernel's work is independent of the values), drawn on the GPU
from the case's seed.

Chains: ``n_q`` ciphertext primes below 2^``q_bits`` and ``n_p`` special
primes below 2^``p_bits``; ``chain`` "windowed" is the 25-30 prime system
(terminal primes of about 25 bits and 30-bit main primes) with ``n_p`` special
primes, whose levels are windows of the prime list.
"""
from __future__ import annotations

import math
import random

import torch

import paper_2407_13055_amd as ck
from paper_2407_13055_amd import primes

_contexts: dict = {}

# Calls on ciphertexts of one level; calls on many ciphertexts (or many
# rotations of one) at once; calls between two windows; calls on plain limbs.
SINGLE = ("hmult_rescale", "hmult", "hrot", "hconj", "keyswitch")
LIGHT = ("rescale", "hadd", "padd", "pmult")
MANY = ("hmult_rescale_batch", "hmult_batch", "hrot_batch", "hrot_hoisted", "hrot_sum_hoisted")
LIMBS = ("ntt_intt", "ntt", "intt", "bconv")
WINDOWED = ("hmult_rescale", "hmult", "hrot", "rescale_rational")


def _case(op, log_n, n_q, n_p, level=0, q_bits=30, p_bits=31, chain="prefix", **more):
    return {"op": op, "chain": chain, "log_n": log_n, "n_q": n_q, "n_p": n_p, "q_bits": q_bits, "p_bits": p_bits,
            "level": level, **more}


def listed():
    top = dict(log_n=16, n_q=24, n_p=8)  # the headline chain: 24 x 30-bit and 8 x 31-bit primes, three digits
    return [
        # the smallest ring with a short chain: a shallow circuit, where the
        # launches and their latency are all there is
        dict(_case("hmult_rescale", 12, 3, 1, level=3, q_bits=28, p_bits=30), name="hmult_rescale_small"),
        # multiplication at the top of the headline chain: the benchmark's own step
        dict(_case("hmult_rescale", level=24, **top), name="hmult_rescale_top"),
        # a rotation half-way down the chain in the serving loop's smaller
        # ring (ragged last digit)
        dict(_case("hrot", 15, 24, 8, level=17, k=-5), name="hrot_mid"),
        # many independent multiplications at uneven levels in one call: throughput
        dict(_case("hmult_rescale_batch", level=24, low=4, count=64, **top), name="hmult_rescale_batch64"),
        # a serving batch: rotations of ciphertexts at uneven levels, each by its own offset and key
        dict(_case("hrot_batch", 15, 24, 8, level=23, low=1, count=13), name="hrot_batch13"),
        # one ciphertext rotated many times: the baby steps of a linear transform
        dict(_case("hrot_hoisted", level=24, count=32, **top), name="hrot_hoisted32"),
        # the inner sum of a linear transform: plaintext-weighted rotations added up
        dict(_case("hrot_sum_hoisted", level=24, count=32, **top), name="hrot_sum32"),
        # multiplication in the 25-30 prime system, merged with its rational rescaling
        dict(_case("hmult_rescale", 16, 15, 4, level=15, chain="windowed"), name="hmult_rescale_window"),
        # rescaling by itself (after a plaintext product or a sum of products)
        dict(_case("rescale", level=24, **top), name="rescale_top"),
        # a polynomial to the evaluation domain and back (encoding, decoding)
        dict(_case("ntt_intt", level=24, **top), name="ntt_intt_24"),
        # base conversion by itself, one digit to the rest of the chain
        dict(_case("bconv", n_in=8, n_out=24, **top), name="bconv_8_24"),
        # a product with a plaintext: one pass over memory
        dict(_case("pmult", level=24, **top), name="pmult_top"),
    ]


def _log_uniform(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case: any of the calls, on any ring degree, chain, level and
    count of the range that the listed cases span."""
    most = max(_cost(c) for c in listed())
    while True:
        op = rng.choice(SINGLE * 2 + MANY + LIGHT + LIMBS + ("window",))
        log_n = rng.randint(12, 16)
        if op == "window":
            levels = [t + m for t, m in primes.LEVELS]
            op = rng.choice(WINDOWED)
            low = 1 if op in ("hmult_rescale", "rescale_rational") else 0  # these need a window below
            case = _case(op, log_n, max(levels), rng.randint(2, 5), level=rng.choice(sorted(levels)[low:]),
                         chain="windowed")
        else:
            n_p = rng.randint(1, 8)
            n_q = rng.randint(max(2, n_p), min(24, 4 * n_p))
            q_bits = rng.choice((28, 29, 30, 30))
            level = _log_uniform(rng, 2, n_q)
            case = _case(op, log_n, n_q, n_p, level=level, q_bits=q_bits, p_bits=rng.randint(max(q_bits + 1, 30), 31))
            if op in MANY:
                case["count"] = _log_uniform(rng, 2, 64 if "batch" in op else 32)
                if "batch" in op:
                    case["low"] = rng.randint(2, level)
            elif op == "bconv":
                case["n_in"], case["n_out"] = rng.randint(1, n_q), rng.randint(1, n_q + n_p)
        if case["op"] == "hrot":
            case["k"] = rng.choice((-1, 1)) * _log_uniform(rng, 1, 1 << (log_n - 2))
        if _cost(case) <= most:
            return case


def _cost(case):
    w = work(case)
    return max(w["bytes"], w["flops"] / 50)


def _chain(case):
    if case["chain"] == "windowed":
        q, ids = primes.context_primes(case["log_n"])
        return q, ck.prime_chain(case["p_bits"], case["log_n"], case["n_p"]), [(w[0], len(w)) for w in ids]
    q = ck.prime_chain(case["q_bits"], case["log_n"], case["n_q"])
    return q, ck.prime_chain(case["p_bits"], case["log_n"], case["n_p"]), None


def _context(case):
    key = tuple(case[k] for k in ("chain", "log_n", "n_q", "n_p", "q_bits", "p_bits"))
    if key not in _contexts:
        _contexts[key] = ck.Context(case["log_n"], *_chain(case))
    return _contexts[key]


def _levels(case):
    """The levels of a batch: spread evenly over [low, level], in a mixed order."""
    n, low, span = case["count"], case["low"], case["level"] - case["low"] + 1
    levels = [low + i * span // n for i in range(n)]
    random.Random(n).shuffle(levels)
    return levels


def prepare(case, seed):
    C = _context(case)
    op, n, level = case["op"], C.n, case["level"]
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    chain = C.q + C.p
    base = 0
    if C.windows is not None:
        base = next(start for start, length in C.windows if length == level)
    mods = chain[base:base + level]

    def residues(moduli, *lead):
        m = torch.tensor(moduli, dtype=torch.int64, device="cuda").view(-1, 1)
        out = torch.empty(*lead, len(moduli), n, dtype=torch.int32, device="cuda")
        for part in out.view(-1, len(moduli), n):
            part.copy_(torch.randint(0, 1 << 62, part.shape, generator=g, device="cuda") % m)
        return out

    def empty(*shape):
        return torch.empty(*shape, n, dtype=torch.int32, device="cuda")

    def offsets(count):  # distinct rotations, both directions
        return [(-1) ** i * (1 + (i * 37) % (n // 2 - 1)) for i in range(count)]

    s = {"op": op, "C": C, "level": level}
    if op in ("hmult_rescale", "hmult"):
        s["a"], s["b"], s["key"] = residues(mods, 2), residues(mods, 2), residues(chain, C.dnum, 2)
        s["out"] = empty(2, C.rescaled_level(level) if op == "hmult_rescale" else level)
    elif op in ("hrot", "hconj"):
        s["a"], s["key"], s["out"], s["k"] = residues(mods, 2), residues(chain, C.dnum, 2), empty(2, level), case.get("k")
    elif op == "keyswitch":
        s["a"], s["key"], s["out"] = residues(mods), residues(chain, C.dnum, 2), (empty(level), empty(level))
    elif op in ("hmult_rescale_batch", "hmult_batch"):
        count = case["count"]
        s["a"], s["b"], s["key"] = residues(mods, count, 2), residues(mods, count, 2), residues(chain, C.dnum, 2)
        # an item below the top level leaves the last rows of its slot as they were
        s["out"] = empty(count, 2, C.rescaled_level(level) if op == "hmult_rescale_batch" else level).zero_()
        s["items"] = C.batch_items(_levels(case))
    elif op == "hrot_batch":
        count = case["count"]
        s["a"], s["key"] = residues(mods, count, 2), residues(chain, min(count, 8), C.dnum, 2)
        s["out"] = empty(count, 2, level).zero_()
        s["items"] = C.batch_items(_levels(case), keys=[i % min(count, 8) for i in range(count)],
                                   rots=[offsets(8)[i % 8] for i in range(count)])
    elif op in ("hrot_hoisted", "hrot_sum_hoisted"):
        count = case["count"]
        s["a"], s["key"] = residues(mods, 2), residues(chain, count, C.dnum, 2)
        s["items"] = C.batch_items([level] * count, keys=list(range(count)), rots=offsets(count))
        if op == "hrot_sum_hoisted":
            s["pt"], s["out"] = residues(chain, count), empty(2, level)
        else:
            s["out"] = empty(count, 2, level)
    elif op == "rescale":
        s["a"], s["out"] = residues(mods, 2), empty(2, level - 1)
    elif op == "rescale_rational":
        below = C.rescaled_level(level)
        start = next(start for start, length in C.windows if length == below)
        s["a"], s["out"] = residues(mods, 2), empty(2, below)
        s["ids"], s["out_ids"] = list(range(base, base + level)), list(range(start, start + below))
    elif op == "hadd":
        s["a"], s["b"], s["out"] = residues(mods, 2), residues(mods, 2), empty(2, level)
    elif op in ("padd", "pmult"):
        s["a"], s["pt"], s["out"] = residues(mods, 2), residues(mods), empty(2, level)
    elif op in ("ntt", "intt", "ntt_intt"):
        s["a"], s["ids"] = residues(mods), list(range(level))
    elif op == "bconv":
        # consecutive primes of the chain to the ones that follow (round the end)
        n_in, n_out = case["n_in"], case["n_out"]
        s["ids"] = list(range(n_in))
        s["out_ids"] = [(n_in + i) % len(chain) for i in range(n_out)]
        s["a"], s["out"] = residues([chain[i] for i in s["ids"]]), empty(n_out)
    else:
        raise ValueError("no call named %r" % op)
    return s


def run(s):
    op, C, level = s["op"], s["C"], s["level"]
    if op == "hmult_rescale":
        C.hmult_rescale(s["a"], s["b"], s["key"], level, s["out"])
    elif op == "hmult":
        C.hmult(s["a"], s["b"], s["key"], level, s["out"])
    elif op == "hrot":
        C.hrot(s["a"], level, s["k"], s["key"], s["out"])
    elif op == "hconj":
        C.hconj(s["a"], level, s["key"], s["out"])
    elif op == "keyswitch":
        C.keyswitch(s["a"], level, s["key"], *s["out"])
    elif op == "hmult_rescale_batch":
        C.hmult_rescale_batch(s["a"], s["b"], s["items"], level, s["key"], s["out"])
    elif op == "hmult_batch":
        C.hmult_batch(s["a"], s["b"], s["items"], level, s["key"], s["out"])
    elif op == "hrot_batch":
        C.hrot_batch(s["a"], s["items"], level, s["key"], s["out"])
    elif op == "hrot_hoisted":
        C.hrot_hoisted(s["a"], level, s["items"], s["key"], s["out"])
    elif op == "hrot_sum_hoisted":
        C.hrot_sum_hoisted(s["a"], level, s["items"], s["key"], s["pt"], s["out"])
    elif op == "rescale":
        C.rescale(s["a"], s["out"])
    elif op == "rescale_rational":
        C.rescale_rational(s["a"], s["ids"], s["out_ids"], s["out"])
    elif op == "hadd":
        C.hadd(s["a"], s["b"], level, s["out"])
    elif op == "padd":
        C.padd(s["a"], s["pt"], level, s["out"])
    elif op == "pmult":
        C.pmult(s["a"], s["pt"], level, s["out"])
    elif op == "bconv":
        C.bconv(s["a"], s["ids"], s["out"], s["out_ids"])
    else:  # the transforms work in place; ntt_intt ends where it began
        if op != "intt":
            C.ntt(s["a"], s["ids"])
        if op != "ntt":
            C.intt(s["a"], s["ids"])
        return s["a"]
    return s["out"]


def exact(case, seed):
    """Every output is a residue, a whole number: there is no rounding to measure."""
    return None


def work(case):
    """Bytes: every input row, key row, plaintext row and output row once.
    flops: integer operations, three per butterfly (a product, a sum, a
    difference) and two per multiply-add, of the transforms, base conversions
    and products that the call consists of."""
    op, level, n_p, log_n = case["op"], case["level"], case["n_p"], case["log_n"]
    n = 1 << log_n
    ntt = 3 * (n // 2) * log_n  # one limb's transform

    def switch(lv):
        """(key rows read, operations) of one key switch at lv limbs."""
        digits, rows = -(-lv // n_p), lv + n_p
        up = digits * rows - lv
        ops = (lv + up + 2 * n_p + 2 * lv) * ntt + 2 * n * (up * n_p + 2 * digits * rows + 2 * n_p * lv)
        return 2 * digits * rows, ops

    limbs, ops = 0, 0
    if op in SINGLE:
        key, ops = switch(level)
        limbs = key + {"hmult_rescale": 4 * level + 2 * (level - 1), "hmult": 6 * level, "hrot": 4 * level,
                       "hconj": 4 * level, "keyswitch": 3 * level}[op]
    elif op in ("hmult_rescale_batch", "hmult_batch", "hrot_batch"):
        for lv in _levels(case):
            limbs += {"hmult_rescale_batch": 6 * lv - 2, "hmult_batch": 6 * lv, "hrot_batch": 4 * lv}[op]
            ops += switch(lv)[1]
        limbs += switch(level)[0] * (min(case["count"], 8) if op == "hrot_batch" else 1)
    elif op in ("hrot_hoisted", "hrot_sum_hoisted"):
        count, rows = case["count"], level + n_p
        key, _ = switch(level)
        digits = -(-level // n_p)
        up, products = (digits * rows) * ntt + 2 * n * (digits * rows - level) * n_p, 4 * n * digits * rows
        down = (2 * n_p + 2 * level) * ntt + 4 * n * n_p * level
        if op == "hrot_hoisted":
            limbs, ops = 2 * level + count * (key + 2 * level), up + count * (products + down)
        else:
            limbs, ops = 4 * level + count * (key + rows), up + count * (products + 4 * n * rows) + down
    elif op in ("rescale", "rescale_rational"):
        below = level - 1 if op == "rescale" else max(t + m for t, m in primes.LEVELS if t + m < level)
        limbs, ops = 2 * level + 2 * below, (2 + 2 * below) * ntt + 4 * n * below
    elif op in ("hadd", "padd", "pmult"):
        limbs, ops = (6 if op == "hadd" else 5) * level, 2 * n * level
    elif op in ("ntt", "intt", "ntt_intt"):
        times = 2 if op == "ntt_intt" else 1
        limbs, ops = 2 * level * times, level * ntt * times
    elif op == "bconv":
        limbs, ops = case["n_in"] + case["n_out"], 2 * n * case["n_in"] * (case["n_out"] + 1)
    return {"bytes": 4 * n * limbs, "flops": ops}

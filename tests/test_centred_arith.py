"""Host checks of the centred arithmetic of the transform kernels (no GPU).

A constant w of a prime q is the centred representative with
ws = round(w 2^32 / q); a product is x w - e q with e = round(x ws / 2^32),
for any signed 32-bit x.  Checked here, in exact integers:

1. ws fits 32 bits, w comes back from ws alone, and the product lies in
   (-3q/4, 3q/4), for primes of every size below 2^31;
2. the forward stages of primes below 2^30 (a centred every other stage)
   never leave signed 32 bits, whatever 32-bit values enter: the bound of
   |values| after each stage, over primes of every ratio to 2^30;
3. KeyMult's 64-bit sums: the bound of a forward value times the quarters
   that the kernel counts stays within what the last reduction takes.
"""
import random

import pytest

import paper_2407_13055_amd as ck

LIM = 1 << 31


def centred(v, q):
    v %= q
    return v if 2 * v < q else v - q


def rnd_div(a, b):
    return (2 * a + b) // (2 * b)  # round to nearest, b > 0


def quot(x, ws):
    return (x * ws + (1 << 31)) >> 32


def pair(w, q):
    w = centred(w, q)
    ws = rnd_div(abs(w) << 32, q)
    return w, ws if w >= 0 else -ws


ODD = [40961, 65537, 786433, (1 << 20) + 7, 33292289, (1 << 28) + 1, (1 << 29) - 3, (1 << 29) + 1,
       954437177, 954437175, 1020054733, (1 << 30) - 1, (1 << 30) + 1, (1 << 30) + (1 << 29) + 1, LIM - 1]


@pytest.mark.parametrize("q", ODD)
def test_products_by_a_centred_constant(q):
    rnd = random.Random(q)
    ws_of = [0, 1, q - 1, (q - 1) // 2, (q + 1) // 2, q // 3] + [rnd.randrange(q) for _ in range(300)]
    xs = [0, 1, -1, LIM - 1, -LIM, q // 2] + [rnd.randrange(-LIM, LIM) for _ in range(100)]
    for w0 in ws_of:
        w, ws = pair(w0, q)
        assert -LIM <= ws < LIM
        assert quot(ws, q) == w
        for x in xs:
            t = x * w - quot(x, ws) * q
            assert 4 * abs(t) < 3 * q and (t - x * w0) % q == 0


def grow(q, x, stages):
    """Largest |value| a stage can leave, stage by stage, from |x| <= x: t is at
    most q/2 + |x| q / 2^33, a centred a at most q/2 + |x| e q / 2^32 with e the
    distance of 2^32 / q from the integer that stands for it."""
    e = abs((1 << 32) / q - rnd_div(1 << 32, q))
    out = []
    for u in range(stages):
        t = q * (0.5 + x / 2**33) + 1
        a = x if u & 1 else q * (0.5 + x * e / 2**32) + 1
        x = a + t
        out.append(x)
    return out


def test_forward_values_stay_in_32_bits():
    # primes just below 2^30, of every distance of 2^32 / q from an integer, and small ones
    worst = 0.0
    for q in [(1 << 30) - 1 - 65536 * i for i in range(1 << 13)] + [(1 << 30) // k for k in range(2, 30000, 7)]:
        for first in (LIM, q):
            g = grow(q, first, 16)
            assert max(g) < LIM
            # passes end after an even number of stages, or after a centring one
            worst = max(worst, max(g[1:]) / LIM)
    assert worst < 0.97
    # KeyMult: three row products (or the own digit, P d0 and two row products)
    # end below 3/2 q 2^32, and the reduction adds q / 2: within (-2q, 2q)
    assert 3 * 0.97 / 2 < 1.5 and 2 * 0.97 / 2 + 0.5 < 1.5


def test_forward_bounds_hold_for_the_benchmark_chain():
    for q in ck.prime_chain(30, 16, 24) + ck.prime_chain(28, 12, 3):
        assert max(grow(q, LIM, 16)) < 0.97 * LIM

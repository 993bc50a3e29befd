"""GPU parity at N = 2^13 with ciphertext and special primes of both classes of
the transform kernels (below and above 2^30) in one chain, among them the ones
where 2^32 / q is farthest from an integer: the general passes under the default
launch shapes, which N = 2^12 does not take.  Digits of 1 and 2 primes (column
passes and conversion in one launch), of 4, and of 8 (whose conversions to
31-bit primes need their range fix); single, batched and hoisted calls,
bit-exact against the oracle."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2407_13055_amd as ck  # noqa: E402

LOG_N = 13
NEAR = [(1 << 30) - 1, 954437177, (1 << 31) - 1, (1 << 29) + 5, 1 << 21, (1 << 30) + (1 << 22), 1020054733, 1 << 25,
        (1 << 31) - (1 << 24), 859000000, (1 << 30) + (1 << 29)]
P_NEAR = [(1 << 31) - (1 << 20), (1 << 30) - (1 << 20), (1 << 30) + (1 << 24), 954400000, (1 << 31) - (1 << 22),
          (1 << 29), (1 << 31) - (1 << 26), (1 << 30) - (1 << 24)]


def near(target, taken):
    """The largest prime at or below target that is 1 mod 2N and not taken."""
    c = (target - 1) // (2 << LOG_N) * (2 << LOG_N) + 1
    while c in taken or not oracle.is_prime(c):
        c -= 2 << LOG_N
    taken.append(c)
    return c


@pytest.fixture(scope="module", params=[1, 2, 4, 8])
def case(request):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n_p = request.param
    taken = []
    q, p = [near(t, taken) for t in NEAR], [near(t, taken) for t in P_NEAR[:n_p]]
    P = oracle.Params(LOG_N, q, p)
    C = ck.Context(LOG_N, q, p)
    st = synth.stream(121, "gpu/prime classes/%d" % n_p)
    ct = [np.stack([st.residues(q, P.n), st.residues(q, P.n)]) for _ in range(2)]
    keys = np.stack([np.stack([np.stack([st.residues(q + p, P.n), st.residues(q + p, P.n)]) for _ in range(P.dnum)])
                     for _ in range(2)])
    pts = np.stack([st.residues(q + p, P.n) for _ in range(2)])
    yield P, C, ct, keys, pts
    C.close()


def empty(P, *lead):
    return torch.full((*lead, P.n), -1, dtype=torch.int32, device="cuda")


@pytest.mark.parametrize("level", [11, 6, 3, 2])
def test_single_calls(case, level):
    P, C, (a, b), keys, _ = case
    key = keys[0]
    print("prime classes: %d special primes, level %d" % (len(P.p), level), flush=True)
    da, db, dk = ck.to_device(a), ck.to_device(b), ck.to_device(key)
    out, rot, rs, one = empty(P, 2, level), empty(P, 2, level), empty(P, 2, level - 1), empty(P, 2, level - 1)
    C.hmult(da, db, dk, level, out)
    C.hmult_rescale(da, db, dk, level, rs)
    C.hrot(da, level, 5, dk, rot)
    ct = np.ascontiguousarray(a[:, :level])
    C.rescale(ck.to_device(ct), one)
    torch.cuda.synchronize()
    prod = oracle.hmult(P, a, b, key, level)
    assert np.array_equal(ck.to_host(out), prod)
    assert np.array_equal(ck.to_host(rs), oracle.rescale(P, prod, level))
    assert np.array_equal(ck.to_host(rot), oracle.hrot(P, a, level, oracle.galois_element(5, LOG_N), key))
    assert np.array_equal(ck.to_host(one), oracle.rescale(P, ct, level))


def test_batched_calls(case):
    P, C, (a, b), keys, _ = case
    levels = [11, 4, 7]
    print("prime classes: %d special primes, batch" % len(P.p), flush=True)
    items = C.batch_items(levels, keys=[0, 1, 0], rots=[3, -8, 1], srcs=[0, 0, 0])
    out, rot = empty(P, 3, 2, 10), empty(P, 3, 2, 11)
    mults = C.batch_items(levels, srcs=[0, 0, 0])  # a multiplication has one key
    C.hmult_rescale_batch(ck.to_device(a[None]), ck.to_device(b[None]), mults, 11, ck.to_device(keys[0]), out)
    C.hrot_batch(ck.to_device(a[None]), items, 11, ck.to_device(keys), rot)
    torch.cuda.synchronize()
    for i, (lv, k, r) in enumerate(zip(levels, [0, 1, 0], [3, -8, 1])):
        want = oracle.rescale(P, oracle.hmult(P, a, b, keys[0], lv), lv)
        assert np.array_equal(ck.to_host(out[i, :, :lv - 1]), want), i
        want = oracle.hrot(P, a, lv, oracle.galois_element(r, LOG_N), keys[k])
        assert np.array_equal(ck.to_host(rot[i, :, :lv]), want), i


def test_hoisted_calls(case):
    P, C, (a, _), keys, pts = case
    level, rots = 9, [7, -2]
    print("prime classes: %d special primes, hoisted" % len(P.p), flush=True)
    items = C.batch_items([level] * 2, keys=[0, 1], rots=rots)
    ct = np.ascontiguousarray(a[:, :level])
    outs, total = empty(P, 2, 2, level), empty(P, 2, level)
    C.hrot_hoisted(ck.to_device(ct), level, items, ck.to_device(keys), outs)
    C.hrot_sum_hoisted(ck.to_device(ct), level, items, ck.to_device(keys), ck.to_device(pts), total)
    torch.cuda.synchronize()
    gs = [oracle.galois_element(r, LOG_N) for r in rots]
    assert np.array_equal(ck.to_host(outs), oracle.hrot_hoisted(P, ct, level, gs, list(keys)))
    assert np.array_equal(ck.to_host(total), oracle.hrot_sum_hoisted(P, ct, level, gs, list(keys), list(pts)))


def test_transforms(case):
    P, C, (a, _), _, _ = case
    ids = list(range(P.n_q))
    x = ck.to_device(a[0])
    C.ntt(x, ids)
    torch.cuda.synchronize()
    assert np.array_equal(ck.to_host(x), oracle.ntt(a[0], P.q, LOG_N))
    C.intt(x, ids)
    torch.cuda.synchronize()
    assert np.array_equal(ck.to_host(x), a[0])

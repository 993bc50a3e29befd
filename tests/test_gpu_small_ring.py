"""GPU parity of the four-launch key switching at N = 2^12 against the oracle,
bit-exact: digit widths 1 to 8 with ragged last digits, every call that
switches keys, and the levels where it can go wrong (one limb, a digit's edge,
the top)."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2407_13055_amd as ck  # noqa: E402

LOG_N = 12


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ck.lib()


def draw(st, mods, n):
    return np.stack([st.residues(mods, n), st.residues(mods, n)])


@pytest.mark.parametrize("n_q,n_p", [(6, 1), (5, 2), (7, 3), (9, 8), (17, 5)])
def test_key_switching(n_q, n_p):
    P = oracle.Params(LOG_N, oracle.prime_chain(30, LOG_N, n_q), oracle.prime_chain(31, LOG_N, n_p))
    C = ck.Context(LOG_N, P.q, P.p)
    st = synth.stream(91, "gpu/small/%d/%d" % (n_q, n_p))
    a, b = draw(st, P.q, P.n), draw(st, P.q, P.n)
    key = np.stack([draw(st, P.q + P.p, P.n) for _ in range(P.dnum)])
    da, db, dk = ck.to_device(a), ck.to_device(b), ck.to_device(key)

    def empty(level):
        return torch.full((2, level, P.n), -1, dtype=torch.int32, device="cuda")

    for level in sorted({1, 2, n_p, min(n_p + 1, n_q), n_q}):
        print("small ring: %d + %d primes, level %d" % (n_q, n_p, level), flush=True)
        prod = oracle.hmult(P, a, b, key, level)
        out, rot, con, ks = empty(level), empty(level), empty(level), empty(level)
        C.hmult(da, db, dk, level, out)
        C.hrot(da, level, 21, dk, rot)
        C.hconj(da, level, dk, con)
        C.keyswitch(ck.to_device(a[1, :level]), level, dk, ks[0], ks[1])
        torch.cuda.synchronize()
        assert np.array_equal(ck.to_host(out), prod)
        assert np.array_equal(ck.to_host(rot), oracle.hrot(P, a, level, oracle.galois_element(21, LOG_N), key))
        assert np.array_equal(ck.to_host(con), oracle.hconj(P, a, level, key))
        assert np.array_equal(ck.to_host(ks), np.stack(oracle.keyswitch(P, a[1, :level], level, key)))
        if level >= 2:
            rs = empty(level - 1)
            C.hmult_rescale(da, db, dk, level, rs)
            torch.cuda.synchronize()
            assert np.array_equal(ck.to_host(rs), oracle.rescale(P, prod, level))
    C.close()


@pytest.mark.parametrize("n_limbs", [1, 9, 131])
def test_transforms(n_limbs):
    """Stand-alone transforms of a limb per work-group, both prime classes, one
    launch and more than one."""
    P = oracle.Params(LOG_N, oracle.prime_chain(30, LOG_N, 6), oracle.prime_chain(31, LOG_N, 3))
    C = ck.Context(LOG_N, P.q, P.p)
    mods = P.q + P.p
    pids = [(5 * i) % len(mods) for i in range(n_limbs)]
    x = synth.stream(92, "gpu/small/ntt/%d" % n_limbs).residues([mods[i] for i in pids], P.n)
    want = oracle.ntt(x, [mods[i] for i in pids], LOG_N)
    d = ck.to_device(x)
    C.ntt(d, pids)
    torch.cuda.synchronize()
    assert np.array_equal(ck.to_host(d), want)
    C.intt(d, pids)
    torch.cuda.synchronize()
    assert np.array_equal(ck.to_host(d), x)
    C.close()


@pytest.mark.parametrize("n_q", [2, 7])
def test_rescale(n_q):
    P = oracle.Params(LOG_N, oracle.prime_chain(30, LOG_N, n_q), oracle.prime_chain(31, LOG_N, 1))
    C = ck.Context(LOG_N, P.q, P.p)
    a = draw(synth.stream(93, "gpu/small/rescale/%d" % n_q), P.q, P.n)
    for level in sorted({2, n_q}):
        out = torch.full((2, level - 1, P.n), -1, dtype=torch.int32, device="cuda")
        C.rescale(ck.to_device(np.ascontiguousarray(a[:, :level])), out)
        torch.cuda.synchronize()
        assert np.array_equal(ck.to_host(out), oracle.rescale(P, np.ascontiguousarray(a[:, :level]), level))
    C.close()

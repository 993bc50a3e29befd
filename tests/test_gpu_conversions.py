"""GPU parity of the base conversions' launch rules against the oracle,
bit-exact: the stand-alone conversion around the size that fits one launch
(512 matrix entries), with ragged groups of targets and targets that are
input primes themselves; key switching with digits of one and two primes and
rescaling at small and odd target counts, whose column passes and conversion
are one launch."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2407_13055_amd as ck  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ck.lib()


@pytest.fixture(scope="module")
def wide():
    q, p = oracle.prime_chain(30, 12, 56), oracle.prime_chain(31, 12, 8)
    C = ck.Context(12, q, p)
    yield C, q + p
    C.close()


@pytest.mark.parametrize("n_in,n_out,first", [(1, 1, 1), (3, 9, 3), (8, 56, 8), (8, 64, 0), (9, 56, 8), (9, 57, 3),
                                              (24, 40, 24), (56, 9, 50), (64, 64, 0)])
def test_bconv_sizes(wide, n_in, n_out, first):
    C, mods = wide
    print("bconv", n_in, "->", n_out, flush=True)
    ins, outs = list(range(n_in)), [(first + i) % 64 for i in range(n_out)]
    x = synth.stream(71, "gpu/conv/%d/%d" % (n_in, n_out)).residues([mods[i] for i in ins], C.n)
    out = torch.empty((n_out, C.n), dtype=torch.int32, device="cuda")
    C.bconv(ck.to_device(x), ins, out, outs)
    torch.cuda.synchronize()
    want = oracle.bconv(x, [mods[i] for i in ins], [mods[i] for i in outs], 12)
    assert np.array_equal(ck.to_host(out), want)


@pytest.mark.parametrize("log_n,n_q,n_p,tpw", [(12, 3, 1, 2), (12, 5, 2, 1), (13, 4, 1, 4), (13, 5, 2, 2)])
def test_narrow_digits(log_n, n_q, n_p, tpw):
    P = oracle.Params(log_n, oracle.prime_chain(30, log_n, n_q), oracle.prime_chain(31, log_n, n_p))
    C = ck.Context(log_n, P.q, P.p)
    C.tune(bconv_tpw_up=tpw, bconv_tpw_down=tpw)
    st = synth.stream(72, "gpu/narrow/%d/%d" % (log_n, n_p))
    a = np.stack([st.residues(P.q, P.n), st.residues(P.q, P.n)])
    b = np.stack([st.residues(P.q, P.n), st.residues(P.q, P.n)])
    key = np.stack([np.stack([st.residues(P.q + P.p, P.n), st.residues(P.q + P.p, P.n)]) for _ in range(P.dnum)])
    da, db, dk = ck.to_device(a), ck.to_device(b), ck.to_device(key)

    def empty(level):
        return torch.empty((2, level, P.n), dtype=torch.int32, device="cuda")

    for level in range(1, n_q + 1):
        print("narrow digits: N = 2^%d, %d + %d primes, level %d" % (log_n, n_q, n_p, level), flush=True)
        prod = oracle.hmult(P, a, b, key, level)
        out = empty(level)
        C.hmult(da, db, dk, level, out)
        torch.cuda.synchronize()
        assert np.array_equal(ck.to_host(out), prod)
        C.hrot(da, level, 9, dk, out)
        torch.cuda.synchronize()
        assert np.array_equal(ck.to_host(out), oracle.hrot(P, a, level, oracle.galois_element(9, log_n), key))
        if level >= 2:
            want = oracle.rescale(P, prod, level)
            rs = empty(level - 1)
            C.hmult_rescale(da, db, dk, level, rs)
            torch.cuda.synchronize()
            assert np.array_equal(ck.to_host(rs), want)
            C.rescale(ck.to_device(prod), rs)
            torch.cuda.synchronize()
            assert np.array_equal(ck.to_host(rs), want)
    C.close()

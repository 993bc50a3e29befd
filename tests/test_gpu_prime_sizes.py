"""GPU parity with primes of every size the library takes, in one context:
just below and above 2^30 (where the transform kernels change class), where
2^32 / q is farthest from an integer, 20 to 29 bits, and special primes of
both classes; four digits, so that KeyMult folds its sums.  Bit-exact against
the oracle, under the default launch shapes and under the 16-residue ones."""
import sys

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2407_13055_amd as ck  # noqa: E402

LOG_N = 12
NEAR = [(1 << 30) - 1, 954437177, (1 << 30) + (1 << 22), (1 << 29) + 5, 1 << 20, (1 << 31) - 1, 1020054733, 1 << 25]
P_NEAR = [(1 << 31) - (1 << 20), (1 << 30) - (1 << 20)]


def near(target, taken):
    """The largest prime at or below target that is 1 mod 2N and not taken."""
    c = (target - 1) // (2 << LOG_N) * (2 << LOG_N) + 1
    while c in taken or not oracle.is_prime(c):
        c -= 2 << LOG_N
    taken.append(c)
    return c


@pytest.fixture(scope="module")
def case():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ck.lib()
    taken = []
    q, p = [near(t, taken) for t in NEAR], [near(t, taken) for t in P_NEAR]
    P = oracle.Params(LOG_N, q, p)
    C = ck.Context(LOG_N, q, p)
    st = synth.stream(61, "gpu/prime sizes")
    ct = [np.stack([st.residues(q, P.n), st.residues(q, P.n)]) for _ in range(2)]
    key = np.stack([np.stack([st.residues(q + p, P.n), st.residues(q + p, P.n)]) for _ in range(P.dnum)])
    yield P, C, ct, key
    C.close()


SHAPES = [{}, dict(rows_per_thread_single=16, keymult_rows_single=16, cols_per_thread_single=16)]


@pytest.mark.parametrize("shape", range(len(SHAPES)))
@pytest.mark.parametrize("level", [8, 5, 2])
def test_key_switching(case, shape, level):
    P, C, (a, b), key = case
    C.tune(**SHAPES[shape])
    print("prime sizes: shape", shape, "level", level, flush=True)
    sys.stdout.flush()
    da, db, dk = ck.to_device(a), ck.to_device(b), ck.to_device(key)
    out = torch.empty((2, level - 1, P.n), dtype=torch.int32, device="cuda")
    C.hmult_rescale(da, db, dk, level, out)
    rot = torch.empty((2, level, P.n), dtype=torch.int32, device="cuda")
    C.hrot(da, level, 3, dk, rot)
    torch.cuda.synchronize()
    want = oracle.rescale(P, oracle.hmult(P, a, b, key, level), level)
    assert np.array_equal(ck.to_host(out), want)
    assert np.array_equal(ck.to_host(rot), oracle.hrot(P, a, level, oracle.galois_element(3, LOG_N), key))


@pytest.mark.parametrize("shape", range(len(SHAPES)))
def test_transforms_and_rescale(case, shape):
    P, C, (a, _), _ = case
    C.tune(**SHAPES[shape])
    ids = list(range(P.n_q))
    x = ck.to_device(a[0])
    C.ntt(x, ids)
    torch.cuda.synchronize()
    assert np.array_equal(ck.to_host(x), oracle.ntt(a[0], P.q, LOG_N))
    C.intt(x, ids)
    torch.cuda.synchronize()
    assert np.array_equal(ck.to_host(x), a[0])
    for level in (8, 6, 3):
        ct = np.ascontiguousarray(a[:, :level])
        out = torch.empty((2, level - 1, P.n), dtype=torch.int32, device="cuda")
        C.rescale(ck.to_device(ct), out)
        torch.cuda.synchronize()
        assert np.array_equal(ck.to_host(out), oracle.rescale(P, ct, level))

"""GPU parity of HMult + rescale with narrow digits on both sides of the size up
to which ModDown's conversion and its column passes are one launch (inputs and
the rescaling's row times groups of targets), bit-exact against the oracle."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2407_13055_amd as ck  # noqa: E402


@pytest.mark.parametrize("log_n,n_p,levels", [(16, 2, (7, 8)), (15, 2, (13, 14)), (16, 1, (11, 12))])
def test_hmult_rescale(log_n, n_p, levels):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    P = oracle.Params(log_n, oracle.prime_chain(30, log_n, max(levels)), oracle.prime_chain(31, log_n, n_p))
    C = ck.Context(log_n, P.q, P.p)
    st = synth.stream(141, "gpu/fused line/%d/%d" % (log_n, n_p))
    a = np.stack([st.residues(P.q, P.n), st.residues(P.q, P.n)])
    b = np.stack([st.residues(P.q, P.n), st.residues(P.q, P.n)])
    key = np.stack([np.stack([st.residues(P.q + P.p, P.n), st.residues(P.q + P.p, P.n)]) for _ in range(P.dnum)])
    da, db, dk = ck.to_device(a), ck.to_device(b), ck.to_device(key)
    for level in levels:
        print("fused line: N = 2^%d, %d special primes, level %d" % (log_n, n_p, level), flush=True)
        out = torch.full((2, level - 1, P.n), -1, dtype=torch.int32, device="cuda")
        C.hmult_rescale(da, db, dk, level, out)
        torch.cuda.synchronize()
        assert np.array_equal(ck.to_host(out), oracle.rescale(P, oracle.hmult(P, a, b, key, level), level))
    C.close()

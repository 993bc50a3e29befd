"""GPU parity of hoisted rotations and of their weighted sum at row counts that
are no multiple of 8, whose last rows are shared by several XCDs: bit-exact
against the oracle, with 1 to 7 rows past the multiple, fewer than 8 rows, and
rotation counts that do not divide evenly among the XCDs."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2407_13055_amd as ck  # noqa: E402


@pytest.mark.parametrize("log_n,n_q,n_p,level,count", [
    (12, 2, 1, 1, 3), (12, 2, 1, 2, 5), (13, 3, 1, 3, 4), (12, 4, 1, 4, 1), (13, 6, 4, 6, 3), (13, 7, 4, 7, 2),
    (12, 9, 4, 9, 2), (14, 7, 2, 4, 3), (13, 12, 5, 10, 2), (12, 5, 4, 5, 7)])
def test_rows_past_a_multiple_of_eight(log_n, n_q, n_p, level, count):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    P = oracle.Params(log_n, oracle.prime_chain(30, log_n, n_q), oracle.prime_chain(31, log_n, n_p))
    C = ck.Context(log_n, P.q, P.p)
    st = synth.stream(101, "gpu/hoisted rows/%d/%d/%d" % (log_n, level, n_p))
    mods = P.q + P.p
    ct = np.stack([st.residues(P.q[:level], P.n) for _ in range(2)])
    keys = np.stack([np.stack([np.stack([st.residues(mods, P.n), st.residues(mods, P.n)]) for _ in range(P.dnum)])
                     for _ in range(count)])
    pts = np.stack([st.residues(mods, P.n) for _ in range(count)])
    rots = [(-1) ** i * (1 + 37 * i) for i in range(count)]
    items = C.batch_items([level] * count, keys=list(range(count)), rots=rots)
    dc, dk = ck.to_device(ct), ck.to_device(keys)
    print("hoisted: N = 2^%d, %d rows, %d rotations" % (log_n, level + n_p, count), flush=True)
    outs = torch.full((count, 2, level, P.n), -1, dtype=torch.int32, device="cuda")
    total = torch.full((2, level, P.n), -1, dtype=torch.int32, device="cuda")
    C.hrot_hoisted(dc, level, items, dk, outs)
    C.hrot_sum_hoisted(dc, level, items, dk, ck.to_device(pts), total)
    torch.cuda.synchronize()
    gs = [oracle.galois_element(k, log_n) for k in rots]
    assert np.array_equal(ck.to_host(outs), oracle.hrot_hoisted(P, ct, level, gs, list(keys)))
    assert np.array_equal(ck.to_host(total), oracle.hrot_sum_hoisted(P, ct, level, gs, list(keys), list(pts)))
    C.close()

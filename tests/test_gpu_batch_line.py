"""GPU parity of batches on both sides of the work-group count from which key
switching's inverse column passes take 16 residues per thread (2816; ModUp's
8-limb launches reach it before or after ModDown's of 10): every item of a batch
that reads one input slot at one level equals the oracle."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2407_13055_amd as ck  # noqa: E402


@pytest.mark.parametrize("log_n,count", [(12, 281), (12, 282), (12, 352), (13, 175), (13, 176), (14, 88), (15, 44)])
def test_items_about_the_line(log_n, count):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    P = oracle.Params(log_n, oracle.prime_chain(30, log_n, 8), oracle.prime_chain(31, log_n, 4))
    C = ck.Context(log_n, P.q, P.p)
    st = synth.stream(131, "gpu/batch line/%d" % log_n)
    a = np.stack([st.residues(P.q, P.n), st.residues(P.q, P.n)])
    b = np.stack([st.residues(P.q, P.n), st.residues(P.q, P.n)])
    key = np.stack([np.stack([st.residues(P.q + P.p, P.n), st.residues(P.q + P.p, P.n)]) for _ in range(P.dnum)])
    da, db, dk = ck.to_device(a[None]), ck.to_device(b[None]), ck.to_device(key)
    level = [8, 5]
    items = C.batch_items([level[i % 2] for i in range(count)], srcs=[0] * count)
    print("batch line: N = 2^%d, %d items" % (log_n, count), flush=True)
    out = torch.zeros((count, 2, 7, P.n), dtype=torch.int32, device="cuda")
    C.hmult_rescale_batch(da, db, items, 8, dk, out)
    torch.cuda.synchronize()
    for i, lv in enumerate(level):
        want = ck.to_device(oracle.rescale(P, oracle.hmult(P, a, b, key, lv), lv))
        assert bool((out[i::2, :, :lv - 1] == want).all())
    C.close()

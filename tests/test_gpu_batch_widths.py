"""GPU parity of large batches, whose inverse column passes take 16 residues
per thread while the conversions that read them keep 4 (and the other way
round): every item of a batch that reads one input slot at one level equals the
oracle, at ring degrees of even and odd column passes and counts on both sides
of the rule."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2407_13055_amd as ck  # noqa: E402


@pytest.mark.parametrize("cols", [4, 16])
@pytest.mark.parametrize("log_n,count", [(12, 100), (12, 256), (13, 129), (14, 70)])
def test_items_of_a_large_batch(log_n, count, cols):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    P = oracle.Params(log_n, oracle.prime_chain(30, log_n, 8), oracle.prime_chain(31, log_n, 4))
    C = ck.Context(log_n, P.q, P.p)
    C.tune(cols_per_thread=cols)
    st = synth.stream(81, "gpu/widths/%d" % log_n)
    a = np.stack([st.residues(P.q, P.n), st.residues(P.q, P.n)])
    b = np.stack([st.residues(P.q, P.n), st.residues(P.q, P.n)])
    key = np.stack([np.stack([st.residues(P.q + P.p, P.n), st.residues(P.q + P.p, P.n)]) for _ in range(P.dnum)])
    da, db, dk = ck.to_device(a[None]), ck.to_device(b[None]), ck.to_device(key)
    level = [8, 5]
    levels = [level[i % 2] for i in range(count)]
    items = C.batch_items(levels, srcs=[0] * count)
    print("batch widths: N = 2^%d, %d items, %d residues" % (log_n, count, cols), flush=True)
    out = torch.zeros((count, 2, 7, P.n), dtype=torch.int32, device="cuda")
    C.hmult_rescale_batch(da, db, items, 8, dk, out)
    torch.cuda.synchronize()
    for i, lv in enumerate(level):
        want = ck.to_device(oracle.rescale(P, oracle.hmult(P, a, b, key, lv), lv))
        assert bool((out[i::2, :, :lv - 1] == want).all())
    C.close()

"""GPU parity of stand-alone transforms on both sides of the limb counts where
the column passes change their width, with primes of both classes, bit-exact
against the oracle and back."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2407_13055_amd as ck  # noqa: E402


@pytest.mark.parametrize("log_n,counts", [(16, (1, 15, 16, 17, 31, 32)), (15, (63, 64, 65)), (14, (129,))])
def test_limb_counts(log_n, counts):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    mods = oracle.prime_chain(30, log_n, 5) + oracle.prime_chain(31, log_n, 2)
    C = ck.Context(log_n, mods[:5], mods[5:])
    few = synth.stream(111, "gpu/ntt widths/%d" % log_n).residues(mods, C.n)
    done = oracle.ntt(few, mods, log_n)
    for count in counts:
        print("ntt: N = 2^%d, %d limbs" % (log_n, count), flush=True)
        ids = [(3 * i) % 7 for i in range(count)]
        x = ck.to_device(few[ids])
        C.ntt(x, ids)
        torch.cuda.synchronize()
        assert np.array_equal(ck.to_host(x), done[ids]), count
        C.intt(x, ids)
        torch.cuda.synchronize()
        assert np.array_equal(ck.to_host(x), few[ids]), count
    C.close()

"""GPU parity of the base conversions' launch rules against the oracle,
bit-exact: the stand-alone conversion around the size that fits one launch
(512 matrix entries), with ragged groups of targets and targets that are
input primes themselves."""
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

"""GPU parity of hoisted rotations on both sides of the key size from which the
keys are loaded past the caches (128 MiB): the same rotations alone, by a call
with few keys, and by a call with many."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import oracle  # noqa: E402
import paper_2407_13055_amd as ck  # noqa: E402


def test_few_and_many_keys():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    log_n, level, count = 14, 9, 40  # 2 digits x 2 x 17 rows of 64 KB: 4.25 MiB a rotation
    q, p = oracle.prime_chain(30, log_n, level), oracle.prime_chain(31, log_n, 8)
    C = ck.Context(log_n, q, p)
    g = torch.Generator(device="cuda")
    g.manual_seed(3)

    def residues(mods, *lead):
        m = torch.tensor(mods, dtype=torch.int64, device="cuda").view(-1, 1)
        return (torch.randint(0, 1 << 62, (*lead, len(mods), C.n), generator=g, device="cuda") % m).to(torch.int32)

    ct, keys = residues(q, 2), residues(q + p, count, C.dnum, 2)
    rots = [(-1) ** i * (1 + 91 * i) for i in range(count)]
    want = torch.empty((count, 2, level, C.n), dtype=torch.int32, device="cuda")
    for i, k in enumerate(rots):
        C.hrot(ct, level, k, keys[i], want[i])
    for n in (count, 31, 30, 1):  # 170, 131.75, 127.5 and 4.25 MiB
        out = torch.full((n, 2, level, C.n), -1, dtype=torch.int32, device="cuda")
        print("hoisted: %d keys" % n, flush=True)
        C.hrot_hoisted(ct, level, C.batch_items([level] * n, keys=list(range(n)), rots=rots[:n]), keys[:n], out)
        assert torch.equal(out, want[:n]), n
    # many rotations by few keys: rotation i by key i mod 3
    for i in range(count):
        C.hrot(ct, level, rots[i], keys[i % 3], want[i])
    out = torch.full_like(want, -1)
    C.hrot_hoisted(ct, level, C.batch_items([level] * count, keys=[i % 3 for i in range(count)], rots=rots), keys[:3], out)
    assert torch.equal(out, want)
    C.close()

"""GPU parity of a hoisted call with more rotations than one grid dimension of
256-thread work-groups can count (2^32 work-items): 32768 rotations at
N = 2^16.  Most items are skipped (no level 0), the first, the last and those
about the middle are rotated and equal the single rotation."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import oracle  # noqa: E402
import paper_2407_13055_amd as ck  # noqa: E402


def test_hoisted_rotations_beyond_one_grid_dimension():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    log_n, count = 16, 1 << 15
    q, p = oracle.prime_chain(30, log_n, 1), oracle.prime_chain(31, log_n, 1)
    C = ck.Context(log_n, q, p)
    need = C.workspace_size(ck.OP_HROT_HOISTED, 1, count) + count * 2 * C.n * 4
    if torch.cuda.mem_get_info()[0] < need + (8 << 30):
        C.close()
        pytest.skip("needs %d GiB of device memory" % (need >> 30))
    g = torch.Generator(device="cuda")
    g.manual_seed(5)

    def residues(mods, *lead):
        m = torch.tensor(mods, dtype=torch.int64, device="cuda").view(-1, 1)
        return (torch.randint(0, 1 << 62, (*lead, len(mods), C.n), generator=g, device="cuda") % m).to(torch.int32)

    ct, keys = residues(q, 2), residues(q + p, 2, C.dnum, 2)
    live = {0: 1, 1: -3, count // 2: 77, count - 2: 4095, count - 1: -1}
    levels, rots = [0] * count, [0] * count
    for i, k in live.items():
        levels[i], rots[i] = 1, k
    items = C.batch_items(levels, keys=[i & 1 for i in range(count)], rots=rots)
    outs = torch.empty((count, 2, 1, C.n), dtype=torch.int32, device="cuda")
    outs[2].fill_(-1)
    ws = torch.empty(C.workspace_size(ck.OP_HROT_HOISTED, 1, count), dtype=torch.uint8, device="cuda")
    print("hoisted: N = 2^16, %d rotations" % count, flush=True)
    C.hrot_hoisted(ct, 1, items, keys, outs, ws=ws)
    want = torch.empty((2, 1, C.n), dtype=torch.int32, device="cuda")
    for i, k in live.items():
        C.hrot(ct, 1, k, keys[i & 1], want)
        assert torch.equal(outs[i], want), i
    assert bool((outs[2] == -1).all())
    del ws, outs
    C.close()
    torch.cuda.empty_cache()

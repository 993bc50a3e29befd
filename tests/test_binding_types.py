"""Buffers of the Python binding are torch tensors (no GPU): an object that only
answers like a device tensor is refused before its address is taken."""
import pytest

torch = pytest.importorskip("torch")
import paper_2407_13055_amd as ck  # noqa: E402


class Like:
    """Answers every question that the binding asks a dense tensor on cuda:0."""
    is_cuda, dtype, device = True, torch.int32, torch.device("cuda:0")

    def __init__(self, *shape):
        self.shape = shape

    def get_device(self):
        return 0

    def is_contiguous(self):
        return True

    def numel(self):
        return 1 << 30

    def dim(self):
        return len(self.shape)

    def data_ptr(self):
        raise AssertionError("the address was taken")


def test_only_torch_tensors_are_buffers():
    C = ck.Context.__new__(ck.Context)
    C.log_n, C.q, C.p, C.windows = 12, list(range(3)), [3], None
    C.device, C.h, C._ws, C._ws_sizes = 0, None, {}, {}
    n = C.n
    for call in (lambda: C._buf(Like(16), "x", 16), lambda: C._ct(Like(2, 3, n), "ct", 3),
                 lambda: C._cts(Like(4, 2, 3, n), "cts", 3), lambda: C._pt(Like(3, n), 3)):
        with pytest.raises(ck.CkksError, match="expected a torch tensor"):
            call()

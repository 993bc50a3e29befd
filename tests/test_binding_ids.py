"""Prime id lists of the Python binding (no GPU): every sequence of integers
reaches the C call as one 32-bit id per element, as many as its length says
(the C side reads that many), whatever the container."""
import array

import numpy as np
import pytest

torch = pytest.importorskip("torch")
import paper_2407_13055_amd as ck  # noqa: E402


@pytest.mark.parametrize("ids", [
    [0, 1, 2, 3, 4], (0, 1, 2, 3, 4), range(5), bytes([0, 1, 2, 3, 4]), bytearray([0, 1, 2, 3, 4]), "01234",
    array.array("b", [0, 1, 2, 3, 4]), np.arange(5), np.arange(5, dtype=np.uint8), np.arange(5.0),
    torch.arange(5), [0.0, 1, np.int64(2), "3", True + 3], memoryview(bytes([0, 1, 2, 3, 4]))], ids=lambda v: type(v).__name__)
def test_one_id_per_element(ids):
    a = ck._ids(ids)
    assert len(a) == len(ids)
    assert list(a) == [0, 1, 2, 3, 4]


def test_lengths_of_byte_strings():
    for n in range(9):
        assert list(ck._ids(bytes(range(n)))) == list(range(n))
    assert len(ck._ids([])) == 0


def test_ids_beyond_32_bits_keep_their_low_word():
    assert list(ck._ids([1, (1 << 32) + 2, -1])) == [1, 2, -1]

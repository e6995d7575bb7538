"""The descriptors of batch calls on the host: counts are taken as a ctypes
field takes them, whatever else they are refused, and each field lands where
falcon_series has it."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")


class _Tensor:
    """What a descriptor reads of a device tensor."""
    is_cuda, device = True, "cuda:0"

    def __init__(self, n, dtype, ptr):
        self.n, self.dtype, self.ptr = n, dtype, ptr

    def is_contiguous(self):
        return True

    def numel(self):
        return self.n

    def data_ptr(self):
        return self.ptr if self.n else 0

    def element_size(self):
        return self.dtype.itemsize


class _Index:
    def __index__(self):
        return 7


def _fields(d):
    from paper_2511_04140_amd import codec as C
    return tuple(getattr(d, f) for f, _ in C.Series._fields_)


def _decompress(counts, n=1):
    from paper_2511_04140_amd import codec as C
    c = C.Codec.__new__(C.Codec)
    d, _ = c._decompress_descs([_Tensor(100, torch.uint8, 64)] * n, counts, [torch.float64] * n,
                               [_Tensor(10, torch.float64, 128)] * n)
    return [_fields(x) for x in d]


@pytest.mark.parametrize("count,n", [
    (5, 5), (True, 1), (np.int32(5), 5), (np.uint64(2**63 + 1), 2**63 + 1), (torch.tensor(5), 5),
    (torch.tensor([5]), 5), (np.array(5), 5), (_Index(), 7), (-1, 2**64 - 1), (2**64 - 1, 2**64 - 1), (2**65 + 3, 3)])
def test_counts_taken(count, n):
    assert _decompress([count]) == [(64, n, 100, 128, 80, 2, 0)]
    assert [f[1] for f in _decompress([1, count, 9], 3)] == [1, n, 9]
    assert [f[1] for f in _decompress({0: count})] == [n]


@pytest.mark.parametrize("count", [5.0, np.float64(5), torch.tensor(5.0), "5", None, np.array([5]), [5]])
def test_counts_refused(count):
    with pytest.raises(TypeError):
        _decompress([count])


def test_a_count_is_missing():
    with pytest.raises(IndexError):
        _decompress([1], 2)


def test_fields_of_a_compression():
    from paper_2511_04140_amd import codec as C
    c = C.Codec.__new__(C.Codec)
    xs = [_Tensor(0, torch.float64, 999), _Tensor(3, torch.float32, 64)]
    d, views = c._compress_descs(xs, [_Tensor(9000 + i, torch.uint8, 256 + i) for i in range(2)])
    assert [_fields(x) for x in d] == [(None, 0, 0, 256, 9000, 2, 0), (64, 3, 0, 257, 9001, 1, 0)]
    assert len(views) == 2
    assert len(c._compress_descs([], None)[0]) == 0 and len(c._decompress_descs([], [], [], None)[0]) == 0

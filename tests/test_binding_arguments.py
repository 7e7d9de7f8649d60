"""What the binding passes to the library, checked without a GPU: tensors are
stood in for by objects with a tensor's address and flags."""
import pytest

from paper_2102_02019_amd import labfm


class DeviceTensor:
    is_cuda = True

    def __init__(self, count, address):
        self.count, self.address = count, address

    def numel(self):
        return self.count

    def is_contiguous(self):
        return True

    def data_ptr(self):
        return self.address


def operators(**kw):
    fields = dict(row_ptr=DeviceTensor(3, 16), col=DeviceTensor(5, 32), w=None, w32=None,
                  kappa=DeviceTensor(2, 48))
    fields.update(kw)
    return labfm.Operators(**fields)


@pytest.mark.parametrize("name", ["row_ptr", "col", "kappa"])
def test_operators_without_a_required_tensor_are_refused(name):
    """The filter reads kappa without a check of its own."""
    with pytest.raises((AttributeError, ValueError)):
        operators(**{name: None})._c()


@pytest.mark.parametrize("part", [0, 1, 2])
def test_tiles_without_a_tensor_are_refused(part):
    tiles = [DeviceTensor(1, 64), DeviceTensor(1024, 80), DeviceTensor(5, 96), 4]
    tiles[part] = None
    with pytest.raises((AttributeError, ValueError)):
        operators(tiles=tuple(tiles))._c()


def test_optional_tensors_become_null_pointers():
    c = operators()._c()
    assert (c.n, c.nnz, c.row_ptr, c.col, c.kappa) == (2, 5, 16, 32, 48)
    assert c.w is None and c.w32 is None and c.mom32 is None and c.wall_normal is None
    c = operators(w=DeviceTensor(30, 64), wall_normal=DeviceTensor(4, 80))._c()
    assert (c.w, c.wall_normal) == (64, 80)


def test_stream_without_the_raw_handle_function(monkeypatch):
    """A torch that lacks its private function for the raw handle gives the
    stream through the public one."""
    torch = labfm.torch

    class Stream:
        cuda_stream = 1234

    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", Stream)
    assert labfm._stream().value == 1234

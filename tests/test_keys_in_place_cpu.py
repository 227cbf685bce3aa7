"""Host-side checks of StridedKeys and PagedKeys on stand-ins for GPU tensors: members exchanged or changed in place between
calls are looked at again, and what a first call would refuse is refused by a later one."""
import math

import pytest
import torch

from paper_2507_08045_amd import binding


class Member:
    """What the binding asks of a layer's tensor."""

    def __init__(self, addr, shape=(2, 4, 64, 128), dtype=torch.bfloat16, cuda=True):
        self.set(addr, shape, dtype, cuda)

    def set(self, addr, shape=(2, 4, 64, 128), dtype=torch.bfloat16, cuda=True, stride=None):
        self.addr, self.shape, self.dtype, self.is_cuda = addr, torch.Size(shape), dtype, cuda
        self._stride = stride or tuple(math.prod(shape[i + 1:]) for i in range(len(shape)))

    def data_ptr(self):
        return self.addr

    def dim(self):
        return len(self.shape)

    def stride(self):
        return self._stride


class Queries(Member):
    device = "cpu"

    def is_contiguous(self):
        return True


@pytest.fixture(params=["strided", "paged"])
def case(request, monkeypatch):
    monkeypatch.setattr(binding, "_stream_ptr", lambda: 7)
    layers = [Member(0x1000 * (i + 1)) for i in range(3)]
    if request.param == "strided":
        keys = binding.StridedKeys(layers)
    else:
        table = Member(0x90000, (2, 8), torch.int32)
        table.is_contiguous = lambda: True
        keys = binding.PagedKeys(layers, table, 30)
    return keys, layers, lambda: binding._keys(Queries(0x80000, (2, 3, 8, 5, 128)), keys, 0.0, 0)


def test_table_stands_while_nothing_changes(case):
    keys, layers, call = case
    call()
    table = keys.table
    assert table.tolist() == [0x1000, 0x2000, 0x3000]
    call()
    assert keys.table is table


def test_members_moved_or_exchanged_get_a_new_table(case):
    keys, layers, call = case
    call()
    layers[2].set(0x7000)
    call()
    assert keys.table.tolist() == [0x1000, 0x2000, 0x7000]
    (keys.k_layers if isinstance(keys, binding.StridedKeys) else keys.pools)[0] = Member(0x5000)
    call()
    assert keys.table.tolist() == [0x5000, 0x2000, 0x7000]


@pytest.mark.parametrize("change", [dict(addr=0xA000, cuda=False), dict(addr=0x2000, shape=(2, 4, 32, 128)),
                                    dict(addr=0x2000, dtype=torch.float16), dict(addr=0), dict(addr=0x2000, shape=(8, 64, 128)),
                                    dict(addr=0x2000, stride=(4 * 64 * 128, 128, 4 * 128, 1))],
                         ids=["left the GPU", "shape", "dtype", "freed", "dim", "stride"])
def test_member_changed_in_place_is_refused(case, change):
    keys, layers, call = case
    call()
    layers[1].set(**change)
    with pytest.raises(ValueError):
        call()
    with pytest.raises(ValueError):   # ... and by the call after that
        call()
    layers[1].set(0x2000)
    call()
    assert keys.table.tolist() == [0x1000, 0x2000, 0x3000]


def test_a_callers_table_is_kept_until_a_member_changes(case):
    keys, layers, call = case
    keys.table = mine = torch.tensor([1, 2, 3])
    call()
    assert keys.table is mine
    layers[0].set(0x9000)
    call()
    assert keys.table.tolist() == [0x9000, 0x2000, 0x3000]

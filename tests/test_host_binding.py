"""What the binding does around a call, with a stand-in for the library and for device tensors (nothing runs)."""
import numpy as np
import pytest
import torch

import paper_1802_06905_amd as cc
from paper_1802_06905_amd import binding


class Tensor:
    """What the binding looks at of a contiguous device tensor."""
    def __init__(self, numel, dtype):
        self.n, self.dtype, self.is_cuda = numel, dtype, True

    def element_size(self):
        return self.dtype.itemsize

    def is_contiguous(self):
        return True

    def numel(self):
        return self.n

    def data_ptr(self):
        return 4096


class Library:
    """Records the calls and answers each with the next of the given statuses (then 0)."""
    def __init__(self, *answers):
        self.answers, self.calls = list(answers), []

    def __getattr__(self, name):
        real = getattr(LIB, name)
        if name.endswith("forward") or name.endswith("forward_sized"):
            def call(*args):
                assert len(args) == len(real.argtypes)
                for value, kind in zip(args, real.argtypes):
                    kind.from_param(value)                    # what ctypes would refuse
                self.calls.append((name, args))
                return self.answers.pop(0) if self.answers else 0
            return call
        return real


LIB = binding._lib
PROBLEM = cc.Problem(2, 3, 4, 5, 6, 3, 3, 1, 1)
POOL = cc.Problem(2, 3, 3, 5, 6, 3, 3, 1, 1)


@pytest.fixture
def library(monkeypatch):
    def install(*answers):
        stand_in = Library(*answers)
        monkeypatch.setattr(binding, "_lib", stand_in)
        monkeypatch.setattr(binding, "_Tensor", Tensor)
        return stand_in
    return install


def conv(dtype, kind=torch.float32):
    binding.cacnn_conv_forward(PROBLEM, dtype, Tensor(7 * 8 * 3 * 2, kind), Tensor(4 * 9 * 3, kind), Tensor(4 * 30 * 2, torch.float32), stream=0)


def pool(dtype, kind=torch.float32):
    binding.cacnn_pool_forward(POOL, dtype, 1, Tensor(7 * 8 * 3 * 2, kind), Tensor(3 * 30 * 2, torch.float32), stream=0)


@pytest.mark.parametrize("call", [conv, pool])
@pytest.mark.parametrize("dtype", [1, 1.0, True, np.int64(1), np.float32(1), np.array(1), torch.tensor(1)], ids=lambda d: type(d).__name__)
def test_dtype_may_be_whatever_int_accepts(library, call, dtype):
    lib = library()
    call(dtype, torch.bfloat16)
    assert len(lib.calls) == 1 and int(lib.calls[0][1][1]) == 1


@pytest.mark.parametrize("call", [conv, pool])
@pytest.mark.parametrize("status", [4, 5])
def test_an_error_of_the_runtime_is_raised_and_nothing_is_enqueued_twice(library, call, status):
    lib = library(status)
    with pytest.raises(cc.CacnnError) as error:
        call(0)
    assert error.value.status == status and len(lib.calls) == 1


@pytest.mark.parametrize("call", [conv, pool])
@pytest.mark.parametrize("status", [2, 3])
def test_an_argument_that_the_library_refuses_is_its_error(library, call, status):
    library(status, status)
    with pytest.raises(cc.CacnnError) as error:
        call(0)
    assert error.value.status == status


def test_the_native_call_leaves_what_it_does_not_take_alone():
    """-1, nothing tried: operands that are not device tensors, a problem that is no Problem, other kinds of numbers and streams."""
    assert binding._native is not None
    t = torch.zeros(4)
    for args in ((PROBLEM, 0, t, t, t, None), (PROBLEM, 0, 1, 2, 3, 0), (tuple(range(9)), 0, t, t, t, 0), (PROBLEM, True, t, t, t, 0),
                 (PROBLEM, 2 ** 70, t, t, t, 0), (PROBLEM, 0, t, t, t, "0"), (PROBLEM, 0, Tensor(4, torch.float32), t, t, 0)):
        assert binding._native.conv(*args) == -1
        assert binding._native.pool(args[0], args[1], 1, *args[3:]) == -1
    assert binding._native.conv() == -1 and binding._native.pool(PROBLEM) == -1

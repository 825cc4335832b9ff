"""The extension that marshals AdamW's tensors takes plain tensors only and leaves everything else to the Python loop (no GPU:
an invalid step number makes the library return before it looks at the device)."""
import ctypes as C

import pytest
import torch
from torch.overrides import TorchFunctionMode

from paper_2502_16982_amd import binding

F, H = torch.float32, torch.bfloat16


@pytest.fixture(scope="module")
def native():
    module = binding._marshal()
    assert module, "the extension is built with the library"
    return module


def status(native, tensors):
    hp = binding.muon_adamw_hparams(1e-3, 0.1, 0.9, 0.95, 1e-8, 0)          # steps count from 1
    return native.step(tensors, C.addressof(hp), 0)


def quad(p=F, g=F, m=F, v=F, shape=(6,)):
    return tuple(torch.zeros(shape, dtype=d) for d in (p, g, m, v))


class Sub(torch.Tensor):
    pass


class Mode(TorchFunctionMode):
    def __torch_function__(self, func, types, args=(), kwargs=None):
        return func(*args, **(kwargs or {}))


@pytest.mark.parametrize("tensors", [
    [], [quad()], [quad(H, H)], [quad(F, H)], [quad(H, F)], [quad(shape=()), quad(H, H, shape=(3, 5))],
    [(torch.nn.Parameter(torch.zeros(6)),) + quad()[1:]],
    [tuple(t[2:8] for t in quad(shape=(20,)))],
    [(torch.zeros(2, 3), torch.zeros(6), torch.zeros(3, 2), torch.zeros(6))],
])
def test_plain_tensors_reach_the_library(native, tensors):
    assert status(native, tensors) == -1                                     # MUON_E_INVALID_ARG, from the step number
    with pytest.raises(binding.MuonError):
        binding.muon_adamw_step(tensors, lr=1e-3, weight_decay=0.1, step=0)


@pytest.mark.parametrize("tensors,error", [
    ([quad()[:3]], ValueError),
    ([quad(torch.float16)], binding.MuonError),
    ([quad(m=H)], binding.MuonError),
    ([quad(), quad()[:3] + (torch.zeros(7),)], binding.MuonError),
    ([(torch.zeros(4, 3).t(),) + quad(shape=(3, 4))[1:]], binding.MuonError),
    ([(1, 2, 3, 4)], AttributeError),
])
def test_what_is_refused_is_refused_by_the_loop(native, tensors, error):
    assert status(native, tensors) is None
    with pytest.raises(error):
        binding.muon_adamw_step(tensors, lr=1e-3, weight_decay=0.1, step=0)


def test_subclasses_and_modes_are_left_to_the_loop(native):
    assert status(native, [(torch.zeros(6).as_subclass(Sub),) + quad()[1:]]) is None
    with Mode():
        assert status(native, [quad()]) is None
    assert status(native, [quad()]) == -1

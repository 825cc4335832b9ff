"""The extension that marshals AdamW's tensors takes plain tensors only and leaves everything else to the Python loop (no GPU:
an invalid step number makes the library return before it looks at the device); the library is built with or without it."""
import ctypes as C
import os

import pytest
import torch
from torch.overrides import TorchFunctionMode

import paper_2502_16982_amd
from paper_2502_16982_amd import binding, build

F, H = torch.float32, torch.bfloat16
REAL_RUN = build._run


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


def test_a_default_device_is_no_reason_for_the_loop(native):
    """torch.set_default_device and `with torch.device(..)` are function modes too, of a kind that only changes factory calls."""
    from torch.utils._device import DeviceContext

    class Louder(DeviceContext):
        pass

    tensors = [quad()]
    with torch.device("cpu"):
        assert status(native, tensors) == -1
        with Mode():
            assert status(native, tensors) is None
    with Louder(torch.device("cpu")):
        assert status(native, tensors) is None
    with Mode(), torch.device("cpu"):
        assert status(native, tensors) is None
    torch.set_default_device("cpu")
    try:
        assert status(native, tensors) == -1
    finally:
        torch.set_default_device(None)
    assert status(native, tensors) == -1


@pytest.fixture
def tree(tmp_path, monkeypatch):
    """build.py pointed at an empty folder; compilers replaced by a record of what was run, which leaves the output file."""
    ran = []

    def run(cmd, verbose):
        ran.append(cmd)
        out = cmd[cmd.index("-o") + 1]
        with open(out, "w") as f:
            f.write(cmd[0])

    monkeypatch.setattr(build, "PKG_DIR", str(tmp_path))
    monkeypatch.setattr(build, "OBJ_DIR", str(tmp_path / "_build"))
    monkeypatch.setattr(build, "LIB_PATH", str(tmp_path / build.LIB_NAME))
    monkeypatch.setattr(build, "MARSHAL_PATH", str(tmp_path / "_adamw_marshal.so"))
    monkeypatch.setattr(build, "_run", run)
    return ran


def without_headers(out):
    raise ImportError("no torch here")


def without_compiler(out):
    return ["/nowhere/g++", "-o", out]


@pytest.mark.parametrize("command,reason", [(without_headers, "ImportError: no torch here"), (without_compiler, "FileNotFoundError"),
                                            (lambda out: ["false", "-o", out], "false failed")])
def test_library_is_built_without_the_extension(tree, monkeypatch, capsys, command, reason):
    """hipcc alone makes the library; what the optional extension lacks is said, under its own name."""
    recorded = build._run
    monkeypatch.setattr(build, "marshal_command", command)

    def run(cmd, verbose):
        if os.path.basename(cmd[0]) == "hipcc":
            return recorded(cmd, verbose)
        return REAL_RUN(cmd, verbose)

    monkeypatch.setattr(build, "_run", run)
    assert build.build_library() == build.LIB_PATH and os.path.exists(build.LIB_PATH)
    assert not os.path.exists(build.MARSHAL_PATH) and not os.path.exists(build.MARSHAL_PATH + ".tmp")
    err = capsys.readouterr().err
    assert "_adamw_marshal.so was not built" in err and reason in err and "hipcc" not in err


def test_an_older_extension_goes_before_the_library_changes(tree, monkeypatch):
    """One that an earlier build left, of another record layout maybe, is not there beside the new library, even where no new
    one can be built."""
    open(build.MARSHAL_PATH, "w").write("old")
    open(build.LIB_PATH, "w").write("old")
    replace = os.replace

    def watched(src, dst):
        assert dst != build.LIB_PATH or not os.path.exists(build.MARSHAL_PATH)
        return replace(src, dst)

    monkeypatch.setattr(build.os, "replace", watched)
    monkeypatch.setattr(build, "marshal_command", without_headers)
    build.build_library()
    assert open(build.LIB_PATH).read() != "old" and not os.path.exists(build.MARSHAL_PATH)


SIZES = (C.sizeof(binding.muon_adamw_param), C.sizeof(binding.muon_adamw_hparams))


@pytest.mark.parametrize("marks,used", [
    ({"built_for": build.marshal_stamp(), "record_sizes": SIZES}, True),
    ({"built_for": build.marshal_stamp().replace("torch ", "torch 9."), "record_sizes": SIZES}, False),
    ({"built_for": build.marshal_stamp().replace("python ", "python 9."), "record_sizes": SIZES}, False),
    ({"built_for": build.marshal_stamp(), "record_sizes": (SIZES[0] + 8, SIZES[1])}, False),
    ({"built_for": build.marshal_stamp(), "record_sizes": (SIZES[0], SIZES[1] - 8)}, False),
    ({}, False)])
def test_an_extension_of_another_torch_or_library_is_not_used(monkeypatch, marks, used):
    class Extension:
        def step(*args):
            raise AssertionError("called")
    for name, value in marks.items():
        setattr(Extension, name, value)
    monkeypatch.setattr(paper_2502_16982_amd, "_adamw_marshal", Extension, raising=False)
    monkeypatch.setattr(binding, "_MARSHAL", None)
    assert (binding._marshal() is Extension) == used and (used or binding._marshal() is False)
    if not used:                                 # the loop does its work
        with pytest.raises(binding.MuonError):
            binding.muon_adamw_step([quad()], lr=1e-3, weight_decay=0.1, step=0)


def test_the_built_extension_is_the_one_for_this_torch(native):
    assert native.built_for == build.marshal_stamp() and native.record_sizes == SIZES

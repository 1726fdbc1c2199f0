"""The native call module against the library that is loaded: which module is taken, when it is built again, and what the binding's
functions pass on."""
import os
import types

import pytest
import torch

from paper_2502_17421_amd import binding as ls
from paper_2502_17421_amd import build as ls_build
from test_call_module import calls  # noqa: F401  (fixture)
from test_call_routes import KT, K, LENS, LSE, OUT, PARENTS, Q, V, VT, WORK, desc, lib  # noqa: F401  (lib: fixture)


def test_a_module_that_does_not_fit_is_left_alone(lib, tmp_path, monkeypatch):  # noqa: F811
    """One that does not load, one for another header, torch or Python, and one older than these: ctypes, and a warning."""
    ls_build.build_call_module(force=False)
    for name in ls._DEVICE_CALLS:
        getattr(lib, name).argtypes = getattr(ls.lib(), name).argtypes
    x = desc(8, 2, 128, 8, 300)
    args = [x, Q, K, V, LENS, KT, VT, PARENTS, OUT, LSE, WORK, 1 << 40, None]
    with open(ls.CALL_PATH, "rb") as f:
        image = f.read()
    for i, (old, new) in enumerate(((image, b"no module"), (ls_build.interface_id().encode(), b"0" * 16),
                                    (torch.__version__.encode() + b"\0", b"0" * len(torch.__version__) + b"\0"),
                                    (b"python_version", b"python_versiox"))):
        assert old in image
        path = tmp_path / f"_ls_call_{i}.so"
        path.write_bytes(image.replace(old, new))
        monkeypatch.setattr(ls, "CALL_PATH", str(path))
        with pytest.warns(RuntimeWarning, match="ctypes"):
            made = ls._device_calls(lib)
        assert type(made.ls_kv_commit).__name__ != "Caller"
        assert made.ls_hybrid_tree_attn(*args) == ls.LS_OK and lib.take_route()


def test_an_outdated_module_is_built_again(tmp_path, monkeypatch):
    module = tmp_path / "_ls_call.so"
    monkeypatch.setattr(ls_build, "CALL_PATH", str(module))
    assert ls_build.call_module_is_stale()
    module.write_bytes(b"")
    assert not ls_build.call_module_is_stale()
    for source in (ls_build.CALL_SRC, ls_build.HEADER):
        os.utime(module, (os.path.getmtime(source) - 10,) * 2)
        assert ls_build.call_module_is_stale()


def test_acceptance_takes_the_first_two_axes_of_parents(calls, monkeypatch):  # noqa: F811
    """A trailing axis of one is as good as none."""
    _, made = calls
    seen = []

    def record(*args):
        seen.append(args[3:5])
        return made.ls_tree_accept_greedy(PARENTS, Q, K, *args[3:5], OUT, LENS, LSE, None, None)

    monkeypatch.setattr(ls, "lib", lambda: types.SimpleNamespace(call=types.SimpleNamespace(ls_tree_accept_greedy=record)))
    monkeypatch.setattr(ls, "_stream", lambda stream: None)
    for shape in ((3, 7), (3, 7, 1)):
        x = torch.zeros(shape, dtype=torch.int32)
        assert ls.ls_tree_accept_greedy(x, x, x, x, x, x) == ls.LS_OK
    assert seen == [(3, 7), (3, 7)]


def test_an_argument_too_many_is_an_error(calls):  # noqa: F811
    x = desc(8, 2, 128, 8, 300)
    with pytest.raises(TypeError):
        calls[1].ls_hybrid_tree_attn(x, Q, K, V, LENS, KT, VT, PARENTS, OUT, LSE, WORK, 1 << 40, None, None)


@pytest.mark.parametrize("native", [True, False])
def test_an_integer_is_no_tensor(lib, native, monkeypatch):  # noqa: F811
    """The binding's functions take tensors: a size or an index in the place of one is an error, not an address."""
    ls_build.build_call_module(force=False)
    for name in ls._DEVICE_CALLS:
        getattr(lib, name).argtypes = getattr(ls.lib(), name).argtypes
    if not native:
        monkeypatch.setattr(ls, "CALL_PATH", ls.CALL_PATH + ".missing")
    made = ls._device_calls(lib, addresses=False)
    assert (type(made.ls_kv_commit).__name__ == "Caller") == native
    x = desc(8, 2, 128, 8, 300)

    class Pointer:
        def __init__(self, address):
            self.address = address

        def data_ptr(self):
            return self.address

    args = [x, *[Pointer(a) for a in (Q, K, V, LENS, KT, VT, PARENTS, OUT, LSE, WORK)], 1 << 40, 12345]
    assert made.ls_hybrid_tree_attn(*args) == ls.LS_OK and lib.take_route()
    for at in range(1, 11):
        a = list(args)
        a[at] = 64
        with pytest.raises(AttributeError, match="data_ptr"):
            made.ls_hybrid_tree_attn(*a)
    assert not lib.take_route()
    y = torch.zeros((1, 4), dtype=torch.int32)
    with pytest.raises(AttributeError, match="data_ptr"):
        ls.ls_tree_accept_greedy(y, y, 64, y, y, y, stream=0)

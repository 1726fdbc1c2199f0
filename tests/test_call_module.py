"""The native module between Python and the C ABI, on the CPU: what its callables take for pointers, integers and descriptors, with
the library's host code and launchers that only write down what they are asked for."""
import ctypes
import os
import types

import pytest
import torch

from paper_2502_17421_amd import binding as ls
from paper_2502_17421_amd import build as ls_build
from test_call_routes import KT, K, LENS, LSE, OUT, PARENTS, Q, V, VT, WORK, desc, lib  # noqa: F401  (lib: fixture)


@pytest.fixture(scope="module", params=["native", "ctypes"])
def calls(request, lib):  # noqa: F811
    ls_build.build_call_module(force=False)
    for name in ls._DEVICE_CALLS:
        getattr(lib, name).argtypes = getattr(ls.lib(), name).argtypes
    path, ls.CALL_PATH = ls.CALL_PATH, ls.CALL_PATH if request.param == "native" else ls.CALL_PATH + ".missing"
    try:
        made = ls._device_calls(lib)
        tensors_only = ls._device_calls(lib, addresses=False)
    finally:
        ls.CALL_PATH = path
    assert (type(made.ls_kv_commit).__name__ == "Caller") == (request.param == "native")
    made.tensors_only = tensors_only
    return lib, made


def test_every_pointer_form_reaches_the_library(calls):
    lib, made = calls  # noqa: F811
    x = desc(8, 2, 128, 8, 300)
    args = [x, Q, K, V, LENS, KT, VT, PARENTS, OUT, LSE, WORK, 1 << 40, None]
    for at in (None, *range(1, 11)):
        # a missing pointer is refused, except that of the lengths' order of checks: all of them by the same status
        a = list(args)
        if at is not None:
            a[at] = None
        status = made.ls_hybrid_tree_attn(*a)
        assert status == (ls.LS_OK if at is None else ls.LS_ERR_WORKSPACE if at == 10 else ls.LS_ERR_NULL), at
        assert bool(lib.take_route()) == (at is None)

    class Other(torch.Tensor):
        pass

    class Pointer:
        def data_ptr(self):
            return Q

    odd = torch.zeros(64, dtype=torch.uint8)
    aligned = odd[(-odd.data_ptr()) % 16:]
    for q, expect in ((aligned, ls.LS_OK), (aligned[1:], ls.LS_ERR_STRIDE), (aligned.as_subclass(Other), ls.LS_OK),
                      (torch.nn.Parameter(aligned.float()[:1].new_zeros(64)), ls.LS_OK), (Pointer(), ls.LS_OK),
                      (Q + 8, ls.LS_ERR_STRIDE), (torch.empty(0), ls.LS_ERR_NULL)):
        a = list(args)
        a[1] = q
        assert made.ls_hybrid_tree_attn(*a) == expect, (q, expect)
        lib.take_route()
    # sizes as large as they come, negative integers, and 32-bit results
    assert made.ls_hybrid_tree_attn(*args[:11], 2 ** 64 - 1, None) == ls.LS_OK
    assert made.ls_hybrid_tree_attn(*args[:11], 0, None) == ls.LS_ERR_WORKSPACE
    assert made.ls_prefix_attn_splitkv(x, Q, K, V, LENS, -1, ls.LS_F32, OUT, LSE, None) == ls.LS_ERR_SHAPE
    assert made.ls_tree_accept_greedy(PARENTS, Q, K, 0, 4, OUT, LENS, LSE, None, None) == ls.LS_ERR_SHAPE
    assert made.ls_tree_accept_greedy(PARENTS, Q, K, 1, 4, OUT, LENS, LSE, None, None) == ls.LS_OK
    lib.take_route()


def test_wrong_arguments_are_python_errors(calls):
    _, made = calls
    x = desc(8, 2, 128, 8, 300)
    args = [x, Q, K, V, LENS, KT, VT, PARENTS, OUT, LSE, WORK, 1 << 40, None]
    errors = (TypeError, AttributeError, ctypes.ArgumentError)
    for at, value in ((0, (ctypes.c_char * 8)()), (0, 3.5), (1, "text"), (1, 2.5), (11, "text"), (11, None)):
        a = list(args)
        a[at] = value
        if type(made.ls_kv_commit).__name__ == "Caller" or not isinstance(value, str) or at != 1:
            with pytest.raises(errors):
                made.ls_hybrid_tree_attn(*a)
    with pytest.raises(errors):
        made.ls_hybrid_tree_attn(*args[:-1])
    with pytest.raises(errors):
        made.ls_hybrid_tree_attn(*args, None)


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


def test_acceptance_takes_the_first_two_axes_of_parents(calls, monkeypatch):
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


def test_an_integer_is_no_tensor(calls):
    """The binding's functions take tensors: a size or an index in the place of one is an error, not an address."""
    lib, made = calls  # noqa: F811
    x = desc(8, 2, 128, 8, 300)

    class Pointer:
        def __init__(self, address):
            self.address = address

        def data_ptr(self):
            return self.address

    args = [x, *[Pointer(a) for a in (Q, K, V, LENS, KT, VT, PARENTS, OUT, LSE, WORK)], 1 << 40, 12345]
    assert made.tensors_only.ls_hybrid_tree_attn(*args) == ls.LS_OK and lib.take_route()
    for at in range(1, 11):
        a = list(args)
        a[at] = 64
        with pytest.raises(AttributeError, match="data_ptr"):
            made.tensors_only.ls_hybrid_tree_attn(*a)
    assert not lib.take_route()
    y = torch.zeros((1, 4), dtype=torch.int32)
    with pytest.raises(AttributeError, match="data_ptr"):
        ls.ls_tree_accept_greedy(y, y, 64, y, y, y, stream=0)

"""The native module between Python and the C ABI, on the CPU: what its callables take for pointers, integers and descriptors, with
the library's host code and launchers that only write down what they are asked for."""
import ctypes
import os

import pytest
import torch

from paper_2502_17421_amd import binding as ls
from paper_2502_17421_amd import build as ls_build
from test_call_routes import KT, K, LENS, LSE, OUT, PARENTS, Q, V, VT, WORK, desc, lib  # noqa: F401  (lib: fixture)


@pytest.fixture(scope="module", params=["native", "ctypes"])
def calls(request, lib):  # noqa: F811
    if not os.path.exists(ls.CALL_PATH):
        ls_build.build_call_module()
    for name in ls._DEVICE_CALLS:
        getattr(lib, name).argtypes = getattr(ls.lib(), name).argtypes
    path, ls.CALL_PATH = ls.CALL_PATH, ls.CALL_PATH if request.param == "native" else ls.CALL_PATH + ".missing"
    try:
        made = ls._device_calls(lib)
    finally:
        ls.CALL_PATH = path
    assert (type(made.ls_kv_commit).__name__ == "Caller") == (request.param == "native")
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

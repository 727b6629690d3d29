"""The CPython module that marshals the arguments of attn_update, against a recording callback in place of the library."""
import ctypes as C

import numpy as np
import pytest
import torch


class Fake:
    """What the module asks of a tensor: an address, sizes, bytes."""

    def __init__(self, address, shape, nbytes=0):
        self.address, self.shape, self.nbytes = address, shape, nbytes

    def data_ptr(self):
        return self.address


@pytest.fixture
def call():
    """call(...) -> the arguments that reached the library (with workspace: 19, without: 17)"""
    from paper_2505_15781_amd import binding as b
    got = []
    with_ws = C.CFUNCTYPE(C.c_int, *[C.c_void_p] * 8, *[C.c_int32] * 8, C.c_void_p, C.c_size_t, C.c_void_p)(lambda *a: got.append(a) or 0)
    static = C.CFUNCTYPE(C.c_int, *[C.c_void_p] * 8, *[C.c_int32] * 8, C.c_void_p)(lambda *a: got.append(a) or 0)
    b._marshal.bind(C.cast(with_ws, C.c_void_p).value, C.cast(static, C.c_void_p).value, C.c_int32)

    def run(static=False, **over):
        args = dict(k_cache=Fake(16, (3, 2, 70, 64)), v_cache=Fake(32, (3, 2, 70, 64)), q=Fake(48, (9, 6, 64)), k_new=Fake(64, (9, 2, 64)),
                    v_new=Fake(80, (9, 2, 64)), idx=Fake(96, (9,)), off=Fake(112, (4,)), out=Fake(128, (9, 6, 64)), rows=9, max_rows=5,
                    dtype=0, workspace=Fake(144, (100,), 100), stream=7)
        args.update(over)
        if static:
            del args["workspace"]
        got.clear()
        assert (b._marshal.attn_update_static if static else b._marshal.attn_update)(*args.values()) == 0
        return got[0]

    yield run
    b._marshal.bind(C.cast(b.lib.dkv_attn_update, C.c_void_p).value, C.cast(b.lib.dkv_attn_update_static, C.c_void_p).value,
                    C.c_int32)


def test_arguments_reach_the_library_in_order(call):
    assert call() == (16, 32, 48, 64, 80, 96, 112, 128, 9, 5, 3, 6, 2, 70, 64, 0, 144, 100, 7)
    assert call(static=True) == (16, 32, 48, 64, 80, 96, 112, 128, 9, 5, 3, 6, 2, 70, 64, 0, 7)
    assert call(q=None, workspace=None)[2] is None and call(q=None, workspace=None)[16:18] == (None, 0)
    assert call(q=Fake(48, (9 * 6, 64)), out=Fake(128, (9, 5, 64)))[11] == 5          # query heads from out


@pytest.mark.parametrize("value", [5, np.int64(5), torch.tensor(5), C.c_int32(5)])
def test_whole_numbers_are_taken_as_ctypes_takes_them(call, value):
    assert call(rows=value)[8] == 5 and call(max_rows=value)[9] == 5


@pytest.mark.parametrize("value", [5.0, "5", None, C.c_int64(5)])
def test_other_numbers_are_refused(call, value):
    with pytest.raises(TypeError):
        call(rows=value)


def test_sizes_beyond_32_bits_are_an_error_and_do_not_wrap(call):
    for shape in ((3, 2, 2**32 + 70, 64), (3, 2, 2**31, 64), (2**33, 2, 70, 64)):
        with pytest.raises(OverflowError):
            call(k_cache=Fake(16, shape))
    with pytest.raises(OverflowError):
        call(q=Fake(48, (9, 2**32 + 6, 64)))
    with pytest.raises(OverflowError):
        call(rows=2**32 + 9)


def test_shapes_may_be_any_sequence_of_four_sizes(call):
    assert call(k_cache=Fake(16, [3, 2, 70, 64]))[10:15] == (3, 6, 2, 70, 64)
    for shape in ((3, 2, 70), (1, 3, 2, 70, 64)):
        with pytest.raises(ValueError):
            call(k_cache=Fake(16, shape))


def test_the_module_uses_only_the_stable_abi():
    """Its file name carries no interpreter version: whatever it refers to has to be the same in every Python from 3.10 on."""
    import shutil, subprocess
    from paper_2505_15781_amd import binding as b
    if not shutil.which("nm"):
        pytest.skip("no nm")
    out = subprocess.run(["nm", "-D", "--undefined-only", b._marshal.__file__], capture_output=True, text=True, check=True).stdout
    used = {line.split()[-1] for line in out.splitlines() if "Py" in line}
    stable = {"PyErr_Occurred", "PyErr_SetString", "PyEval_RestoreThread", "PyEval_SaveThread", "PyExc_IndexError", "PyExc_OverflowError",
              "PyExc_RuntimeError", "PyExc_TypeError", "PyExc_ValueError", "PyLong_AsLong", "PyLong_AsSize_t", "PyLong_AsVoidPtr",
              "PyLong_FromLong", "PyModule_Create2", "PyObject_CallMethodObjArgs", "PyObject_GetAttr", "PyObject_IsInstance",
              "PySequence_Tuple", "PyTuple_GetItem", "PyTuple_Size", "PyType_GetFlags", "PyUnicode_InternFromString", "_Py_Dealloc",
              "_Py_NoneStruct", "Py_IncRef", "Py_DecRef"}
    assert used and used <= stable, used - stable

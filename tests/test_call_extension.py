"""The extension that marshals arguments (csrc/hfx_call.c): every form of an argument that the ctypes calls took is taken, and what they refused is
refused.  On functions of the library that run on the host."""
import ctypes
import os
import shutil
import subprocess
import sys
import sysconfig
import threading

import numpy as np
import pytest
import torch

from paper_2508_15919_amd import binding as hb

KIND, Q, CTX = [0, 0, 1, 1], [1, 1, 40, 17], [37, 300, 40, 64]
INDPTR, PAGES = [0, 3, 22, 25, 29], list(range(29))


@pytest.fixture(scope="module")
def fill():
    lib = hb.load()
    from paper_2508_15919_amd import _hfxcall
    return _hfxcall.Caller(ctypes.cast(lib.hfx_fill_batch_desc, ctypes.c_void_p).value, "SKAAAAB", hb.hfx_shape, hb._ptr, hb._as_int32)


def reference():
    shape = hb.make_shape(8, 2, 64, 32)
    size = hb.hfx_batch_desc_sizes(shape, KIND, Q, CTX)[0]
    blob = np.zeros(size, np.uint8)
    hb.hfx_fill_batch_desc(shape, KIND, Q, CTX, INDPTR, PAGES, blob)
    return shape, blob


FORMS = {
    "int32": lambda a: np.array(a, np.int32), "list": list, "tuple": tuple, "int64": lambda a: np.array(a, np.int64), "float": lambda a: np.array(a, np.float64),
    "strided": lambda a: np.repeat(np.array(a, np.int32), 2)[::2], "read-only": lambda a: np.frombuffer(np.array(a, np.int32).tobytes(), np.int32),
    "uint32": lambda a: np.array(a, np.uint32), "big-endian": lambda a: np.array(a, ">i4"), "tensor": lambda a: torch.tensor(a, dtype=torch.int32),
    "bytes of others": lambda a: np.array(a, np.int16), "row": lambda a: np.array(a, np.int32).reshape(-1, 1)[:, 0]}


@pytest.mark.parametrize("form", sorted(FORMS))
def test_arrays_of_every_form(fill, form):
    shape, ref = reference()
    make = FORMS[form]
    blob = np.zeros_like(ref)
    assert fill(shape, make(KIND), make(Q), make(CTX), make(INDPTR), make(PAGES), blob) == hb.HFX_OK
    assert np.array_equal(blob, ref)


def test_pointers_of_every_form(fill):
    shape, ref = reference()
    for make in (lambda n: np.zeros(n, np.uint8), lambda n: torch.zeros(n, dtype=torch.uint8)):
        blob = make(len(ref))
        assert fill(shape, KIND, Q, CTX, INDPTR, PAGES, blob) == hb.HFX_OK
        assert np.array_equal(np.asarray(blob), ref)
    assert fill(shape, KIND, Q, CTX, INDPTR, PAGES, None) == hb.HFX_ERR_NULL
    assert fill(shape, KIND, Q, CTX, INDPTR, PAGES, np.zeros(len(ref) - 1, np.uint8)) == hb.HFX_ERR_BUFSIZE
    assert fill(shape, KIND, None, CTX, INDPTR, PAGES, np.zeros_like(ref)) == hb.HFX_ERR_NULL


@pytest.mark.parametrize("change", [dict(shape=None), dict(shape=hb.hfx_decision()), dict(kind=None), dict(pages="abc"), dict(blob="text"), dict(blob=1.5),
                                    dict(blob=ctypes.c_void_p(0)), dict(pages=[[1, 2], [3]])])
def test_what_is_refused(fill, change):
    shape, ref = reference()
    a = dict(shape=shape, kind=KIND, q=Q, ctx=CTX, indptr=INDPTR, pages=PAGES, blob=np.zeros_like(ref))
    a.update(change)
    with pytest.raises((TypeError, ValueError)):
        fill(*a.values())


def test_number_of_arguments(fill):
    shape, ref = reference()
    with pytest.raises(TypeError):
        fill(shape, KIND)
    with pytest.raises(TypeError):
        fill(shape, KIND, Q, CTX, INDPTR, PAGES, blob=ref)
    from paper_2508_15919_amd import _hfxcall
    for kinds, address in (("SX", 1), ("S", 0), ("B" * 7, 1), ("P" * 17, 1), ("S" * 9, 1), ("SSSKKKAAA", 1), ("A" * 12, 1), ("a" * 9, 1), ("k" * 7, 1)):
        with pytest.raises(ValueError):
            _hfxcall.Caller(address, kinds, hb.hfx_shape, hb._ptr, hb._as_int32)
    with pytest.raises(TypeError):
        _hfxcall.Caller.__new__(_hfxcall.Caller)()


def test_validation_of_the_public_calls():
    """No GPU is touched: the calls are refused before that."""
    shape, ref = reference()
    with pytest.raises(hb.HfxError) as e:
        hb.hfx_mixed_paged_attention(shape, None, 16, ref, 16, None, 16)
    assert e.value.code == hb.HFX_ERR_NULL
    with pytest.raises(hb.HfxError) as e:
        hb.hfx_append_kv(shape, 16, 16, 16, np.zeros(512, np.uint8), 16, stream=None)
    assert e.value.code == hb.HFX_ERR_DESC
    with pytest.raises(hb.HfxError) as e:
        hb.hfx_gather_kv(shape, 16, ref, 16, np.int64(99), 16, 16, 0)
    assert e.value.code == hb.HFX_ERR_LEN
    with pytest.raises(hb.HfxError) as e:
        hb.hfx_copy_pages(shape, 16, 16, 32, [1, 40], np.array([2, 3]), np.zeros(16, np.uint8), 16, stage_bytes=16)
    assert e.value.code == hb.HFX_ERR_PAGE_ID
    with pytest.raises(AssertionError):
        hb.hfx_copy_pages(shape, 16, 16, 32, [1], [2, 3], np.zeros(16, np.uint8), 16, stage_bytes=16)
    with pytest.raises(hb.HfxError) as e:
        hb.hfx_build_batch_desc(shape, KIND, Q, CTX, INDPTR, PAGES, np.zeros(64, np.uint8), torch.zeros(64, dtype=torch.uint8))
    assert e.value.code == hb.HFX_ERR_BUFSIZE
    with pytest.raises(AttributeError):
        hb.hfx_append_kv(shape, 16, 16, 16, ref, 16, stream="none")


def test_lists_that_are_read_once_are_passed_in_place():
    from paper_2508_15919_amd import _hfxcall
    base = np.arange(5, dtype=np.int32)
    seen = []

    @ctypes.CFUNCTYPE(ctypes.c_int32, ctypes.c_int64, ctypes.c_void_p, ctypes.c_void_p)
    def look(length, first, second):
        seen.append((length, first, second))
        return 0

    call = _hfxcall.Caller(ctypes.cast(look, ctypes.c_void_p).value, "ka", hb.hfx_shape, hb._ptr, hb._as_int32)
    call(base, base)
    assert seen == [(5, base.ctypes.data, base.ctypes.data)]


@pytest.mark.parametrize("one", [lambda i: i, np.int64, np.int32, lambda i: np.array(i, np.int32), lambda i: torch.tensor(i)])
def test_a_single_page_is_a_list_of_one(one):
    """hfx_copy_pages with a number in the place of a list: 40 is outside the pool, 3 is inside, and the call gets as far as the staging buffers' size."""
    shape = hb.make_shape(8, 2, 64, 32)
    for i, code in ((40, hb.HFX_ERR_PAGE_ID), (3, hb.HFX_ERR_BUFSIZE)):
        with pytest.raises(hb.HfxError) as e:
            hb.hfx_copy_pages(shape, 16, 16, 32, one(i), one(5), np.zeros(16, np.uint8), 16, stage_bytes=8 if i == 40 else 7)
        assert e.value.code == code
    with pytest.raises(AssertionError):
        hb.hfx_copy_pages(shape, 16, 16, 32, one(1), [2, 3], np.zeros(16, np.uint8), 16, stage_bytes=16)


@pytest.mark.parametrize("form", ["int32", "list", "tensor", "strided"])
@pytest.mark.parametrize("n", [0, 1, 300, 4095])
def test_small_arrays_are_read_before_the_lock_is_released(n, form):
    """What a call checks is what it uses: arrays of less than 16 KB that change after it has begun are seen as they were.  (The function called here
    changes the caller's array and then looks at its arguments.)"""
    from paper_2508_15919_amd import _hfxcall
    base = np.arange(1, n + 1, dtype=np.int32)
    given = FORMS[form](base)
    if form == "tensor":
        given = torch.from_numpy(base)
    seen = []

    @ctypes.CFUNCTYPE(ctypes.c_int32, ctypes.c_int64, ctypes.c_void_p, ctypes.c_void_p)
    def look(length, first, second):
        if form in ("int32", "strided"):
            given[:] = -1
        base[:] = -1
        seen.append([length] + [np.ctypeslib.as_array(ctypes.cast(p, ctypes.POINTER(ctypes.c_int32)), (n,)).tolist() if n else p != 0 for p in (first, second)])
        return 7

    call = _hfxcall.Caller(ctypes.cast(look, ctypes.c_void_p).value, "KA", hb.hfx_shape, hb._ptr, hb._as_int32)
    assert call(given, given) == 7
    was = list(range(1, n + 1)) if n else True
    assert seen == [[n, was, was]]


def test_the_extension_is_of_this_python(fill):
    """Another interpreter, whose type records may be laid out otherwise, does not find it."""
    from paper_2508_15919_amd import _hfxcall
    suffix = sysconfig.get_config_var("EXT_SUFFIX")
    assert suffix != ".so" and os.path.basename(_hfxcall.__file__) == "_hfxcall" + suffix
    assert not os.path.exists(os.path.join(os.path.dirname(_hfxcall.__file__), "_hfxcall.so"))


WITHOUT = """
import sys
sys.modules["paper_2508_15919_amd._hfxcall"] = None          # importing it fails
import numpy as np
from paper_2508_15919_amd import binding as hb
shape = hb.make_shape(8, 2, 64, 32)
size = hb.hfx_batch_desc_sizes(shape, [0], [1], [37])[0]
hb.hfx_fill_batch_desc(shape, [0], [1], [37], [0, 3], [0, 1, 2], np.zeros(size, np.uint8))
assert hb.hfx_token_budget(1.0, 0.5, hb.hfx_latency_model(0.01, 0.001, 0.1)) > 0
assert len(hb.hfx_compose_step(1.0, 0.5, hb.hfx_latency_model(0.01, 0.001, 0.1), [5], [10])) == 5
try:
    hb.hfx_append_kv(shape, 16, 16, 16, np.zeros(size, np.uint8), 16)
except RuntimeError as e:
    print(e)
"""


def test_calls_that_do_not_use_the_extension_do_not_need_it():
    root = os.path.dirname(os.path.dirname(hb.LIB_PATH))
    res = subprocess.run([sys.executable, "-c", WITHOUT], cwd=root, capture_output=True, text=True, timeout=120)
    assert res.returncode == 0 and "the call extension is missing" in res.stdout, res.stderr


@pytest.mark.parametrize("target", [["-U__x86_64__"], ["-D__ILP32__"], ["-D_WIN32"]])
def test_other_calling_conventions_are_refused(target):
    if shutil.which("gcc") is None:
        pytest.skip("gcc not available")
    source = os.path.join(os.path.dirname(hb.LIB_PATH), "csrc", "hfx_call.c")
    res = subprocess.run(["gcc", "-E", "-o", os.devnull, *target, source], capture_output=True, text=True)
    assert res.returncode != 0 and "System V convention" in res.stderr


def test_several_threads(fill):
    shape, ref = reference()
    wrong = []

    def work():
        for _ in range(300):
            blob = np.zeros_like(ref)
            if fill(shape, KIND, np.array(Q), CTX, INDPTR, np.array(PAGES, np.int32), blob) != hb.HFX_OK or not np.array_equal(blob, ref):
                wrong.append(1)

    threads = [threading.Thread(target=work) for _ in range(4)]
    [t.start() for t in threads]
    [t.join() for t in threads]
    assert not wrong

"""The native call path of sqllm_dense_sparse_matvec takes and refuses the arguments that the ctypes path takes and refuses.  No GPU: every
call here fails validation on the host, or is not for the native path."""
import ctypes
import os
import sys

import numpy as np
import pytest

import paper_2306_07629_amd as sq
from paper_2306_07629_amd import binding, build

GOOD = dict(M=4, N=128, bits=3, nnz=0, B=1, qidx=4096, lut=4096, rowptr=None, cols=None, vals=None, plan=None, x=4096, y=4096, stream=0)


class Tensor:
    def __init__(self, p):
        self.p = p

    def data_ptr(self):
        return self.p


class Stream:
    cuda_stream = 0


@pytest.fixture(scope="module")
def native():
    if build.pycall_is_stale():
        build.build_pycall()
    from paper_2306_07629_amd import _pycall
    asked = []
    _pycall.bind(ctypes.cast(sq.lib().sqllm_dense_sparse_matvec, ctypes.c_void_p).value, lambda: 3, lambda dev: asked.append(dev) or 0)
    yield _pycall.matvec, asked
    binding._matvec = binding._matvec_first                              # binds again, to the real streams


@pytest.mark.parametrize("change", [dict(bits=5), dict(N=100), dict(N=-128), dict(M=-1), dict(B=17), dict(B=0), dict(nnz=-1), dict(nnz=1 << 40), dict(nnz=5),
                                    dict(qidx=None), dict(lut=4098), dict(x=None), dict(x=4100), dict(y=4097), dict(nnz=3, plan=4100), dict(M=0, bits=9),
                                    dict(N=(1 << 32) + 100), dict(qidx=Tensor(4104)), dict(x=Tensor(0)), dict(bits=True), dict(bits=5, stream=Stream())])
def test_same_status_and_message_as_ctypes(native, change):
    args = list({**GOOD, **change}.values())
    want = binding._matvec_ctypes(*args)
    text = sq.lib().sqllm_last_error_string()
    assert want != 0
    assert native[0](*args) == want and sq.lib().sqllm_last_error_string() == text


@pytest.mark.parametrize("change", [dict(M=4.0), dict(N="128"), dict(bits=np.int64(3)), dict(qidx=Tensor(1.5)), dict(stream=Tensor(0))])
def test_other_arguments_are_left_to_ctypes(native, change):
    args = list({**GOOD, **change, "B": 99}.values())                    # 99 columns: no launch, whichever path
    try:
        got = native[0](*args)
    except AttributeError:
        with pytest.raises(AttributeError):
            binding._matvec_ctypes(*args)
        return
    assert got is None
    if isinstance(change.get("bits"), np.integer):                       # ctypes takes what has an index
        assert binding._matvec_ctypes(*args) == 6
    else:
        with pytest.raises((ctypes.ArgumentError, AttributeError)):
            binding._matvec_ctypes(*args)


def test_current_stream_is_asked_for_the_current_device(native):
    del native[1][:]
    assert native[0](*{**GOOD, "bits": 7, "stream": None}.values()) == 2
    assert native[1] == [3]


def test_errors_of_data_ptr_arrive(native):
    class Gone:
        def data_ptr(self):
            raise RuntimeError("freed")
    with pytest.raises(RuntimeError, match="freed"):
        native[0](*{**GOOD, "x": Gone()}.values())
    with pytest.raises(AttributeError):
        native[0](*{**GOOD, "x": object()}.values())


@pytest.fixture
def fresh(monkeypatch):
    """a process that has not called yet"""
    monkeypatch.setattr(binding, "_matvec", binding._matvec_first)
    return monkeypatch


def call(**change):
    a = {**GOOD, **change}
    return sq.sqllm_dense_sparse_matvec(a["M"], a["N"], a["bits"], a["nnz"], a["B"], a["qidx"], a["lut"], a["rowptr"], a["cols"], a["vals"],
                                        a["x"], a["y"], stream=a["stream"], plan=a["plan"])


def test_public_call_takes_the_native_path_whatever_the_stream(native, fresh):
    from paper_2306_07629_amd import _pycall
    with pytest.raises(sq.SqllmError) as e:
        call(bits=7, stream=0)                                           # a program that always passes its stream
    assert e.value.status == 2 and binding._matvec is _pycall.matvec
    with pytest.raises(sq.SqllmError) as e:                              # left to ctypes by the native path
        call(bits=np.int64(3), B=99)
    assert e.value.status == 6


@pytest.mark.parametrize("cause", ["no compiler", "no module"])
def test_without_the_module_calls_go_through_ctypes(native, fresh, capfd, cause):
    import paper_2306_07629_amd as package
    if cause == "no compiler":
        fresh.setattr(build, "PYCALL", "/nonexistent/_pycall.so")
        fresh.setattr(build, "CC", "/nonexistent/gcc")
    else:
        fresh.delattr(package, "_pycall")
        fresh.setitem(sys.modules, "paper_2306_07629_amd._pycall", None)   # import raises ImportError
    for _ in range(2):
        with pytest.raises(sq.SqllmError) as e:
            call(bits=7)
        assert e.value.status == 2 and binding._matvec is binding._matvec_ctypes
    assert capfd.readouterr().err.count("through ctypes") == 1


def test_a_library_without_the_module_is_not_stale(monkeypatch):
    sq.lib()
    monkeypatch.setattr(build, "PYCALL", "/nonexistent/_pycall.so")
    assert build.pycall_is_stale() and not build.is_stale()


def test_the_library_is_built_without_a_c_compiler(monkeypatch, capfd):
    monkeypatch.setattr(build, "HIPCC", "true")                          # stands for a compiler that succeeds
    monkeypatch.setattr(build, "CC", "/nonexistent/gcc")
    before = os.path.getmtime(build.PYCALL) if os.path.exists(build.PYCALL) else None
    assert build.build() == build.LIB
    assert "was not built" in capfd.readouterr().err
    assert before is None or os.path.getmtime(build.PYCALL) == before    # what was there stays


def test_the_module_is_named_for_its_interpreter():
    import importlib.machinery
    assert os.path.basename(build.PYCALL) == "_pycall" + importlib.machinery.EXTENSION_SUFFIXES[0]


def test_binding_raises_with_the_status():
    with pytest.raises(sq.SqllmError) as e:
        sq.sqllm_dense_sparse_matvec(4, 128, 7, 0, 1, 4096, 4096, None, None, None, 4096, 4096, stream=0)
    assert e.value.status == 2

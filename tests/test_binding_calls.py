"""The caller behind the binding's hot entry points: argument kinds, refusals, agreement with the ctypes prototypes."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2509_09679_amd import binding as B


class Fake:  # a tensor as far as the binding looks at one
    def data_ptr(self):
        return 0x7F0000001000

    def numel(self):
        return 64

    def element_size(self):
        return 1


def _rows(**kw):
    r = B.bq_rows()
    r.rows, r.n, r.heads, r.ld_x, r.ld_y, r.dtype = 4, 64, 1, 64, 64, B.BQ_F16
    for k, v in kw.items():
        setattr(r, k, v)
    return r


def test_kinds_match_the_ctypes_prototypes():
    L = B.lib()
    kind = {ctypes.c_void_p: "ps", ctypes.c_int32: "i", ctypes.c_size_t: "u", ctypes.POINTER(B.bq_rows): "r", ctypes.POINTER(B.bq_quant): "q"}
    for name, kinds in B._KINDS.items():
        types = getattr(L, name).argtypes
        assert len(types) == len(kinds) and all(k in kind[t] for k, t in zip(kinds, types)), name


def test_arguments_arrive_and_errors_come_back():
    # every call ends in the library's own checks: nothing is launched
    x, s = Fake(), 0
    with pytest.raises(B.BqError, match="power of two") as e:
        B.bq_butterfly_fwd(x, x, x, _rows(n=12, ld_x=12, ld_y=12), stream=type("S", (), {"cuda_stream": s}))
    assert e.value.status == 2
    for args in ((None, x, x), (x, None, x), (x, x, None)):
        with pytest.raises(B.BqError) as e:
            B.bq_butterfly_inv(*args, _rows(), stream=type("S", (), {"cuda_stream": s}))
        assert e.value.status == 1
    with pytest.raises(B.BqError) as e:  # a workspace of 64 bytes: size_t and the ninth argument
        B.bq_butterfly_bwd(x, x, x, x, x, x, _rows(), stream=type("S", (), {"cuda_stream": s}))
    assert e.value.status == 5
    q = B.make_quant(3, 32, "f16")
    with pytest.raises(B.BqError):
        B.bq_butterfly_fwd_quant(x, x, x, x, q, _rows(), stream=type("S", (), {"cuda_stream": s}))
    with pytest.raises(B.BqError):
        B.bq_plan_build(x, 64, -1, x, stream=type("S", (), {"cuda_stream": s}))


def test_what_is_not_an_argument_is_refused():
    c, x = B._calls(), Fake()
    for bad in ((x, x, x, None, 0), (x, x, x, B.bq_quant(), 0), (x, x, x, _rows()), (x, x, x, _rows(), 0, 0), (x, x, x, _rows(), 0.0),
                (x, x, x, _rows(), None)):
        with pytest.raises(TypeError):
            c.butterfly_fwd(*bad)
    with pytest.raises(AttributeError):
        c.butterfly_fwd(x, 3, x, _rows(), 0)
    with pytest.raises(TypeError):
        c.plan_build(x, 64.0, 1, x, 64, 0)
    with pytest.raises(TypeError):
        c.butterfly_fwd(x, x, x, rows=_rows(), stream=0)

    class Raises(Fake):
        def data_ptr(self):
            raise RuntimeError("no storage")

    with pytest.raises(RuntimeError, match="no storage"):
        c.butterfly_fwd(x, Raises(), x, _rows(), 0)


class Index:
    def __index__(self):
        return 64


class Parameter:
    _as_parameter_ = 64


@pytest.mark.parametrize("n", [64, np.int64(64), np.int32(64), np.array(64), torch.tensor(64), ctypes.c_int32(64), Index(), Parameter(),
                               (1 << 32) + 64])
def test_integers_that_are_not_python_s(n):
    # whatever a ctypes prototype takes for an int32 and a size_t; the calls end in the library's checks, whose texts show the values
    stream, x = type("S", (), {"cuda_stream": 0}), Fake()
    with pytest.raises(B.BqError, match=f"64 bytes, {B.bq_plan_bytes(64)} needed"):
        B.bq_plan_build(x, n, 1, x, stream=stream)
    with pytest.raises(B.BqError, match="n=64 heads=-3"):
        B.bq_plan_build(x, n, np.int64(-3), x, stream=stream)
    for f in (B.bq_kron_fwd, B.bq_kron_inv):
        with pytest.raises(B.BqError, match=f.__name__ + ": d1=65 outside"):
            f(x, x, x, np.int64(65), x, _rows(), stream=stream)

    class Sizes(Fake):
        def numel(self):
            return np.int64(32)

        def data_ptr(self):
            return np.uint64(0x7F0000001000)

    with pytest.raises(B.BqError, match="plan buffer has 32 bytes"):
        B.bq_plan_build(Sizes(), n, 1, Sizes(), stream=stream)


def test_numbers_that_are_no_integers_stay_refused():
    stream, x = type("S", (), {"cuda_stream": 0}), Fake()
    for n in (64.0, np.float32(64), "64", None, ctypes.c_long(64)):
        with pytest.raises(TypeError):
            B.bq_plan_build(x, n, 1, x, stream=stream)


def test_the_caller_is_the_one_built_for_this_python():
    import sysconfig

    assert B.CALL_PATH.endswith(sysconfig.get_config_var("EXT_SUFFIX"))
    assert all(type(getattr(B._calls(), name[3:])).__name__ == "Caller" for name in B._KINDS)


def test_calls_without_the_caller(monkeypatch):
    # another Python, a host without a compiler: the same calls through ctypes
    monkeypatch.setattr(B, "_CALLS", B._Calls("/nonexistent/bqcall.so"))
    assert all(type(getattr(B._calls(), name[3:])).__name__ == "function" for name in B._KINDS)
    test_arguments_arrive_and_errors_come_back()
    test_integers_that_are_not_python_s(np.int64(64))
    test_numbers_that_are_no_integers_stay_refused()


def test_build_without_python_headers(monkeypatch, tmp_path):
    from paper_2509_09679_amd import build

    stale = tmp_path / "bqcall.so"
    stale.write_bytes(b"")
    monkeypatch.setattr(build, "CALL", str(stale))
    monkeypatch.setattr(build.sysconfig, "get_paths", lambda: {"include": str(tmp_path)})
    assert build.build_caller() is False and not stale.exists()

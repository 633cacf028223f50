"""The vector calls of csrc/pycall.c against the ctypes functions that they stand in for: the same statuses, errors and
exceptions for every way of passing the arguments.  CPU only: every call here is refused before any HIP call."""
import ctypes
import inspect

import pytest

import paper_2512_16465_amd as lg
import paper_2512_16465_amd.binding as binding

pytestmark = pytest.mark.skipif(binding._pycall is None, reason="the extension is not built for this Python")

NAMES = ("gemm_run", "gemm_run_noalloc", "gemm_run_batched")


def ctypes_functions():
    """The module's ctypes functions, as they are without the extension."""
    import importlib.util
    import sys
    spec = importlib.util.spec_from_file_location("plain_binding.binding", binding.__file__)      # (in a package without the extension)
    m = importlib.util.module_from_spec(spec)
    sys.modules["plain_binding.binding"] = m
    spec.loader.exec_module(m)
    assert m._pycall is None
    return m


PLAIN = ctypes_functions()
EPI = dict(out_dtype=lg.GEMM_BF16, bias=0, bias_dtype=lg.GEMM_F32, act=lg.GEMM_ACT_NONE)


def outcome(f, args, kw):
    try:
        return ("returned", f(*args, **kw))
    except Exception as e:
        return (type(e).__name__, getattr(e, "status", None), str(e).replace("_slow", ""))


def calls(m, which):
    """(args, kw): a null handle throughout, so nothing is launched."""
    epi = m.make_epilogue(**EPI)
    one = [0, 8, 8, 8, 0, 1, lg.GEMM_BF16, 1.0, 4096, 8, 4096, 8, 0.0, 4096, 8]
    if which == "gemm_run_batched":
        one = [0, 2, 8, 8, 8, 0, 1, lg.GEMM_BF16, 1.0, 4096, 8, 64, 4096, 8, 64, 0.0, 4096, 8, 64]
    names = list(inspect.signature(getattr(m, which)).parameters)
    yield one, {}
    yield one + [epi], {}
    yield one + [epi, 0], dict(check=False)
    yield one + [epi, 0, False], {}
    yield one + [None, 0, 0], {}
    yield [], dict(zip(names, one), check=False)
    yield one[:3], dict(zip(names[3:], one[3:]), epilogue=epi, check=False)
    yield [None] + one[1:], dict(check=False)                                   # pointers may be None
    yield one[:-1] + [1 << 70], dict(check=False)                               # ctypes keeps the low 64 bits
    yield one[:1] + [-5] + one[2:], dict(check=False)
    yield [x if not isinstance(x, float) else int(x) for x in one], dict(check=False)      # an int where a float belongs
    yield [True if x == 1 else x for x in one], dict(check=False)
    yield one[:-1], {}                                                          # one missing
    yield one + [epi, 0, True, 1], {}                                           # one too many
    yield one, dict(nonsense=1)
    yield one, {names[0]: 0}                                                    # twice
    yield one[:1] + ["8"] + one[2:], {}
    yield one[:1] + [8.0] + one[2:], {}
    yield one + ["epilogue"], {}
    yield one + [ctypes.c_int(3)], {}
    yield one + [epi, None], dict(check=False)


@pytest.mark.parametrize("which", NAMES)
def test_every_way_of_calling_has_the_same_outcome(which):
    fast, plain = getattr(lg, which), getattr(PLAIN, which)
    assert fast is getattr(binding._pycall, which) and fast is not plain
    parameters = [[(p.name, p.default) for p in inspect.signature(f).parameters.values()] for f in (fast, plain)]
    assert parameters[0] == parameters[1]
    for (args, kw), (pargs, pkw) in zip(calls(lg, which), calls(PLAIN, which)):
        a, b = outcome(fast, args, kw), outcome(plain, pargs, pkw)
        if a[0] == "GemmError" or a[0] == "returned":
            assert a == b, (args, kw)
        else:
            assert a[0] == b[0], (args, kw, a, b)


def test_a_library_put_in_place_of_the_other_is_called():
    before = binding._lib
    try:
        lg.gemm_run(0, 1, 1, 1, 0, 0, 0, 1.0, 0, 1, 0, 1, 0.0, 0, 1, None, 0, check=False)
        assert binding._lib is not None

        calls_seen = []

        class Other:
            pass
        fn = ctypes.CFUNCTYPE(ctypes.c_int, *binding._lib.gemm_run.argtypes)(lambda *a: calls_seen.append(a[1:4]) or 3)
        other = Other()
        other.gemm_run = other.gemm_run_noalloc = other.gemm_run_batched = fn
        other.gemm_status_string = binding._lib.gemm_status_string
        binding._lib = other
        for _ in range(2):
            assert lg.gemm_run(0, 5, 6, 7, 0, 0, 0, 1.0, 0, 7, 0, 6, 0.0, 0, 6, None, 0, check=False) == 3
        assert calls_seen == [(5, 6, 7)] * 2
    finally:
        binding._lib = before
    assert lg.gemm_run(0, 1, 1, 1, 0, 0, 0, 1.0, 0, 1, 0, 1, 0.0, 0, 1, None, 0, check=False) == lg.GEMM_ERR_INVALID_ARG

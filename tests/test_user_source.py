"""User likelihood sources that compile (hipRTC needs no GPU): their names and macros are theirs."""
import ctypes as C

import pytest

from paper_2601_19957_amd import _lib

BODY = "__device__ double {0}(const double *x, int d, const double *p) {{ return x[0] * {1}; }}"


def compiles(source, name):
    """True where the source compiles (loading the code needs a GPU)."""
    fn = C.c_void_p()
    st = _lib.lib().sb_user_compile(source.encode(), name.encode(), C.byref(fn))
    if st == _lib.OK:
        _lib.lib().sb_user_release(fn)
    return st in (_lib.OK, _lib.E_DEVICE)


@pytest.mark.parametrize("word", ["N", "R", "X", "ds", "npt", "eps", "lane", "n", "r", "r0", "e0",
                                  "b0", "q", "v", "step", "sgn", "F", "B", "params", "l", "b"])
def test_source_macros(word):
    assert compiles(f"#define {word} 3\n" + BODY.format("like", word), "like")


@pytest.mark.parametrize("name", ["N", "R", "n", "r", "v", "eps", "lane", "step", "q", "i", "j", "t",
                                  "F", "b", "x0", "l"])
def test_source_function_names(name):
    assert compiles(BODY.format(name, 2), name)


def test_error_names_the_source_line():
    assert not compiles("// a likelihood\n__device__ double f(const double *x, int d, "
                        "const double *p) { return missing; }", "f")
    assert ":2:" in _lib.last_error() and "missing" in _lib.last_error()

"""The extension module's calls against the ctypes wrappers that they stand in for: the same result, status or exception for every form
of arguments.  Nothing is launched in any of them: outputs are empty, or two arguments are wrong of which a case mends one at most."""
import ctypes
import os
import subprocess
import sys

import pytest

import paper_2305_13525_amd as axo
from paper_2305_13525_amd import binding

_calls = pytest.importorskip("paper_2305_13525_amd._calls", reason="the extension module is not built")

A, B, C, D = (i << 32 for i in range(1, 5))
LONG = axo.Problem.make((1, 1, 1), (0, 0, 0), 64, 32, 2000)  # rows longer than the pitches below
PRODUCTS = {
    "axo_fc_fwd": (A, 32, B, 48, None, 0, C, 48),
    "axo_fc_dgrad": (A, 48, B, 48, C, 32),
    "axo_fc_wgrad": (A, 32, B, 48, None, 48),
    "axo_fc_dgrad_act": (A, 48, B, 48, D, 32, 2, C, 32),
    "axo_fc_wgrad_acc": (A, 32, B, 48, None, 48),
}
SUMS = {"axo_bias_grad": (A, 48, None), "axo_bias_grad_ws": (A, 48, None), "axo_bias_grad_static": (A, 48, None)}


class Sub(axo.Problem):
    pass


def outcome(f, *a, **k):
    try:
        return f(*a, **k)
    except Exception as e:  # noqa: BLE001
        return type(e), str(e)


def empty(name, kind=axo.Problem):
    """A problem whose result has no elements."""
    return kind.make((1, 1, 1), (0, 0, 0), *((0, 32, 48) if name in ("axo_fc_fwd", "axo_fc_dgrad", "axo_fc_dgrad_act") else (64, 0, 0)))


def forms(name):
    EMPTY = empty(name)
    plain = {**PRODUCTS, **SUMS}[name]
    tail = (None, 0, None) if name in PRODUCTS else (0, None, 0, None) if name.endswith("_ws") else (0, None)
    yield (EMPTY,) + plain + tail + (False,), {}
    yield (LONG,) + plain + tail + (True,), {}
    for p in (EMPTY, None, empty(name, Sub), 7, axo.Problem.make((0, 1, 1), (0, 0, 0), 8, 8, 8)):
        yield (p,) + plain, {"check": False}
        yield (p,) + plain + tail + (False,), {}
    for n in range(len(plain)):
        yield (EMPTY,) + plain[:n], {}
    yield (EMPTY,) + plain + tail + (False, 1), {}
    yield (EMPTY,) + plain, {"nonsense": 1}
    yield (), {}
    for i in range(len(plain)):                                  # other types, and values outside the C types
        for v in (1.5, "x", b"x", None, True, -1, 2 ** 31, 2 ** 63, 2 ** 64, -2 ** 63 - 1, ctypes.c_int64(48), 3):
            args = list(plain)
            args[i] = v
            yield (LONG,) + tuple(args) + tail + (False,), {}
            yield (EMPTY,) + tuple(args), {}
    for i in range(len(tail)):
        for v in (2.5, -1, 1, 2 ** 40, "x"):
            args = list(tail)
            args[i] = v
            yield (LONG,) + plain + tuple(args) + (0,), {}
            yield (EMPTY,) + plain + tuple(args), {}


@pytest.mark.parametrize("name", [*PRODUCTS, *SUMS])
def test_same_as_the_ctypes_wrapper(name):
    quick, wrapper = getattr(_calls, name), None
    assert getattr(axo, name) is quick and getattr(binding, name) is quick
    axo.library()
    wrapper = binding._WRAPPERS[name]
    n = 0
    for args, kw in forms(name):
        want = outcome(wrapper, *args, **kw)
        assert outcome(quick, *args, **kw) == want, (args, kw)
        n += 1
    assert n > 60


# One product without outputs for each function, in a process of its own, through wrappers that count their calls.
EACH_ONCE = """
import ctypes
import sys
sys.path.insert(0, "tests")
import paper_2305_13525_amd as axo
from paper_2305_13525_amd import _calls, binding
assert binding._lib is None
import test_calls
assert binding._lib is None
counts = []
def counted(name):
    def wrapper(*a, **k):
        counts.append(name)
        return binding._WRAPPERS[name](*a, **k)
    return wrapper
_calls.set_up(axo.Problem, {name: counted(name) for name in binding._QUICK}, binding._check)
def each():
    del counts[:]
    for name in binding._QUICK:
        assert getattr(axo, name)(test_calls.empty(name), *{**test_calls.PRODUCTS, **test_calls.SUMS}[name]) == 0, name
    return list(counts)
"""


def in_a_process(code):
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", EACH_ONCE + code], cwd=root, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert r.returncode == 0, r.stdout


@pytest.mark.parametrize("first", binding._QUICK)
def test_not_loaded_yet(first):
    """Before the library is loaded the wrapper is called, which loads it; from then on none is."""
    in_a_process(f"""
assert getattr(axo, {first!r})(test_calls.empty({first!r}), *{{**test_calls.PRODUCTS, **test_calls.SUMS}}[{first!r}]) == 0
assert counts == [{first!r}] and binding._lib is not None
assert each() == []
""")


def test_library_of_another_version():
    """Its functions may take other arguments than the module passes: the wrappers are called."""
    in_a_process("""
L = axo.library()
addresses = {name: ctypes.cast(getattr(L, name), ctypes.c_void_p).value for name in binding._QUICK}
assert each() == []
assert _calls.bind(addresses, L.axo_version() + 1) is False
assert each() == list(binding._QUICK)
assert _calls.bind(addresses, L.axo_version()) is True
assert each() == []
""")

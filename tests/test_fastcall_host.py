"""The binding's way into the entry points without ctypes (csrc/fastcall.c): what arrives at the C side, which arguments it
leaves to ctypes, that every function of the binding reaches its own entry point with its own arguments on both ways, and that
both answer alike."""
import ctypes
import os
import shutil
import sysconfig

import pytest

from paper_2108_13191_amd import binding

try:
    from paper_2108_13191_amd import _fastcall as fast
except ImportError:
    if os.path.exists(os.path.join(sysconfig.get_paths()["include"], "Python.h")) and any(map(shutil.which, ("gcc", "cc", "amdclang", "clang"))):
        raise                           # it can be built here: a build that lost it is a fault
    pytest.skip("no Python.h or no C compiler: everything goes through ctypes", allow_module_level=True)

I64, VP, CI = ctypes.c_int64, ctypes.c_void_p, ctypes.c_int
PLAIN = [I64, I64, I64, VP, I64, VP, I64, VP, I64, VP]
SIGNATURES = {"plain": PLAIN, "bias_act": PLAIN[:9] + [VP, CI, VP], "workspace": PLAIN[:9] + [VP, I64, VP]}


class Tensor:
    def __init__(self, address):
        self.address = address

    def data_ptr(self):
        if isinstance(self.address, BaseException):
            raise self.address
        return self.address


def recorder(name):
    seen = []
    kind = ctypes.CFUNCTYPE(CI, *SIGNATURES[name])
    f = kind(lambda *a: (seen.append(a), -77)[1])
    return seen, f, ctypes.cast(f, VP).value


@pytest.mark.parametrize("name", SIGNATURES)
def test_arguments_arrive_as_through_ctypes(name):
    seen, f, address = recorder(name)
    base = [3, 5, 7, Tensor(4096), 8, 1 << 47, 9, Tensor(512), 10]
    tails = {"plain": [[None], [Tensor(2**64 - 1)], [77]], "bias_act": [[None, 1, 0], [Tensor(64), -1, 5], [0, 2**32 + 3, None]],
             "workspace": [[None, 0, 0], [Tensor(16), 2**40, 1], [32, -1, None]]}[name]
    for tail in tails:
        for head in (base, [-1, True, 2**31] + base[3:], [2**63, 2**64 + 5, -2**63] + base[3:]):
            args = head + tail
            assert getattr(fast, name)(address, *args) == -77
            got = seen.pop()
            assert f(*[binding._ptr(x) if t is VP else x for x, t in zip(args, SIGNATURES[name])]) == -77
            assert got == seen.pop()


@pytest.mark.parametrize("name", SIGNATURES)
def test_other_arguments_are_left_to_ctypes(name):
    seen, f, address = recorder(name)
    good = [3, 5, 7, Tensor(4096), 8, 256, 9, None, 10] + {"plain": [0], "bias_act": [0, 1, 0], "workspace": [0, 16, 0]}[name]
    call = getattr(fast, name)
    for i, t in enumerate(SIGNATURES[name]):
        for bad in (1.5, "7", object(), Tensor("x"), Tensor(1.0), Tensor(ValueError("no storage"))) + (() if t is VP else (None,)):
            assert call(address, *good[:i], bad, *good[i + 1:]) is NotImplemented
    assert call(address, *good[:-1]) is NotImplemented and call(address, *good, 0) is NotImplemented
    assert call() is NotImplemented
    with pytest.raises(KeyboardInterrupt):
        call(address, *good[:3], Tensor(KeyboardInterrupt()), *good[4:])
    assert not seen


ENTRY_POINTS = {"gemm_f16_f32acc": "plain", "gemm_f16_f16acc": "plain", "gemm_f16_f16acc_static_workspace": "plain",
                "gemm_f16_f32acc_bias_act": "bias_act", "gemm_f16_f16acc_bias_act": "bias_act", "gemm_f16_f16acc_workspace": "workspace"}


@pytest.mark.parametrize("way", ["extension", "ctypes"])
def test_each_function_reaches_its_own_entry_point(monkeypatch, way):
    """Six recorders in the library's place, pairwise different arguments: which recorder got them, in which order."""
    assert (binding._plain, binding._bias_act, binding._workspace) == (fast.plain, fast.bias_act, fast.workspace)
    seen, calls = [], []
    class Library:
        pass
    lib = Library()
    for number, (name, form) in enumerate(ENTRY_POINTS.items()):
        kind = ctypes.CFUNCTYPE(CI, *SIGNATURES[form])
        f = kind(lambda *a, name=name, number=number: (seen.append((name, a)), -100 - number)[1])
        setattr(lib, name, lambda *a, f=f: (calls.append("ctypes"), f(*a))[1])
        setattr(lib, name + "_address", ctypes.cast(f, VP).value)
        setattr(lib, name + "_keep", f)
    monkeypatch.setattr(binding, "load", lambda: lib)
    if way == "ctypes":
        for name in ("_plain", "_bias_act", "_workspace"):
            monkeypatch.setattr(binding, name, binding._no_fast_way)
    for number, (name, form) in enumerate(ENTRY_POINTS.items()):
        args = [101 + i if t is not VP else Tensor(4096 * (i + 1)) for i, t in enumerate(SIGNATURES[form])]
        assert getattr(binding, name)(*args) == -100 - number
        assert seen.pop() == (name, tuple(x.address if isinstance(x, Tensor) else x for x in args)) and not seen
        assert getattr(binding, name)(*args[:-1]) == -100 - number                                  # the stream defaults to 0
        assert seen.pop() == (name, (*(x.address if isinstance(x, Tensor) else x for x in args[:-1]), None)) and not seen
    assert len(calls) == (12 if way == "ctypes" else 0)


def test_addresses_are_those_of_the_library():
    lib = binding.load()
    addresses = {name: getattr(lib, name + "_address") for name in ENTRY_POINTS}
    assert addresses == {name: ctypes.cast(getattr(lib, name), VP).value for name in ENTRY_POINTS} and len(set(addresses.values())) == 6


def test_both_ways_answer_alike(monkeypatch):
    np = pytest.importorskip("numpy")
    calls = [(binding.gemm_f16_f32acc, (0, 4, 4, None, 4, None, 4, None, 4)), (binding.gemm_f16_f32acc, (4, 4, 4, 256, 3, 256, 4, 256, 4)),
             (binding.gemm_f16_f16acc, (-1, 4, 4, 256, 4, 256, 4, 256, 4, None)), (binding.gemm_f16_f16acc, (np.int64(4), 4, 4, 256, 4, None, 4, 256, 4)),
             (binding.gemm_f16_f32acc_bias_act, (4, 4, 4, 256, 4, 256, 4, 256, 4, None, 9)), (binding.gemm_f16_f16acc_bias_act, (4, 4, 4, 256, 4, 256, 4, 256, 4, 257, 1)),
             (binding.gemm_f16_f16acc_workspace, (4, 4, 4, 256, 4, 256, 4, 256, 4, 8, 64)), (binding.gemm_f16_f16acc_static_workspace, (4, 4, 4, 256, 4, 256, 3, 256, 4)),
             (binding.gemm_f16_f32acc, (4.0, 4, 4, 256, 4, 256, 4, 256, 4)), (binding.gemm_f16_f32acc, (4, 4, 4, "x", 4, 256, 4, 256, 4))]

    def answers():
        out = []
        for f, args in calls:
            try:
                out.append(f(*args))
            except Exception as e:
                out.append((type(e), str(e)))
        return out

    here = answers()
    for name in ("_plain", "_bias_act", "_workspace"):
        monkeypatch.setattr(binding, name, binding._no_fast_way)
    assert here == answers()
    assert {binding.OK, binding.ERR_PITCH, binding.ERR_SIZE, binding.ERR_NULL, binding.ERR_CONFIG, binding.ERR_ALIGN} <= set(here)

"""The launching entry points through the extension module: what they convert themselves and what they leave to the Python function
gives the same answers (host only: every call here is refused before a launch)."""
import copy
import ctypes
import inspect
import pickle
import weakref

import pytest

import paper_2603_29010_amd as ucl
from paper_2603_29010_amd import binding

P = 4096                      # an aligned address that nothing reads
NAMES = ["ucl_gemm", "ucl_gemm_static_workspace", "ucl_batched_gemm", "ucl_conv2d_fprop", "ucl_conv2d_dgrad", "ucl_conv2d_wgrad", "ucl_transpose"]
EPI, TUNE = ucl.Epilogue([("relu",)]), ucl.Tuning(1, 2, 3, 4)
# (each refused for two reasons: changing one argument does not make it a call that launches)
BAD = {
    "ucl_gemm": (0, 8, -1, P, "bf16", 8, 1, P, "bf16", 1, 8, P, "f32", 8, 1),
    "ucl_gemm_static_workspace": (0, 8, -1, P, "bf16", 8, 1, P, "bf16", 1, 8, P, "f32", 8, 1),
    "ucl_batched_gemm": (0, 8, -1, 8, P, "bf16", 8, 1, 64, P, "bf16", 1, 8, 64, P, "f32", 8, 1, 64),
    "ucl_conv2d_fprop": (0, 8, 8, -1, 8, 3, 3, 1, 1, 1, 1, 1, 1, P, "bf16", P, "bf16", P, "bf16"),
    "ucl_conv2d_dgrad": (0, 2, 2, -1, 8, 3, 3, 0, 0, 1, 1, 1, 1, P, "bf16", P, "bf16", P, "bf16"),
    "ucl_conv2d_wgrad": (0, 8, 8, -1, 8, 3, 3, 1, 1, 1, 1, 1, 1, P, "bf16", P, "bf16", P, "bf16"),
    "ucl_transpose": (-1, -1, 8, P, "f32", P, "bf16"),
}


def outcome(f, *a, **k):
    try:
        return f(*a, **k)
    except ucl.UclError as e:
        return (e.status, e.message)
    except Exception as e:          # a bad argument: the kind of error
        return type(e)


def test_the_module_is_built():
    assert binding._calls is not None and all(isinstance(getattr(ucl, n), binding._calls.Call) for n in NAMES)


@pytest.mark.parametrize("name", NAMES)
def test_same_as_the_python_function(name):
    ucl.ucl_version()
    native, python, bad = getattr(ucl, name), getattr(ucl, name).__wrapped__, BAD[name]
    assert inspect.signature(native) == inspect.signature(python) and native.__name__ == name
    tail = () if name == "ucl_transpose" else (EPI, TUNE)
    variants = [bad, bad + tail, bad + tail + (0,), bad + tail + (None,), bad[:-1], bad + tail + (0, 0), bad + tuple(None for _ in tail) + (16,)]
    for i, v in enumerate(bad):
        for other in (None, 1 << 70, -1, 2.5, "x", "f16", ctypes.c_int64(3), True, b"f16"):
            if isinstance(v, int) and v == P and other in (1 << 70, -1, True):
                continue                                    # (addresses: the refusal must come before anything could be read there)
            variants.append(bad[:i] + (other,) + bad[i + 1:])
    if tail:
        variants += [bad + (TUNE, EPI), bad + (EPI.c,), bad + (EPI, 3)]
    for args in variants:
        first = outcome(native, *args)
        assert first == outcome(python, *args), args
        assert first is not None, args
    assert outcome(native, *bad, stream=0) == outcome(python, *bad, stream=0)
    assert outcome(native, *bad, nonsense=0) is TypeError


@pytest.mark.parametrize("name", NAMES + ["ucl_grouped_gemm"])
def test_programs_may_treat_them_as_the_functions_they_were(name):
    f = getattr(ucl, name)
    assert pickle.loads(pickle.dumps(f)) is f and pickle.loads(pickle.dumps({"call": f}, protocol=2))["call"] is f
    assert copy.copy(f) is f and copy.deepcopy([f])[0] is f and weakref.ref(f)() is f
    python = getattr(f, "__wrapped__", f)
    assert f.__defaults__ == python.__defaults__ and f.__defaults__[-1] == 0
    assert f.__code__ is python.__code__ and f.__kwdefaults__ is None and f.__qualname__ == name and f.__module__ == binding.__name__
    assert not hasattr(f, "nothing_of_that_name")

    class Holder:
        call = f
    assert Holder.call is f and Holder().call.__self__.__class__ is Holder
    f.noted = 3
    assert f.noted == 3
    del f.noted


def test_the_structures_are_passed_through():
    # refused for what stands in the chain and in the tuning
    with pytest.raises(ucl.UclError, match="clamp"):
        ucl.ucl_gemm(8, 8, 8, P, "bf16", 8, 1, P, "bf16", 1, 8, P, "f32", 8, 1, ucl.Epilogue([("clamp", 2.0, 1.0)]))
    with pytest.raises(ucl.UclError, match="tile_k=3"):
        ucl.ucl_gemm(8, 8, 8, P, "bf16", 8, 1, P, "bf16", 1, 8, P, "f32", 8, 1, None, TUNE)

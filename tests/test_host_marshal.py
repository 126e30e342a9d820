"""The native half of the binding against the ctypes half: the addresses and values that reach the C functions (callbacks that
write them down, no GPU), and the forms that it leaves to ctypes."""
import ctypes
import os
import sys

import pytest
import torch

import paper_2505_10183_amd as kt

vp, f32, i32 = ctypes.c_void_p, ctypes.c_float, ctypes.c_int
PP, FP = ctypes.POINTER(vp), ctypes.POINTER(f32)
T, NB = 3, 2
SIGNATURES = {      # argument types after (plan, bucket); "T", "N", "P", "Q": arrays of T, NB, NB * K, NB * (K - 1) addresses
    "pack": "TNs", "reduce": "PKwNs", "unpack": "NfTs", "fused": "TQKwfTs", "sgd": "NfTTfffis", "master": "NfTTTfffis",
    "fused_sgd": "TQKwfTTTfffis",
}
CTYPE = {"T": PP, "N": PP, "P": PP, "Q": PP, "K": i32, "w": FP, "f": f32, "i": i32, "s": vp}


@pytest.fixture(scope="module")
def native():
    kt.binding.lib()
    assert os.path.exists(kt.binding.MARSHAL_PATH), "run __graft_entry__.build()"
    kt.binding._native()
    seen, keep = [], []

    def recorder(name):
        codes = SIGNATURES[name]

        def f(plan, bucket, *args):
            K = args[codes.index("K")] if "K" in codes else 0
            size = {"T": T, "N": NB, "P": NB * K, "Q": NB * (K - 1), "w": K}
            seen.append((name, plan, bucket) + tuple([a[i] for i in range(size[c])] if c in size and a else (a or 0) for c, a in zip(codes, args)))
            return 0
        keep.append(ctypes.CFUNCTYPE(i32, vp, i32, *[CTYPE[c] for c in codes])(f))
        return ctypes.cast(keep[-1], vp).value

    calls = type(kt.binding._calls)(*[recorder(n) for n in SIGNATURES])
    return calls, seen, keep


def tensors(n):
    return [torch.zeros(5)[1:] for _ in range(n)]


def arguments(name, K, form):
    """Arguments in the order of the native call, and what has to arrive."""
    got, want, k_at = [], [], None
    for c in SIGNATURES[name]:
        if c in "TNPQ":
            l = tensors({"T": T, "N": NB, "P": NB * K, "Q": NB * (K - 1)}[c])
            want.append([t.data_ptr() for t in l])
            got.append(kt.binding._ptr_array(l) if form == "marshalled" else tuple(l) if form == "tuple" else l)
            arguments.keep.append(l)
        elif c == "K":
            want.append(K)
        elif c == "w":
            l = [0.5 / (k + 1) for k in range(K)]
            want.append([f32(x).value for x in l])
            got.append((f32 * K)(*l) if form == "marshalled" else l)
        elif c == "f":
            want.append(f32(0.1).value)
            got.append(0.1)
        elif c == "i":
            want.append(1)
            got.append(True)
        else:
            want.append(77)
            got.append(77)
    return ([K] if "K" in SIGNATURES[name] else []) + got, want


arguments.keep = []


@pytest.mark.parametrize("form", ["list", "tuple", "marshalled"])
@pytest.mark.parametrize("K", [1, 2, 64])
@pytest.mark.parametrize("name", list(SIGNATURES))
def test_what_arrives(native, name, K, form):
    calls, seen, _ = native
    args, want = arguments(name, K, form)
    if K == 1 and "Q" in SIGNATURES[name]:      # no peers: an array of one unused entry
        want[SIGNATURES[name].index("Q")] = []
    del seen[:]
    assert getattr(calls, name)(1234, T, NB, -1, *args) == 0
    assert seen == [(name, 1234, -1) + tuple(want)]


class Sub(torch.Tensor):
    pass


@pytest.mark.parametrize("tens,bufs,bucket", [
    ("short", "list", 0), ("long", "list", 0), ("list", "short", 0), ("ints", "list", 0), ("none", "list", 0), ("subclass", "list", 0),
    ("generator", "list", 0), ("longs", "list", 0), ("floats", "list", 0), ("list", "list", 1 << 40), ("list", "list", 1.0), ("sparse", "list", 0),
])
def test_what_is_left_to_ctypes(native, tens, bufs, bucket):
    calls, seen, _ = native

    def make(form, n):
        l = tensors(n)
        arguments.keep.append(l)
        return {"list": l, "short": l[:-1], "long": l + l[:1], "ints": [t.data_ptr() for t in l], "none": l[:-1] + [None],
                "subclass": [t.as_subclass(Sub) for t in l], "generator": (t for t in l), "longs": (ctypes.c_int64 * n)(),
                "floats": (f32 * n)(), "sparse": [torch.zeros(2, 2).to_sparse()] * n}[form]

    del seen[:]
    assert calls.pack(1, T, NB, bucket, make(tens, T), make(bufs, NB), 0) is None
    assert seen == []


def test_a_function_mode_sees_the_calls(native):
    calls, seen, _ = native

    class Mode(torch.overrides.TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))

    l, b = tensors(T), tensors(NB)
    del seen[:]
    with Mode():
        assert calls.pack(1, T, NB, 0, l, b, 0) is None
    assert seen == [] and calls.pack(1, T, NB, 0, l, b, 0) == 0


def test_weights_none_and_no_model_copy(native):
    calls, seen, _ = native
    del seen[:]
    assert calls.reduce(1, T, NB, 0, 2, tensors(4), None, tensors(2), 0) == 0
    assert calls.fused_sgd(1, T, NB, 0, 1, tensors(T), [], [1.0], 1.0, tensors(T), tensors(T), None, 0.1, 0.9, 0.0, False, 0) == 0
    assert seen[0][5] == 0 and seen[1][10] == 0


def test_references_are_left_as_they_were(native):
    calls, _, _ = native
    l, b = tensors(T), tensors(NB)
    a = kt.binding._ptr_array(l)
    before = [sys.getrefcount(x) for x in (l, b, a, *l, *b)]
    for _ in range(50):
        calls.pack(1, T, NB, 0, l, b, 0)
        calls.pack(1, T, NB, 0, a, b, 0)
        calls.pack(1, T, NB, 0, a, l, 0)
    assert [sys.getrefcount(x) for x in (l, b, a, *l, *b)] == before

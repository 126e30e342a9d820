"""The native half of the binding against the ctypes half: the addresses and values that reach the C functions (callbacks that
write them down, no GPU), and the forms that it leaves to ctypes."""
import ctypes
import os
import sys

import numpy as np
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


def arguments(name, K, form, first=True):
    """Arguments in the order of the native call, no two alike, and what has to arrive."""
    got, want, reals = [], [], iter([0.1, -0.2, 3.0, 0.4])
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
            got.append(next(reals))
            want.append(f32(got[-1]).value)
        elif c == "i":
            want.append(int(first))
            got.append(first)
        else:
            want.append(77)
            got.append(77)
    return ([K] if "K" in SIGNATURES[name] else []) + got, want


arguments.keep = []


@pytest.mark.parametrize("form", ["list", "tuple", "marshalled"])
@pytest.mark.parametrize("K,bucket,first", [(1, -1, True), (2, 1, False), (64, 0, True)])
@pytest.mark.parametrize("name", list(SIGNATURES))
def test_what_arrives(native, name, K, bucket, first, form):
    calls, seen, _ = native
    args, want = arguments(name, K, form, first)
    if K == 1 and "Q" in SIGNATURES[name]:      # no peers: an array of one unused entry
        want[SIGNATURES[name].index("Q")] = []
    del seen[:]
    assert getattr(calls, name)(1234, T, NB, bucket, *args) == 0
    assert seen == [(name, 1234, bucket) + tuple(want)]


class Undecided:
    def __bool__(self):
        raise ValueError


REFUSED = {
    "K": [0, 65, -1, 2.0, "2", None, 1 << 40], "w": [[0.5], [0.5] * 3, [0.5, "x"], (vp * 2)(), (f32 * 3)(), 0.5, (x for x in (0.5, 0.5))],
    "f": ["x", None, 1j, [0.1], 10 ** 400], "i": [Undecided(), torch.zeros(2)], "s": ["x", 1.0, object(), 1 << 80],
    **{c: [[], None, 7, (f32 * 6)(), torch.zeros(6)] for c in "TNPQ"},
}


@pytest.mark.parametrize("name,at", [(n, i) for n, codes in SIGNATURES.items() for i in range(len(codes))])
def test_what_every_call_refuses(native, name, at):
    """One argument at a time in a form that is not taken: no call is made."""
    calls, seen, _ = native
    code = SIGNATURES[name][at]
    bad = list(REFUSED[code])
    size = {"T": T, "N": NB, "P": 2 * NB, "Q": NB}.get(code)
    if size:
        l = tensors(size)
        arguments.keep.append(l)
        bad += [l[:-1], l + l[:1], l[:-1] + [l[-1].data_ptr()], l[:-1] + [None], [l[0].as_subclass(Sub)] + l[1:], (vp * (size + 1))()]
        if name == "fused_sgd" and at == SIGNATURES[name].rindex("T"):
            bad.remove(None)            # no model copy
    elif code == "w":
        bad = [b for b in bad if b is not None]
    for value in bad:
        args, _ = arguments(name, 2, "list")
        places = [i for i, c in enumerate(SIGNATURES[name]) if c != "K"] if "K" in SIGNATURES[name] else list(range(len(SIGNATURES[name])))
        where = 0 if code == "K" else places.index(at) + ("K" in SIGNATURES[name])
        args[where] = value
        del seen[:]
        assert getattr(calls, name)(1, T, NB, 0, *args) is None, (name, at, value)
        assert seen == []
    for bucket in (1 << 40, 1.0, "0", None):
        assert getattr(calls, name)(1, T, NB, bucket, *arguments(name, 2, "list")[0]) is None and seen == []


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


class Stream:
    cuda_stream = 91


class Real:
    """float(x), which makes calls of its own meanwhile."""

    def __init__(self, value, then):
        self.value, self.then = value, then

    def __float__(self):
        self.then()
        return self.value


def sgd(calls, lr=0.1, first=True, stream=0):
    return calls.sgd(1, T, NB, 0, tensors(NB), 1.0, tensors(T), tensors(T), lr, 0.9, 0.0, first, stream)


@pytest.mark.parametrize("stream,want", [(Stream(), 91), (77, 77), (True, 1)])
def test_streams(native, stream, want):
    calls, seen, _ = native
    del seen[:]
    assert calls.pack(1, T, NB, 0, tensors(T), tensors(NB), stream) == 0 and sgd(calls, stream=stream) == 0
    assert seen[0][-1] == want and seen[1][-1] == want


@pytest.mark.parametrize("weights", [[1, 2], (1, 2.0), np.array([1, 2]), np.array([1, 2], "f4"), torch.tensor([1.0, 2.0]), [True, np.float32(2)],
                                     {1: 0, 2: 0}, [Real(1.0, lambda: None), 2]])
def test_weights(native, weights):
    calls, seen, _ = native
    del seen[:]
    assert calls.reduce(1, T, NB, 0, 2, tensors(2 * NB), weights, tensors(NB), 0) == 0
    assert calls.fused(1, T, NB, 0, np.int64(2), tensors(T), tensors(NB), weights, 1.0, tensors(T), 0) == 0
    assert seen[0][5] == [1.0, 2.0] and seen[1][6] == [1.0, 2.0] and seen[0][4] == seen[1][5] == 2


@pytest.mark.parametrize("value,want", [(3, 3.0), (True, 1.0), (np.float64(0.1), 0.1), (np.float32(0.5), 0.5), (np.int32(2), 2.0), (torch.tensor(0.25), 0.25),
                                        (1e300, float("inf"))])
def test_scalars(native, value, want):
    calls, seen, _ = native
    del seen[:]
    assert sgd(calls, lr=value) == 0 and seen[0][7] == f32(want).value


@pytest.mark.parametrize("value,want", [(True, 1), (False, 0), (0, 0), (1, 1), (7, 1), (np.bool_(True), 1), (None, 0), ("", 0), (torch.tensor(True), 1)])
def test_flags(native, value, want):
    calls, seen, _ = native
    del seen[:]
    assert sgd(calls, first=value) == 0 and seen[0][10] == want


def test_calls_made_while_another_one_is_marshalled(native):
    calls, seen, _ = native
    other = tensors(T)
    mine, momenta, bufs = tensors(T), tensors(T), tensors(NB)
    inner = lambda: calls.fused_sgd(1, T, NB, 0, 1, other, [], [1.0], 1.0, other, other, other, 0.1, 0.9, 0.0, True, 0)
    del seen[:]
    assert calls.sgd(1, T, NB, 0, bufs, Real(0.5, inner), mine, momenta, Real(0.1, inner), Real(0.9, inner), 0.0, True, 0) == 0
    assert [s[0] for s in seen] == ["fused_sgd"] * 3 + ["sgd"]
    assert seen[3][3:7] == ([t.data_ptr() for t in bufs], 0.5, [t.data_ptr() for t in mine], [t.data_ptr() for t in momenta])


def test_weights_that_change_while_they_are_read(native):
    calls, seen, _ = native
    w = []
    w += [Real(0.5, w.clear), Real(0.25, w.clear)]
    del seen[:]
    assert calls.reduce(1, T, NB, 0, 2, tensors(2 * NB), w, tensors(NB), 0) == 0
    assert seen[0][5] == [0.5, 0.25]

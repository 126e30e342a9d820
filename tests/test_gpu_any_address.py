"""Tensors and buckets at every kind of element address: a full tile's vectors are laid out from a
64-byte boundary of the destination, so the byte offset of the destination from that boundary (0 to
62) decides which vector wraps to the tile's end and which elements go one by one.  Every element
against the CPU checker's binary32 step mode (bit-identical), with guard elements around every output."""
import sys

import numpy as np
import pytest
import torch

import oracle
import paper_2505_10183_amd as kt
from paper_2505_10183_amd import workloads as wl
from test_gpu_parity import DEV, host, raw, tdtype

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def announce(request):
    print("\n[gpu-case] %s" % request.node.nodeid, file=sys.stderr, flush=True)
    yield
    torch.cuda.synchronize()


GUARD = 64


class Guarded:
    """Views of n elements each that start `shift` bytes past a 64-byte boundary, between guard elements."""

    def __init__(self, sizes, dtype, shift, fill):
        es = torch.empty((), dtype=dtype).element_size()
        assert shift % es == 0
        self.fill = fill
        self.at = GUARD + shift // es       # the allocator's blocks start on 512-byte boundaries
        self.whole = [torch.full((n + self.at + GUARD,), fill, dtype=dtype, device=DEV) for n in sizes]
        self.views = [t[self.at:self.at + n] for t, n in zip(self.whole, sizes)]

    def check_guards(self, what):
        for i, (t, v) in enumerate(zip(self.whole, self.views)):
            assert bool((t[:self.at] == self.fill).all()) and bool((t[self.at + v.numel():] == self.fill).all()), (what, i)


def same(got, want, what):
    for t, (a, b) in enumerate(zip(got, want)):
        assert raw(host(a)).tobytes() == raw(b).tobytes(), (what, t)


def case(dtype, align, K):
    es = 4 if dtype == "f32" else 2
    tile = 16384 // es
    # several full tiles from an odd start, one element, a tile and its neighbours, a short last tile
    numels = [5, 3 * tile + 7, 1, tile, tile - 1, tile + 1, 2 * tile, 9, 4097, 2 * tile + 333]
    w = wl.Workload("any", dtype, tuple((n,) for n in numels), tuple(1.0 - 0.04 * k for k in range(K)), 1024,
                    7 * 16384, 1e-3, 77)
    plan = kt.Plan(numels, dtype, w.bucket_cap_bytes, align)
    layout = oracle.assign_buckets(numels, es, w.bucket_cap_bytes, align)
    shares, weights = kt.kt_plan_shares(w.throughputs, w.global_batch)
    return w, plan, layout, weights, oracle.share_weights(shares, w.global_batch)


@pytest.mark.parametrize("dtype,shift", [("f32", s) for s in (0, 4, 12, 16, 36, 48, 60)] +
                         [("bf16", s) for s in (0, 2, 14, 16, 34, 48, 62)])
@pytest.mark.parametrize("dense", [True, False])
def test_pack_unpack(dtype, shift, dense):
    w, plan, layout, _, _ = case(dtype, (4 if dtype == "f32" else 2) if dense else 16, 1)
    td = tdtype(dtype)
    grads = Guarded(w.numels, td, shift, 3.0)
    for v, g in zip(grads.views, wl.gradient_set(w, 0, DEV)):
        v.copy_(g.reshape(-1))
    hg = [host(v) for v in grads.views]
    want = oracle.pack(layout, hg, dtype)
    for bshift in (0, 64 - shift if shift else 32):
        buckets = Guarded(plan.bucket_elems(), td, bshift, 5.0)
        out = Guarded(w.numels, td, shift, 7.0)
        plan.kt_bucket_pack(-1, grads.views, buckets.views)
        plan.kt_bucket_unpack_scale(-1, buckets.views, 0.37, out.views)
        torch.cuda.synchronize()
        same(buckets.views, want, "pack")
        same(out.views, oracle.unpack_scale(layout, want, w.numels, 0.37, dtype, "S"), "unpack")
        buckets.check_guards("pack")
        out.check_guards("unpack")


@pytest.mark.parametrize("dtype,shift", [("f32", s) for s in (0, 4, 12, 16, 36, 48, 60)] +
                         [("bf16", s) for s in (0, 2, 14, 16, 34, 48, 62)])
@pytest.mark.parametrize("K", [1, 3, 8, 11])
def test_reduce(dtype, shift, K):
    w, plan, layout, weights, wts = case(dtype, 4 if dtype == "f32" else 2, K)
    nb = plan.num_buckets
    td = tdtype(dtype)
    # every copy at another address, then the output beside them and over the first copy
    peers = [Guarded(plan.bucket_elems(), td, (shift + 4 * k) % 64, 3.0) for k in range(K)]
    for k in range(K):
        for b, v in enumerate(peers[k].views):
            v.copy_(wl.flat_normal(v.numel(), dtype, 1e-3, 100 * k + b, DEV))
    want = [oracle.weighted_reduce([host(peers[k].views[b]) for k in range(K)], wts, dtype, "S") for b in range(nb)]
    flat = [peers[k].views[b] for b in range(nb) for k in range(K)]
    out = Guarded(plan.bucket_elems(), td, (64 - shift) % 64, 5.0)
    plan.kt_weighted_reduce(-1, flat, K, weights, out.views)
    plan.kt_weighted_reduce(-1, flat, K, weights, peers[0].views)
    torch.cuda.synchronize()
    for dst in (out, peers[0]):
        same(dst.views, want, "reduce")
        dst.check_guards("reduce")


@pytest.mark.parametrize("dtype,shift", [("f32", s) for s in (0, 4, 12, 16, 36, 48, 60)] +
                         [("bf16", s) for s in (0, 2, 14, 16, 34, 48, 62)])
@pytest.mark.parametrize("K,dense", [(1, True), (4, True), (8, False), (8, True), (11, True)])
def test_fused(dtype, shift, K, dense):
    w, plan, layout, weights, wts = case(dtype, (4 if dtype == "f32" else 2) if dense else 16, K)
    nb = plan.num_buckets
    td = tdtype(dtype)
    sets = [wl.gradient_set(w, k, DEV) for k in range(K)]
    grads = Guarded(w.numels, td, shift, 3.0)
    for v, g in zip(grads.views, sets[0]):
        v.copy_(g.reshape(-1))
    hg = [[host(t.reshape(-1)) for t in s] for s in sets]
    peers = [Guarded(plan.bucket_elems(), td, (shift + 4 * k) % 64, 5.0) for k in range(1, K)]
    for k in range(1, K):
        plan.kt_bucket_pack(-1, sets[k], peers[k - 1].views)
    flat = [peers[k - 1].views[b] for b in range(nb) for k in range(1, K)]
    want = oracle.direct(hg, wts, 0.37, dtype, "S")
    out = Guarded(w.numels, td, (64 - shift) % 64, 7.0)
    plan.kt_fused_step(-1, grads.views, flat, K, weights, 0.37, out.views)
    plan.kt_fused_step(-1, grads.views, flat, K, weights, 0.37, grads.views)     # over the local gradients
    torch.cuda.synchronize()
    for dst in (out, grads):
        same(dst.views, want, "fused")
        dst.check_guards("fused")


@pytest.mark.parametrize("dtype,shift", [("f32", s) for s in (0, 4, 12, 16, 36, 48, 60)] +
                         [("bf16", s) for s in (0, 4, 12, 16, 36, 48, 60)])
@pytest.mark.parametrize("K,dense,master", [(1, True, False), (4, True, True), (8, False, True), (8, True, False), (11, True, True)])
def test_fused_sgd(dtype, shift, K, dense, master):
    w, plan, layout, weights, wts = case(dtype, (4 if dtype == "f32" else 2) if dense else 16, K)
    nb = plan.num_buckets
    td = tdtype(dtype)
    sets = [wl.gradient_set(w, k, DEV) for k in range(K)]
    grads = Guarded(w.numels, td, shift, 3.0)
    for v, g in zip(grads.views, sets[0]):
        v.copy_(g.reshape(-1))
    peers = [Guarded(plan.bucket_elems(), td, (shift + 4 * k) % 64, 5.0) for k in range(1, K)]
    for k in range(1, K):
        plan.kt_bucket_pack(-1, sets[k], peers[k - 1].views)
    flat = [peers[k - 1].views[b] for b in range(nb) for k in range(1, K)]
    p, v = Guarded(w.numels, torch.float32, (64 - shift) % 64, 7.0), Guarded(w.numels, torch.float32, shift, 9.0)
    m = Guarded(w.numels, torch.bfloat16, shift // 2, 11.0)
    for t in range(len(w.numels)):
        p.views[t].copy_(wl.flat_normal(w.numels[t], "f32", 1.0, 300 + t, DEV))
        v.views[t].fill_(float("nan"))          # a first step does not use the momentum
    hp, hv = [host(t) for t in p.views], [host(t) for t in v.views]
    hb = [oracle.weighted_reduce([oracle.pack(layout, [host(t.reshape(-1)) for t in s], dtype)[b] for s in sets], wts, dtype, "S")
          for b in range(nb)]
    for step in range(2):
        plan.kt_fused_step_sgd(-1, grads.views, flat, K, weights, 0.37, p.views, v.views, m.views if master else None,
                               0.1, 0.9, 5e-4, step == 0)
        torch.cuda.synchronize()
        hp, hv = oracle.unpack_sgd(layout, hb, w.numels, 0.37, hp, hv, 0.1, 0.9, 5e-4, step == 0, dtype, "S")
        same(p.views, hp, "p")
        same(v.views, hv, "v")
        for t in range(len(w.numels)):
            if master:
                assert bool((m.views[t] == p.views[t].bfloat16()).all()), ("model", step, t)
    for g, what in ((p, "p"), (v, "v"), (m, "model")):
        g.check_guards(what)


@pytest.mark.parametrize("dtype,shift", [("f32", s) for s in (0, 4, 12, 16, 36, 48, 60)] +
                         [("bf16", s) for s in (0, 4, 12, 16, 36, 48, 60)])
@pytest.mark.parametrize("dense,master", [(True, False), (True, True), (False, True)])
def test_unpack_sgd(dtype, shift, dense, master):
    w, plan, layout, _, _ = case(dtype, (4 if dtype == "f32" else 2) if dense else 16, 1)
    buckets = Guarded(plan.bucket_elems(), tdtype(dtype), (shift + 4) % 64, 5.0)
    for b, t in enumerate(buckets.views):
        t.copy_(wl.flat_normal(t.numel(), dtype, 1e-3, 500 + b, DEV))
    p, v = Guarded(w.numels, torch.float32, shift, 7.0), Guarded(w.numels, torch.float32, (shift if dense else 8), 9.0)
    m = Guarded(w.numels, torch.bfloat16, shift // 2, 11.0)
    for t in range(len(w.numels)):
        p.views[t].copy_(wl.flat_normal(w.numels[t], "f32", 1.0, 300 + t, DEV))
        v.views[t].fill_(float("nan"))          # a first step does not use the momentum
    hp, hv, hb = [host(t) for t in p.views], [host(t) for t in v.views], [host(t) for t in buckets.views]
    for step in range(2):
        if master:
            plan.kt_bucket_unpack_sgd_master(-1, buckets.views, 0.37, p.views, v.views, m.views, 0.1, 0.9, 5e-4, step == 0)
        else:
            plan.kt_bucket_unpack_sgd(-1, buckets.views, 0.37, p.views, v.views, 0.1, 0.9, 5e-4, step == 0)
        torch.cuda.synchronize()
        hp, hv = oracle.unpack_sgd(layout, hb, w.numels, 0.37, hp, hv, 0.1, 0.9, 5e-4, step == 0, dtype, "S")
        same(p.views, hp, "p")
        same(v.views, hv, "v")
        for t in range(len(w.numels)):
            if master:
                assert bool((m.views[t] == p.views[t].bfloat16()).all()), ("model", step, t)
    for g, what in ((p, "p"), (v, "v"), (m, "model")):
        g.check_guards(what)

"""Tiles that hold 1 to 6 tensors (the table of up to 4 goes to registers in SGD on unpack of bf16 gradients): large
tensors with a few small and empty ones between them, at 64-byte and other addresses; every kernel, every element."""
import sys

import pytest
import torch

import paper_2505_10183_amd as kt
from paper_2505_10183_amd import workloads as wl
from test_gpu_any_address import Guarded
from test_gpu_large_any_address import LR, MU, SCALE, WD, every_kernel
from test_gpu_parity import DEV

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def announce(request):
    print("\n[gpu-case] %s" % request.node.nodeid, file=sys.stderr, flush=True)
    yield
    torch.cuda.synchronize()
    torch.cuda.empty_cache()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shift,dense", [(0, False), (32, False), (4, True), (36, True)])
@pytest.mark.parametrize("small", [(), (0,), (1,), (9, 4), (64, 3, 1), (0, 0, 7, 5), (1, 2, 3, 4, 5)])
def test_few_tensors_in_a_tile(dtype, small, shift, dense):
    numels = []
    for large in (20000, 8192, 8200, 30011, 4096, 17, 9001):
        numels += [large, *small]
    every_kernel(numels, dtype, 0, 3, shift, dense)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shift,dense", [(0, False), (32, False), (4, True)])
@pytest.mark.parametrize("large,small", [(9001, (1,)), (20000, (0, 0, 7, 5)), (8192, (1, 2, 3, 4, 5)), (3000001, (9, 4)), (3000064, ())])
def test_sgd_without_the_model_copy(dtype, large, small, shift, dense):
    """Parameters and momentum of SGD on unpack: the bits of the form with the model copy, which every_kernel compares
    with the CPU checker; the large ones hold workgroups per CU."""
    es = 4 if dtype == "f32" else 2
    numels = [n for i in range(12) for n in (large + i, *small)]
    plan = kt.Plan(numels, dtype, 25 << 20, es if dense else 16)
    buckets = [wl.flat_normal(n, dtype, 1e-3, 50 + b, DEV) for b, n in enumerate(plan.bucket_elems())]
    sets = []
    for master in (False, True):
        p, v = Guarded(numels, torch.float32, shift, 3.0), Guarded(numels, torch.float32, (shift + 16) % 64, 5.0)
        for t, n in enumerate(numels):
            p.views[t].copy_(wl.flat_normal(max(n, 1), "f32", 1.0, 300 + t, DEV)[:n])
            v.views[t].copy_(wl.flat_normal(max(n, 1), "f32", 0.1, 900 + t, DEV)[:n])
        if master:
            m = Guarded(numels, torch.bfloat16, shift // 2, 7.0)
            plan.kt_bucket_unpack_sgd_master(-1, buckets, SCALE, p.views, v.views, m.views, LR, MU, WD, False)
        else:
            plan.kt_bucket_unpack_sgd(-1, buckets, SCALE, p.views, v.views, LR, MU, WD, False)
        sets.append((p, v))
    torch.cuda.synchronize()
    for (a, b), what in zip(zip(*sets), ("p", "v")):
        a.check_guards(what)
        for t, (x, y) in enumerate(zip(a.views, b.views)):
            assert torch.equal(x.view(torch.int32), y.view(torch.int32)), (what, t)

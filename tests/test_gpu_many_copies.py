"""9 and more copies: quarter tiles, whole ones and store windows at the limits that choose them, every number
of copies left for the last chunk, device-resident weights; every kernel, every element, odd tensor sizes."""
import sys

import pytest
import torch

import paper_2505_10183_amd as kt
from test_gpu_large_any_address import every_kernel

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def announce(request):
    print("\n[gpu-case] %s" % request.node.nodeid, file=sys.stderr, flush=True)
    yield
    torch.cuda.synchronize()
    torch.cuda.empty_cache()


@pytest.mark.parametrize("dtype,tiles,K,shift,dense", [
    ("f32", 5, 9, 0, False), ("bf16", 20, 10, 4, True), ("f32", 30, 11, 36, True), ("bf16", 30, 12, 0, False),
    ("f32", 20, 13, 4, False), ("bf16", 5, 14, 12, True), ("f32", 30, 15, 0, True), ("bf16", 20, 16, 60, False),
    ("f32", 20, 17, 0, False), ("bf16", 30, 23, 4, True), ("f32", 30, 24, 4, True),
    ("f32", 255, 9, 0, False), ("bf16", 258, 16, 36, True), ("f32", 600, 12, 4, True), ("bf16", 700, 11, 0, False),
    ("f32", 896, 12, 60, False), ("f32", 1152, 10, 4, True), ("bf16", 1152, 13, 0, False),
    ("f32", 2560, 16, 4, True), ("bf16", 2560, 9, 20, False),
    # inside the store windows: the fused pass and the one-pass SGD, with 24 copies the reduce as well
    ("f32", 8937, 11, 0, False), ("bf16", 12288, 16, 4, True), ("f32", 10923, 24, 36, True), ("bf16", 10923, 24, 0, False),
])
def test_tiles_of_many_copies(dtype, tiles, K, shift, dense):
    n = -(-tiles * (16384 // (4 if dtype == "f32" else 2)) // 24) | 1
    plan = every_kernel([n + 2 * t for t in range(24)], dtype, 0 if tiles < 2000 else 64 << 20, K, shift, dense)
    assert plan.num_tiles >= tiles


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("K", [9, 16, 21, 64])
def test_zeros_keep_their_signs(dtype, K):
    """The sum starts with the product of the first copy: -0 where all products are -0, +0 otherwise; and weights
    from device memory give the same bits."""
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    n = 8192 * 3 + 5
    plan = kt.Plan([n], dtype, 0, 16)
    m = plan.bucket_elems()[0]
    x = [torch.full((m,), -0.0, dtype=td, device="cuda") for _ in range(K)]
    x[K - 1][1::2] = 0.0
    out, out_dev = torch.ones(m, dtype=td, device="cuda"), torch.ones(m, dtype=td, device="cuda")
    w = [1.0 / K] * K
    plan.kt_weighted_reduce(-1, x, K, w, [out])
    plan.kt_plan_set_weights(w)
    plan.kt_weighted_reduce(-1, x, K, None, [out_dev])
    torch.cuda.synchronize()
    assert bool(torch.signbit(out[0::2]).all()) and not bool(torch.signbit(out[1::2]).any())
    assert bool((out == 0).all()) and bool((torch.signbit(out) == torch.signbit(out_dev)).all())


@pytest.mark.parametrize("dtype,tiles,K", [("f32", 20, 12), ("bf16", 700, 16), ("f32", 2560, 9), ("bf16", 2560, 16), ("f32", 8937, 11),
                                           ("bf16", 551, 6), ("f32", 4096, 8)])
def test_resident_weights(dtype, tiles, K):
    """Weights and optimizer scalars from device memory: the bits of the same calls by value, in shared tiles, in whole
    ones and inside the store windows."""
    td, es = (torch.float32, 4) if dtype == "f32" else (torch.bfloat16, 2)
    n = -(-tiles * (16384 // es) // 24) | 1
    numels = [n + 2 * t for t in range(24)]
    plan = kt.Plan(numels, dtype, 0 if tiles < 2000 else 64 << 20, 16)
    elems, nb = plan.bucket_elems(), plan.num_buckets
    _, weights = kt.kt_plan_shares([1.0 - 0.01 * k for k in range(K)], 4096)
    gen = torch.Generator("cuda").manual_seed(5)
    copies = [[torch.empty(m, dtype=td, device="cuda").normal_(0, 1e-3, generator=gen) for m in elems] for _ in range(K)]
    grads = [torch.empty(m, dtype=td, device="cuda").normal_(0, 1e-3, generator=gen) for m in numels]
    p0 = [torch.empty(m, device="cuda").normal_(0, 1, generator=gen) for m in numels]
    flat = [copies[k][b] for b in range(nb) for k in range(K)]
    others = [copies[k][b] for b in range(nb) for k in range(1, K)]
    plan.kt_plan_set_weights(weights)
    plan.kt_plan_set_sgd(0.37, 0.1, 0.9, 5e-4)
    got = []
    for resident in (False, True):
        red, out = [torch.zeros(m, dtype=td, device="cuda") for m in elems], [torch.zeros_like(g) for g in grads]
        p, v, m = [t.clone() for t in p0], [t * 0.1 for t in p0], [torch.zeros(t.numel(), dtype=torch.bfloat16, device="cuda") for t in p0]
        plan.kt_weighted_reduce(-1, flat, K, None if resident else weights, red)
        plan.kt_fused_step(-1, grads, others, K, None if resident else weights, 0.37, out)
        if resident:
            plan.kt_fused_step_sgd_resident(-1, grads, others, K, p, v, m, False)
        else:
            plan.kt_fused_step_sgd(-1, grads, others, K, weights, 0.37, p, v, m, 0.1, 0.9, 5e-4, False)
        torch.cuda.synchronize()
        got.append([*red, *out, *p, *v, *m])
    for i, (a, b) in enumerate(zip(*got)):
        kind = torch.int32 if a.element_size() == 4 else torch.int16
        assert torch.equal(a.view(kind), b.view(kind)), i

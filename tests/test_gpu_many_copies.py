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

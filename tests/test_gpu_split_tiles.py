"""Launches whose tiles are shared by several workgroups, at the limits of the rules that choose it (and below
them): every kernel, every element, with tensors of odd sizes away from 64-byte boundaries."""
import sys

import pytest
import torch

from test_gpu_large_any_address import every_kernel

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def announce(request):
    print("\n[gpu-case] %s" % request.node.nodeid, file=sys.stderr, flush=True)
    yield
    torch.cuda.synchronize()
    torch.cuda.empty_cache()


@pytest.mark.parametrize("dtype,tiles,K,shift,dense", [
    ("f32", 20, 8, 0, False), ("bf16", 20, 8, 4, True),                     # a part of the chip
    ("f32", 300, 2, 4, True), ("bf16", 300, 4, 0, False), ("f32", 300, 7, 12, False), ("bf16", 600, 6, 4, True),
    ("bf16", 1024, 5, 0, False), ("bf16", 1024, 8, 20, True),
    ("f32", 3072, 8, 4, True), ("bf16", 2048, 7, 0, False), ("f32", 2048, 6, 36, False), ("f32", 4096, 7, 0, True),
    ("f32", 6144, 5, 4, True), ("bf16", 5120, 5, 4, False), ("f32", 8192, 4, 60, False), ("f32", 12288, 2, 0, True),
    ("bf16", 32768, 4, 0, False), ("f32", 16384, 8, 0, False),              # the latter: fused pass inside the windows
])
def test_shared_tiles(dtype, tiles, K, shift, dense):
    n = -(-tiles * (16384 // (4 if dtype == "f32" else 2)) // 24) | 1
    plan = every_kernel([n + 2 * t for t in range(24)], dtype, 0 if tiles < 2000 else 64 << 20, K, shift, dense)
    assert plan.num_tiles > tiles

"""Tiles that hold 1 to 6 tensors (the table of up to 4 goes to registers in SGD on unpack of bf16 gradients): large
tensors with a few small and empty ones between them, at 64-byte and other addresses; every kernel, every element."""
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


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shift,dense", [(0, False), (32, False), (4, True), (36, True)])
@pytest.mark.parametrize("small", [(), (0,), (1,), (9, 4), (64, 3, 1), (0, 0, 7, 5), (1, 2, 3, 4, 5)])
def test_few_tensors_in_a_tile(dtype, small, shift, dense):
    numels = []
    for large in (20000, 8192, 8200, 30011, 4096, 17, 9001):
        numels += [large, *small]
    every_kernel(numels, dtype, 0, 3, shift, dense)

"""Which launches hold back workgroups per CU (they ask for LDS beyond the kernel's own), share tiles between
workgroups or store in windows (whole tiles, nothing held): read from the kernel nodes of a recorded
graph, around the limits of the launch rules."""
import ctypes
import os
import subprocess
import sys

import pytest
import torch

import paper_2505_10183_amd as kt

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(autouse=True)
def announce(request):
    print("\n[gpu-case] %s" % request.node.nodeid, file=sys.stderr, flush=True)
    yield
    torch.cuda.synchronize()
    torch.cuda.empty_cache()


class Dim3(ctypes.Structure):
    _fields_ = [("x", ctypes.c_uint32), ("y", ctypes.c_uint32), ("z", ctypes.c_uint32)]


class KernelNodeParams(ctypes.Structure):      # hipKernelNodeParams
    _fields_ = [("blockDim", Dim3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("gridDim", Dim3),
                ("kernelParams", ctypes.c_void_p), ("sharedMemBytes", ctypes.c_uint)]


def hip():
    kt.binding.lib()
    return ctypes.CDLL("libamdhip64.so")       # the runtime the process already holds


def recorded_kernel(call, argument=None):
    """Lanes, workgroups and dynamic LDS of the one kernel that `call(stream)` launches (its tables are on the device already),
    and the 32 bits at the place `argument` of its arguments (-1: the address of its function)."""
    h, s = hip(), torch.cuda.Stream()
    graph = ctypes.c_void_p()
    assert h.hipStreamBeginCapture(ctypes.c_void_p(s.cuda_stream), 0) == 0
    try:
        call(s)
    finally:
        assert h.hipStreamEndCapture(ctypes.c_void_p(s.cuda_stream), ctypes.byref(graph)) == 0
    n = ctypes.c_size_t(0)
    assert h.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    nodes = (ctypes.c_void_p * n.value)()
    assert h.hipGraphGetNodes(graph, nodes, ctypes.byref(n)) == 0
    got = []
    for node in nodes:
        kind = ctypes.c_int(-1)
        assert h.hipGraphNodeGetType(ctypes.c_void_p(node), ctypes.byref(kind)) == 0
        if kind.value == 0:                    # hipGraphNodeTypeKernel
            p = KernelNodeParams()
            assert h.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(p)) == 0
            got.append((p.blockDim.x, p.gridDim.x, p.sharedMemBytes))
            if argument == -1:
                got[-1] += (p.func,)
            elif argument is not None:
                where = ctypes.cast(p.kernelParams, ctypes.POINTER(ctypes.c_void_p))[argument]
                got[-1] += (ctypes.cast(where, ctypes.POINTER(ctypes.c_uint32))[0],)
    assert h.hipGraphDestroy(graph) == 0
    assert len(got) == 1, got
    return got[0]


def launch(op, dtype, K, tiles):
    lanes, grid, lds = kernel(op, dtype, K, tiles)
    assert lanes == 256
    return grid, lds


def kernel(op, dtype, K, tiles, argument=None):
    es, td = (4, torch.float32) if dtype == "f32" else (2, torch.bfloat16)
    numels = [tiles * (16384 // es)]
    plan = kt.Plan(numels, dtype, 0, 16)
    assert plan.num_tiles == tiles
    mk = plan.marshal
    keep = [torch.zeros(numels[0], dtype=td, device=DEV) for _ in range(K + 1)]
    state = [torch.zeros(numels[0], device=DEV) for _ in range(2)] if op in ("sgd", "fused_sgd") else []
    grads, out, others, copies = mk(keep[:1]), mk(keep[K:]), mk(keep[1:K]), mk(keep[:K])
    w = [1.0 / K] * K

    def call(stream=None):
        if op.endswith("reduce"):
            plan.kt_weighted_reduce(-1, copies, K, w, out, stream=stream)
        elif op == "fused":
            plan.kt_fused_step(-1, grads, others, K, w, 1.0, out, stream=stream)
        elif op == "sgd":
            plan.kt_bucket_unpack_sgd(-1, grads, 1.0, mk(state[:1]), mk(state[1:]), 0.1, 0.9, 0.0, False, stream=stream)
        else:
            plan.kt_fused_step_sgd(-1, grads, others, K, w, 1.0, mk(state[:1]), mk(state[1:]), None, 0.1, 0.9, 0.0, False,
                                   stream=stream)

    call()
    if op == "packed reduce":
        plan.kt_bucket_pack(-1, out, grads)
    torch.cuda.synchronize()
    return recorded_kernel(call, argument)


def run_bytes(op, dtype, K, tiles):
    """Lanes, workgroups per tile, and bytes of a copy that an XCD takes in a run (0: launch order)."""
    lanes, grid, _, order = kernel(op, dtype, K, tiles, ORDER[op][K > 8])
    split, g = grid // tiles, order & 7
    assert grid == split * tiles and order >> 3 << 3 == (grid >> 3 + g << 3 + g if g else 0)
    return lanes, split, (16384 // split << g if g else 0)


# place of the order of the pieces among the kernel's arguments: up to 8 copies and above
ORDER = {"fused_sgd": (6, 6), "fused": (7, 6), "reduce": (4, 5), "packed reduce": (4, 5), "sgd": (6, 6)}


def dynamic_lds(op, dtype, K, tiles):
    return launch(op, dtype, K, tiles)[1]


@pytest.mark.parametrize("op,dtype,K,least", [
    ("fused_sgd", "bf16", 1, 1024), ("fused_sgd", "bf16", 2, 1024), ("fused_sgd", "bf16", 4, 2048),
    ("fused_sgd", "bf16", 8, 2048), ("fused_sgd", "f32", 2, 4096), ("fused_sgd", "f32", 4, 4096),
    ("fused_sgd", "f32", 8, 2048), ("reduce", "f32", 3, 8191), ("reduce", "bf16", 4, 4095),
    ("fused", "f32", 3, 8191), ("fused", "bf16", 3, 8191), ("fused", "f32", 4, 2047), ("fused", "bf16", 5, 2047),
    ("sgd", "f32", 1, 4095), ("sgd", "bf16", 1, 4095),
])
def test_workgroups_are_held_above_a_launch_size_only(op, dtype, K, least):
    assert dynamic_lds(op, dtype, K, least) == 0
    assert dynamic_lds(op, dtype, K, least + 1) > 0


@pytest.mark.parametrize("op,dtype,K,own,count", [
    ("reduce", "f32", 4, 0, 2), ("fused", "bf16", 5, 16384, 2), ("sgd", "f32", 1, 16384, 4), ("sgd", "bf16", 1, 16384, 5),
    ("fused_sgd", "bf16", 8, 16384, 2), ("fused_sgd", "f32", 2, 16384, 4), ("fused_sgd", "f32", 8, 16384, 2),
])
def test_held_workgroups_per_cu(op, dtype, K, own, count):
    """160 KiB of LDS in granules of 1280 bytes; `own` is the kernel's static LDS."""
    granules = -(-(own + dynamic_lds(op, dtype, K, 4200)) // 1280)
    assert 163840 // 1280 // granules == count


LARGE = [("reduce", "f32", 4), ("reduce", "bf16", 5), ("fused", "bf16", 4), ("sgd", "f32", 1), ("sgd", "bf16", 1),
         ("fused_sgd", "bf16", 8), ("fused_sgd", "f32", 2)]


@pytest.mark.parametrize("op,dtype,K", LARGE)
def test_nothing_held_where_the_gpu_is_shared(op, dtype, K):
    """KT_STORE_WINDOW_NS=0 (read once per process, hence a child): no LDS beyond the kernel's own."""
    assert dynamic_lds(op, dtype, K, 4200) > 0
    env = dict(os.environ, KT_STORE_WINDOW_NS="0")
    here = os.path.dirname(os.path.abspath(__file__))
    code = "import sys; sys.path[:0] = [%r, %r]; import test_gpu_launch_rules as t; print('LDS', t.dynamic_lds(%r, %r, %d, 4200))" \
        % (os.path.dirname(here), here, op, dtype, K)
    r = subprocess.run([sys.executable, "-c", code], env=env, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    assert "LDS 0" in r.stdout.splitlines(), r.stdout


@pytest.mark.parametrize("dtype,K,tiles,lanes,run", [
    ("bf16", 1, 1024, 256, 131072), ("bf16", 2, 1025, 256, 0), ("bf16", 3, 2048, 256, 131072), ("bf16", 6, 2049, 256, 0), ("bf16", 4, 9700, 256, 0),
    ("bf16", 2, 12288, 256, 0), ("bf16", 3, 12287, 256, 0), ("bf16", 3, 12288, 64, 0), ("bf16", 7, 12288, 64, 0), ("bf16", 8, 8191, 256, 0),
    ("bf16", 8, 8192, 64, 0), ("bf16", 8, 639, 256, 0), ("bf16", 8, 640, 256, 131072),
    ("f32", 2, 639, 256, 0), ("f32", 2, 640, 256, 131072), ("f32", 4, 640, 256, 65536), ("f32", 4, 4096, 256, 65536), ("f32", 4, 4097, 256, 0),
    ("f32", 3, 4097, 256, 0), ("f32", 8, 2048, 256, 65536), ("f32", 8, 2049, 256, 0), ("f32", 5, 44000, 256, 0),
])
def test_lanes_and_runs_of_the_one_pass_sgd(dtype, K, tiles, lanes, run):
    assert run_bytes("fused_sgd", dtype, K, tiles) == (lanes, 16384 // (16 * lanes), run)


@pytest.mark.parametrize("dtype,K,tiles,split,run", [
    ("f32", 4, 2047, 1, 0), ("f32", 4, 2048, 1, 131072), ("f32", 4, 8191, 1, 131072), ("f32", 4, 8192, 4, 32768), ("f32", 4, 32767, 4, 32768),
    ("f32", 4, 32768, 4, 0), ("f32", 5, 6143, 1, 131072), ("f32", 5, 6144, 4, 0), ("f32", 6, 4096, 4, 0), ("f32", 7, 20000, 4, 0), ("f32", 8, 9900, 4, 0),
    ("f32", 3, 9000, 1, 0), ("bf16", 3, 9000, 1, 0), ("bf16", 4, 3000, 1, 131072), ("bf16", 4, 40000, 2, 131072), ("bf16", 5, 5119, 1, 131072),
    ("bf16", 5, 5120, 2, 0), ("bf16", 5, 70000, 2, 0),
    ("bf16", 6, 1023, 2, 0), ("bf16", 6, 1024, 2, 131072), ("bf16", 7, 20000, 2, 131072), ("bf16", 8, 20000, 2, 0),
    ("f32", 9, 639, 4, 0), ("f32", 9, 640, 4, 65536), ("f32", 9, 4095, 4, 65536), ("f32", 9, 4096, 4, 0), ("bf16", 10, 4096, 4, 0),
    ("bf16", 12, 5000, 4, 65536),
])
def test_runs_of_the_fused_pass(dtype, K, tiles, split, run):
    assert run_bytes("fused", dtype, K, tiles) == (256, split, run)


@pytest.mark.parametrize("dtype,K,tiles,run,packed_run", [
    ("f32", 2, 590, 0, 0), ("f32", 2, 20000, 0, 0), ("f32", 3, 8192, 0, 65536), ("bf16", 3, 32767, 0, 65536), ("bf16", 3, 32768, 0, 0),
    ("f32", 5, 590, 65536, 65536), ("f32", 6, 6143, 65536, 65536), ("f32", 6, 6144, 0, 65536), ("f32", 7, 6144, 65536, 65536), ("f32", 8, 32767, 0, 65536),
    ("f32", 8, 32768, 0, 0), ("bf16", 5, 8191, 65536, 65536), ("bf16", 5, 8192, 0, 65536), ("bf16", 8, 20000, 65536, 65536), ("f32", 4, 8192, 0, 65536),
    ("f32", 9, 6143, 65536, 65536), ("f32", 9, 6144, 0, 65536), ("f32", 12, 9000, 0, 65536), ("f32", 16, 8191, 0, 65536), ("f32", 16, 8192, 0, 0),
    ("bf16", 16, 9000, 0, 65536),
])
def test_runs_of_the_reduce(dtype, K, tiles, run, packed_run):
    assert run_bytes("reduce", dtype, K, tiles) == (256, 4, run)
    assert run_bytes("packed reduce", dtype, K, tiles) == (256, 4, packed_run)


@pytest.mark.parametrize("dtype,tiles,run", [
    ("f32", 1023, 0), ("f32", 1024, 131072), ("f32", 32767, 131072), ("f32", 32768, 0), ("bf16", 1791, 0), ("bf16", 1792, 131072), ("bf16", 4095, 131072),
    ("bf16", 4096, 0),
])
def test_runs_of_sgd_on_unpack(dtype, tiles, run):
    assert run_bytes("sgd", dtype, 1, tiles) == (256, 4 if dtype == "f32" else 8, run)


@pytest.mark.parametrize("dtype,K,tiles,alike", [
    ("f32", 7, 1099, True), ("f32", 7, 1100, False), ("bf16", 8, 6143, False), ("bf16", 8, 6144, True), ("f32", 6, 2000, True), ("bf16", 9, 1535, True),
    ("bf16", 9, 1536, False),
])
def test_store_scope_of_the_reduce_behind_a_pack(dtype, K, tiles, alike):
    """7 and more copies: another instantiation, with system-scope stores, between 1 100 (1 536) and 6 143 tiles behind a pack."""
    assert (kernel("reduce", dtype, K, tiles, -1)[3] == kernel("packed reduce", dtype, K, tiles, -1)[3]) == alike


def test_packed_ends_with_the_next_launch():
    plan = kt.Plan([9000 * 4096], "f32", 0, 16)
    mk = plan.marshal
    keep = [torch.zeros(9000 * 4096, device=DEV) for _ in range(6)]
    grads, copies, out, spare = mk(keep[:1]), mk(keep[1:5]), mk(keep[5:]), mk(keep[1:2])
    pack = lambda stream=None: plan.kt_bucket_pack(-1, grads, spare, stream=stream)
    reduce = lambda stream=None: plan.kt_weighted_reduce(-1, copies, 4, [0.25] * 4, out, stream=stream)
    unpack = lambda stream=None: plan.kt_bucket_unpack_scale(-1, out, 1.0, grads, stream=stream)
    order = lambda: recorded_kernel(reduce, 4)[3]
    reduce(), pack(), unpack()
    assert order() == 0
    pack()
    assert order() & 7 and order() == 0 and order() == 0
    with pytest.raises(kt.KtError):
        plan.kt_bucket_pack(5, grads, spare)       # refused: no launch
    assert order() == 0
    recorded_kernel(pack)
    assert order() & 7
    pack(), reduce()
    assert order() == 0
    torch.cuda.synchronize()


@pytest.mark.parametrize("op,tiles,count", [("reduce", 6144, 3), ("packed reduce", 6143, 3), ("packed reduce", 6144, 2), ("packed reduce", 32767, 2),
                                            ("packed reduce", 32768, 3)])
def test_held_workgroups_of_the_reduce_of_7_copies(op, tiles, count):
    assert 163840 // 1280 // -(-kernel(op, "f32", 7, tiles)[2] // 1280) == count


@pytest.mark.parametrize("dtype,K,tiles,count", [("f32", 4, 8192, 4), ("f32", 4, 32768, 3), ("f32", 7, 9000, 3)])
def test_held_workgroups_of_the_fused_pass(dtype, K, tiles, count):
    assert 163840 // 1280 // -(-(16384 + kernel("fused", dtype, K, tiles)[2]) // 1280) == count


@pytest.mark.parametrize("K,tiles,count", [(3, 12288, 6), (4, 12288, 6), (5, 12288, 5), (7, 12288, 5), (8, 8192, 4)])
def test_held_workgroups_of_64_lanes(K, tiles, count):
    lanes, grid, lds = kernel("fused_sgd", "bf16", K, tiles)
    assert (lanes, grid) == (64, 16 * tiles) and 163840 // 1280 // -(-(16384 + lds) // 1280) == count


@pytest.mark.parametrize("K,tiles", [(1, 12288), (4, 12288), (8, 8192)])
def test_full_workgroups_where_the_gpu_is_shared(K, tiles):
    """Workgroups of 64 lanes, unheld, would keep nearly all LDS of a CU with few wavefronts."""
    env = dict(os.environ, KT_STORE_WINDOW_NS="0")
    here = os.path.dirname(os.path.abspath(__file__))
    code = "import sys; sys.path[:0] = [%r, %r]; import test_gpu_launch_rules as t; print('GOT', t.kernel('fused_sgd', 'bf16', %d, %d))" \
        % (os.path.dirname(here), here, K, tiles)
    r = subprocess.run([sys.executable, "-c", code], env=env, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    assert "GOT (256, %d, 0)" % (4 * tiles) in r.stdout.splitlines(), r.stdout


@pytest.mark.parametrize("op,dtype,K,least", [
    ("reduce", "f32", 7, 65536), ("reduce", "f32", 8, 65536), ("reduce", "bf16", 7, 65536), ("reduce", "bf16", 8, 65536),
    ("reduce", "f32", 10, 26215), ("reduce", "f32", 16, 16384), ("reduce", "bf16", 11, 23832), ("reduce", "bf16", 24, 10923),
    ("fused", "f32", 7, 65536), ("fused", "f32", 8, 16384), ("fused", "bf16", 7, 131072), ("fused", "bf16", 8, 131072),
    ("fused", "f32", 10, 6554), ("fused", "f32", 16, 4096), ("fused", "bf16", 11, 5958), ("fused", "bf16", 16, 4096),
    ("fused_sgd", "f32", 11, 8937), ("fused_sgd", "f32", 16, 6144), ("fused_sgd", "bf16", 14, 14044),
])
def test_store_windows_from_a_launch_size_on(op, dtype, K, least):
    """Inside the windows a launch has one workgroup per tile and holds none; just below it shares tiles and holds."""
    below, lds = launch(op, dtype, K, least - 1)
    assert below > least - 1 and lds > 0
    assert launch(op, dtype, K, least) == (least, 0)


@pytest.mark.parametrize("op,dtype,K", [("reduce", "f32", 9), ("reduce", "bf16", 10), ("fused", "f32", 9), ("fused", "bf16", 10),
                                        ("fused_sgd", "f32", 10), ("fused_sgd", "bf16", 13), ("reduce", "f32", 6), ("fused", "bf16", 6)])
def test_no_store_windows_with_fewer_copies(op, dtype, K):
    grid, lds = launch(op, dtype, K, 32768)
    assert grid > 32768 and lds > 0


@pytest.mark.parametrize("op,dtype,K,tiles,split", [
    # nearly full rounds of whole tiles, uneven ones, and where sharing begins
    ("reduce", "f32", 2, 12287, 1), ("reduce", "f32", 2, 12288, 4), ("reduce", "bf16", 3, 8192, 4), ("reduce", "f32", 4, 8191, 1),
    ("reduce", "f32", 4, 8192, 4), ("reduce", "bf16", 4, 12287, 1), ("reduce", "f32", 5, 4095, 1), ("reduce", "f32", 6, 2048, 4),
    ("reduce", "bf16", 7, 2047, 1), ("reduce", "f32", 7, 4096, 4), ("reduce", "f32", 8, 3071, 1), ("reduce", "bf16", 8, 2048, 4),
    ("reduce", "f32", 8, 512, 1), ("reduce", "f32", 8, 551, 4), ("reduce", "bf16", 16, 256, 4), ("reduce", "f32", 12, 2559, 1),
    ("reduce", "f32", 12, 2560, 4),
    ("fused", "bf16", 4, 1023, 2), ("fused", "bf16", 4, 1024, 1), ("fused", "bf16", 5, 5120, 2), ("fused", "f32", 4, 8191, 1),
    ("fused", "f32", 4, 8192, 4), ("fused", "f32", 6, 4096, 4), ("fused", "bf16", 6, 100, 2), ("fused", "f32", 12, 100, 4),
    ("fused_sgd", "f32", 12, 896, 4), ("fused_sgd", "f32", 12, 897, 1), ("fused_sgd", "bf16", 9, 641, 1), ("fused_sgd", "f32", 9, 2560, 4),
])
def test_workgroups_per_tile(op, dtype, K, tiles, split):
    assert launch(op, dtype, K, tiles)[0] == split * tiles

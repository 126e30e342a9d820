"""Launches large enough for the choices that depend on the launch size (workgroups held per CU,
store windows, store scope), with tensors and buckets away from 64-byte boundaries: every kernel,
every element against the CPU checker's binary32 step mode (bit-identical), with guard elements
around every output.  Then the same for tiles that hold hundreds of very small tensors."""
import sys
from concurrent.futures import ThreadPoolExecutor

import pytest
import torch

import oracle
import paper_2505_10183_amd as kt
from paper_2505_10183_amd import workloads as wl
from test_gpu_any_address import Guarded
from test_gpu_parity import DEV, host, raw, tdtype

pytestmark = pytest.mark.gpu
SCALE, LR, MU, WD = 0.37, 0.1, 0.9, 5e-4


@pytest.fixture(autouse=True)
def announce(request):
    print("\n[gpu-case] %s" % request.node.nodeid, file=sys.stderr, flush=True)
    yield
    torch.cuda.synchronize()
    torch.cuda.empty_cache()


def equal(dev, want, what):
    assert raw(host(dev)).tobytes() == raw(want).tobytes(), what


# tiles: just above a limit of the launch rules.  shift: bytes from a 64-byte boundary to the first
# element of the gradients and parameters (the others lie elsewhere).
@pytest.mark.parametrize("dtype,tiles,K,shift,dense", [
    ("bf16", 32768, 8, 36, False),      # one-pass SGD: workgroups of 64 lanes
    ("bf16", 32768, 8, 0, False),
    ("f32", 4096, 2, 4, True),          # one-pass SGD with workgroups held per CU
    ("f32", 4096, 4, 36, False),        # and the held reduce, fused pass and SGD on unpack
    ("bf16", 4096, 4, 12, True),
    ("f32", 8192, 3, 60, True),
    ("bf16", 8192, 3, 16, False),
    ("f32", 4096, 16, 4, False),        # fused pass of many copies inside the store windows (65 536 tiles read)
    ("bf16", 4096, 16, 0, False),
    ("bf16", 8192, 8, 4, True),         # and of 8: half tiles (fused pass) and quarter tiles, held
])
def test_large_launches(dtype, tiles, K, shift, dense):
    n = -(-tiles * (16384 // (4 if dtype == "f32" else 2)) // 24) | 1
    plan = every_kernel([n + 2 * t for t in range(24)], dtype, (25 if dtype == "f32" else 64) << 20, K, shift, dense)
    assert plan.num_tiles > tiles


# 512 and more tensors in a full tile, or too many in a short one, take another way through the
# elements (each_cut_elem).
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("sizes,count,dense", [
    ((1,), 1500, True), ((1,), 1500, False), ((0, 1, 2, 0, 3), 1800, True), ((3, 1, 0, 9), 1400, False),
    ((7,), 1300, True), ((1,), 40, True), ((9,), 513, False),
])
@pytest.mark.parametrize("K", [4, 11])
def test_many_small_tensors(dtype, sizes, count, dense, K):
    numels = [sizes[t % len(sizes)] for t in range(count)]
    numels.insert(count // 2, 20011)           # a tensor of several tiles between them
    every_kernel(numels, dtype, 0, K, 4, dense)


def every_kernel(numels, dtype, cap, K, shift, dense):
    td, es = tdtype(dtype), 4 if dtype == "f32" else 2
    align = es if dense else 16
    plan = kt.Plan(numels, dtype, cap, align)
    L = oracle.assign_buckets(numels, es, cap, align)
    thr = [1.0 - 0.04 * k for k in range(K)]
    shares, weights = kt.kt_plan_shares(thr, 1024)
    wts = oracle.share_weights(shares, 1024)
    nb, elems = plan.num_buckets, plan.bucket_elems()

    def filled(sizes, dt, sh, seed, sigma=1e-3):
        g = Guarded(sizes, dt, sh, 3.0)
        values = wl.flat_normal(sum(sizes), "f32" if dt == torch.float32 else "bf16", sigma, seed, DEV)
        for v, x in zip(g.views, values.split(list(sizes))):
            v.copy_(x)
        return g

    grads = filled(numels, td, shift, 1000)
    peers = [filled(elems, td, (shift + 4 * k) % 64, 2000 + 100 * k) for k in range(1, K)]
    slot0, other = Guarded(elems, td, (64 - shift) % 64, 5.0), Guarded(elems, td, shift, 5.0)
    out, fout = Guarded(numels, td, (64 - shift) % 64, 7.0), Guarded(numels, td, shift, 7.0)
    p, v = filled(numels, torch.float32, shift, 100, 1.0), filled(numels, torch.float32, (shift + 16) % 64, 200, 1.0)
    fp, fv = filled(numels, torch.float32, shift, 100, 1.0), filled(numels, torch.float32, shift, 200, 1.0)
    m, fm = Guarded(numels, torch.bfloat16, shift // 2, 9.0), Guarded(numels, torch.bfloat16, shift, 9.0)
    hp, hv = [host(t) for t in p.views], [host(t) for t in v.views]
    others = [peers[k - 1].views[b] for b in range(nb) for k in range(1, K)]

    plan.kt_bucket_pack(-1, grads.views, slot0.views)
    copies = [slot0.views[b] if k == 0 else peers[k - 1].views[b] for b in range(nb) for k in range(K)]
    plan.kt_weighted_reduce(-1, copies, K, weights, other.views)
    plan.kt_bucket_unpack_scale(-1, other.views, SCALE, out.views)
    plan.kt_bucket_unpack_sgd_master(-1, other.views, SCALE, p.views, v.views, m.views, LR, MU, WD, False)
    plan.kt_fused_step(-1, grads.views, others, K, weights, SCALE, fout.views)
    plan.kt_fused_step_sgd(-1, grads.views, others, K, weights, SCALE, fp.views, fv.views, fm.views, LR, MU, WD, False)
    torch.cuda.synchronize()

    def bucket(b):
        first, cnt = L["bucket_first"][b], L["bucket_count"][b]
        ts = range(first, first + cnt)
        sub = {"tensor_bucket": [0] * cnt, "tensor_offset": [L["tensor_offset"][t] for t in ts], "bucket_elems": [elems[b]]}
        sizes = [numels[t] for t in ts]
        packed = oracle.pack(sub, [host(grads.views[t]) for t in ts], dtype)[0]
        equal(slot0.views[b], packed, ("pack", b))
        red = oracle.weighted_reduce([packed] + [host(peers[k].views[b]) for k in range(K - 1)], wts, dtype, "S")
        equal(other.views[b], red, ("reduce", b))
        scaled = oracle.unpack_scale(sub, [red], sizes, SCALE, dtype, "S")
        wp, wv, wm = oracle.unpack_sgd_master(sub, [red], sizes, SCALE, [hp[t] for t in ts], [hv[t] for t in ts], LR, MU, WD,
                                              False, dtype, "S")
        for i, t in enumerate(ts):
            for what, dev, want in (("unpack", out, scaled), ("fused", fout, scaled), ("sgd p", p, wp), ("sgd v", v, wv),
                                    ("sgd model", m, wm), ("one pass p", fp, wp), ("one pass v", fv, wv),
                                    ("one pass model", fm, wm)):
                equal(dev.views[t], want[i], (what, t))

    with ThreadPoolExecutor(12) as pool:
        list(pool.map(bucket, range(nb)))
    for g, what in ((slot0, "slot0"), (other, "reduced"), (out, "out"), (fout, "fused"), (p, "p"), (v, "v"), (m, "m"),
                    (fp, "one pass p"), (fv, "one pass v"), (fm, "one pass m")):
        g.check_guards(what)
    return plan

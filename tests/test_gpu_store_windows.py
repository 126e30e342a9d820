"""The single pass of 7 and 8 copies inside the store windows: every element against pack, reduce and unpack,
whose results other tests compare with the CPU checker at these sizes, and some buckets against the checker itself."""
import sys

import pytest
import torch

import oracle
import paper_2505_10183_amd as kt
from paper_2505_10183_amd import workloads as wl
from test_gpu_parity import DEV, host, raw, tdtype

pytestmark = pytest.mark.gpu
SCALE = 0.37


@pytest.fixture(autouse=True)
def announce(request):
    print("\n[gpu-case] %s" % request.node.nodeid, file=sys.stderr, flush=True)
    yield
    torch.cuda.synchronize()
    torch.cuda.empty_cache()


def same(a, b):
    kind = torch.int32 if a.element_size() == 4 else torch.int16
    return torch.equal(a.view(kind), b.view(kind))


@pytest.mark.parametrize("dtype,K,tiles", [("f32", 7, 65536), ("f32", 8, 65536), ("bf16", 7, 131072)])
def test_fused_pass_inside_the_windows(dtype, K, tiles):
    w = wl.get("sized_%s_%d" % (dtype, tiles))
    plan = kt.Plan(w.numels, dtype, w.bucket_cap_bytes, 16)
    assert plan.num_tiles >= tiles
    nb, elems, td = plan.num_buckets, plan.bucket_elems(), tdtype(dtype)
    thr = [1.0 - 0.04 * k for k in range(K)]
    shares, weights = kt.kt_plan_shares(thr, 1024)
    wts = oracle.share_weights(shares, 1024)
    grads = [wl.flat_normal(n, dtype, 1e-3, 100 + t, DEV) for t, n in enumerate(w.numels)]
    slot0 = [torch.empty(n, dtype=td, device=DEV) for n in elems]
    peers = [[wl.flat_normal(n, dtype, 1e-3, 3000 + 50 * k + b, DEV) for b, n in enumerate(elems)] for k in range(1, K)]
    chained, fused = [torch.empty_like(t) for t in grads], [torch.empty_like(t) for t in grads]
    plan.kt_bucket_pack(-1, grads, slot0)
    plan.kt_weighted_reduce(-1, [slot0[b] if k == 0 else peers[k - 1][b] for b in range(nb) for k in range(K)], K, weights, slot0)
    plan.kt_bucket_unpack_scale(-1, slot0, SCALE, chained)
    plan.kt_fused_step(-1, grads, [peers[k - 1][b] for b in range(nb) for k in range(1, K)], K, weights, SCALE, fused)
    torch.cuda.synchronize()
    for t in range(len(grads)):
        assert same(chained[t], fused[t]), t
    L = oracle.assign_buckets(w.numels, 4 if dtype == "f32" else 2, w.bucket_cap_bytes, 16)
    for b in (0, nb // 2, nb - 1):
        first, cnt = L["bucket_first"][b], L["bucket_count"][b]
        sub = {"tensor_bucket": [0] * cnt, "tensor_offset": L["tensor_offset"][first:first + cnt], "bucket_elems": [elems[b]]}
        packed = oracle.pack(sub, [host(g) for g in grads[first:first + cnt]], dtype)[0]
        red = oracle.weighted_reduce([packed] + [host(peers[k][b]) for k in range(K - 1)], wts, dtype, "S")
        want = oracle.unpack_scale(sub, [red], list(w.numels[first:first + cnt]), SCALE, dtype, "S")
        for i in range(cnt):
            assert raw(host(fused[first + i])).tobytes() == raw(want[i]).tobytes(), (b, i)

"""Launches whose workgroups take runs of neighbouring pieces per XCD: pieces in whole groups and left over."""
import random
import sys

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
    torch.cuda.empty_cache()


def inputs(dtype, K, elems):
    plan = kt.Plan([elems], dtype, 0, 16)
    _, weights = kt.kt_plan_shares([1.0 - 0.05 * k for k in range(K)], 1024)
    copies = [wl.flat_normal(elems, dtype, 1e-3, 900 + k, DEV) for k in range(K)]
    want = oracle.weighted_reduce([host(c) for c in copies], weights, dtype, "S")
    return plan, weights, copies, want


# tiles shared by four workgroups: 300 tiles are 1 200 pieces (4 groups of 256 in runs of 128 KiB and 176 pieces in launch order, 9 of
# 128 in runs of 64 KiB and 48), 320 are whole groups only, 321 leave one tile over
@pytest.mark.parametrize("dtype,K,tiles,tail", [
    ("f32", 2, 300, 0), ("f32", 3, 320, 0), ("f32", 8, 321, 4), ("bf16", 4, 300, 8), ("bf16", 7, 320, 0), ("f32", 9, 33, 0),
    ("f32", 12, 255, 4), ("bf16", 16, 64, 8), ("f32", 7, 6144, 4), ("f32", 9, 6145, 0), ("bf16", 5, 8200, 8), ("f32", 3, 8195, 4),   # the last four: behind a pack only, or with another hold
])
def test_reduce_in_runs(dtype, K, tiles, tail):
    plan, weights, copies, want = inputs(dtype, K, tiles * (16384 // (4 if dtype == "f32" else 2)) + tail)
    out = torch.empty_like(copies[0])
    plan.kt_weighted_reduce(-1, copies, K, weights, [out])
    torch.cuda.synchronize()
    assert raw(host(out)).tobytes() == raw(want).tobytes()
    packed = torch.zeros_like(copies[0])
    plan.kt_bucket_pack(-1, copies[:1], [packed])
    plan.kt_weighted_reduce(-1, [packed] + copies[1:], K, weights, [out.zero_()])
    torch.cuda.synchronize()
    assert raw(host(out)).tobytes() == raw(want).tobytes()


@pytest.mark.parametrize("dtype,K,tiles,tail", [
    ("f32", 1, 640, 0), ("f32", 4, 660, 4), ("f32", 8, 641, 0), ("bf16", 2, 641, 8), ("bf16", 8, 640, 0), ("bf16", 12, 704, 8), ("f32", 16, 641, 0),
    ("bf16", 1, 12288, 0), ("bf16", 2, 12288, 0), ("bf16", 3, 12289, 8), ("bf16", 5, 12288, 8), ("bf16", 6, 12289, 0), ("bf16", 7, 12288, 0),
    ("bf16", 8, 8251, 8),       # from 3 copies on workgroups of 64 lanes
])
def test_one_pass_sgd_in_runs(dtype, K, tiles, tail):
    plan, weights, copies, want = inputs(dtype, K, tiles * (16384 // (4 if dtype == "f32" else 2)) + tail)
    n = copies[0].numel()
    p, v = wl.flat_normal(n, "f32", 2e-2, 1, DEV), wl.flat_normal(n, "f32", 1e-3, 2, DEV)
    p2, v2 = p.clone(), v.clone()
    m, m2 = (torch.zeros(n, dtype=torch.bfloat16, device=DEV) for _ in range(2))
    plan.kt_fused_step_sgd(-1, copies[:1], copies[1:], K, weights, 0.5, [p], [v], [m], 0.05, 0.9, 5e-4, False)
    # the update of the oracle's sum, in the kernel that other tests compare with the oracle
    red = torch.empty_like(copies[0])
    kind = torch.int32 if dtype == "f32" else torch.int16
    red.view(kind).copy_(torch.from_numpy(raw(want).view("i4" if dtype == "f32" else "i2")))
    plan.kt_bucket_unpack_sgd_master(-1, [red], 0.5, [p2], [v2], [m2], 0.05, 0.9, 5e-4, False)
    torch.cuda.synchronize()
    assert torch.equal(p.view(torch.int32), p2.view(torch.int32)) and torch.equal(v.view(torch.int32), v2.view(torch.int32))
    assert torch.equal(m.view(torch.int16), m2.view(torch.int16))


@pytest.mark.parametrize("dtype,K,tiles,tail", [
    ("f32", 4, 2048, 0), ("f32", 5, 2067, 4), ("f32", 6, 4097, 0), ("bf16", 5, 2049, 8), ("bf16", 6, 1024, 0), ("bf16", 8, 1061, 8),
    ("f32", 9, 640, 4), ("bf16", 12, 673, 0), ("f32", 4, 8195, 4), ("bf16", 7, 1031, 8),
])
def test_fused_pass_in_runs(dtype, K, tiles, tail):
    plan, weights, copies, want = inputs(dtype, K, tiles * (16384 // (4 if dtype == "f32" else 2)) + tail)
    out = torch.empty_like(copies[0])
    plan.kt_fused_step(-1, copies[:1], copies[1:], K, weights, 1.0, [out])       # scale 1: the sum itself
    torch.cuda.synchronize()
    assert raw(host(out)).tobytes() == raw(want).tobytes()


@pytest.mark.parametrize("dtype,tiles,tail,master", [
    ("f32", 1024, 0, False), ("f32", 1061, 4, True), ("bf16", 640, 0, False), ("bf16", 1792, 0, False), ("bf16", 1855, 8, True), ("bf16", 4095, 0, True),
])
def test_sgd_on_unpack_in_runs(dtype, tiles, tail, master):
    n = tiles * (16384 // (4 if dtype == "f32" else 2)) + tail
    g = wl.flat_normal(n, dtype, 1e-3, 7, DEV)
    p, v = wl.flat_normal(n, "f32", 2e-2, 1, DEV), wl.flat_normal(n, "f32", 1e-3, 2, DEV)
    want_p, want_v, want_m = p.clone(), v.clone(), torch.zeros(n, dtype=torch.bfloat16, device=DEV)
    m = torch.zeros_like(want_m)

    def update(grad, params, momenta, models):
        plan = kt.Plan([grad.numel()], dtype, 0, 16)
        if master:
            plan.kt_bucket_unpack_sgd_master(-1, [grad], 0.5, [params], [momenta], [models], 0.05, 0.9, 5e-4, False)
        else:
            plan.kt_bucket_unpack_sgd(-1, [grad], 0.5, [params], [momenta], 0.05, 0.9, 5e-4, False)
        torch.cuda.synchronize()

    update(g, p, v, m)
    part = 512 * (16384 // (4 if dtype == "f32" else 2))       # launches in launch order, which other tests compare with the checker
    for at in range(0, n, part):
        update(*[t[at:at + part] for t in (g, want_p, want_v, want_m)])
    assert torch.equal(p.view(torch.int32), want_p.view(torch.int32)) and torch.equal(v.view(torch.int32), want_v.view(torch.int32))
    assert torch.equal(m.view(torch.int16), want_m.view(torch.int16))


# system-scope stores from 1 100 (many copies: 1 536) to 6 143 tiles, where the output starts on 64 bytes, and outputs that start elsewhere
@pytest.mark.parametrize("dtype,K,tiles,tail,off", [
    ("f32", 2, 1100, 0, 0), ("bf16", 3, 1099, 8, 0), ("f32", 8, 1101, 4, 0), ("f32", 8, 1100, 4, 1), ("bf16", 8, 2048, 8, 1), ("bf16", 8, 2048, 8, 8),
    ("f32", 4, 6143, 0, 0), ("bf16", 12, 1536, 0, 0), ("f32", 9, 2560, 4, 0), ("bf16", 9, 2560, 8, 3),
])
def test_reduce_store_scopes(dtype, K, tiles, tail, off):
    plan, weights, copies, want = inputs(dtype, K, tiles * (16384 // (4 if dtype == "f32" else 2)) + tail)
    n = copies[0].numel()
    memory = torch.full((n + off + 64,), 7.0, dtype=tdtype(dtype), device=DEV)
    out = memory[off:off + n]
    plan.kt_weighted_reduce(-1, copies, K, weights, [out])
    torch.cuda.synchronize()
    assert raw(host(out)).tobytes() == raw(want).tobytes() and bool((memory[:off] == 7).all()) and bool((memory[off + n:] == 7).all())
    in_place = torch.zeros_like(copies[0])         # behind a pack: 7 and more copies take another scope there
    plan.kt_bucket_pack(-1, copies[:1], [in_place])
    plan.kt_weighted_reduce(-1, [in_place] + copies[1:], K, weights, [out.zero_()])
    plan.kt_bucket_pack(-1, copies[:1], [in_place])
    plan.kt_weighted_reduce(-1, [in_place] + copies[1:], K, weights, [in_place])
    torch.cuda.synchronize()
    assert raw(host(out)).tobytes() == raw(want).tobytes() and raw(host(in_place)).tobytes() == raw(want).tobytes()
    assert bool((memory[:off] == 7).all()) and bool((memory[off + n:] == 7).all())


# Workgroups of 64 lanes on large tensors of odd sizes with hundreds of very small ones between them (tiles of one tensor, of a few and of
# more than their table in LDS holds), gradients, parameters, momentum and model copy at odd addresses, and (the same launches) with device-resident weights
# and scalars, against pack, reduce and SGD on unpack of the same sets.
@pytest.mark.parametrize("K,tiles,resident", [(3, 12288, False), (3, 12288, True), (4, 12300, False), (5, 12288, True), (5, 12301, False), (6, 12288, False),
                                              (7, 12295, False), (7, 12288, True), (8, 8192, False), (8, 8200, True)])
def test_one_pass_sgd_of_64_lanes_on_mixed_tiles(K, tiles, resident):
    rng = random.Random(K * tiles + resident)
    numels = []
    for i in range(16):
        numels += [tiles * 512 + rng.randint(1, 40)] + [rng.randint(1, 60) for _ in range(100)] + [rng.randint(1, 12) for _ in range(900)]
    total = sum(numels)
    plan = kt.Plan(numels, "bf16", 0, 2)
    assert plan.num_tiles >= tiles and max(plan.tile_info(i)[3] for i in range(plan.num_tiles)) > 512
    starts = [0]
    for n in numels[:-1]:
        starts.append(starts[-1] + n)
    flats = [wl.flat_normal(total + 3, "bf16", 1e-3, 50, DEV)] + [wl.flat_normal(total + 3, "f32", 2e-2, 51 + i, DEV) for i in range(2)]
    flats.append(torch.zeros(total + 3, dtype=torch.bfloat16, device=DEV))
    views = lambda f, off: [f[off + s:off + s + n] for s, n in zip(starts, numels)]
    grads, params, momenta, models = (views(f, off) for f, off in zip(flats, (1, 3, 2, 1)))
    mine = [f.clone() for f in flats[1:]]
    _, weights = kt.kt_plan_shares([1.0 - 0.05 * k for k in range(K)], 1024)
    peers = [wl.flat_normal(plan.bucket_elems()[0], "bf16", 1e-3, 60 + k, DEV) for k in range(1, K)]
    slot = torch.zeros_like(peers[0])
    if resident:
        plan.kt_plan_set_weights(weights)
        plan.kt_plan_set_sgd(0.5, 0.05, 0.9, 5e-4)
        plan.kt_fused_step_sgd_resident(-1, grads, peers, K, params, momenta, models, False)
    else:
        plan.kt_fused_step_sgd(-1, grads, peers, K, weights, 0.5, params, momenta, models, 0.05, 0.9, 5e-4, False)
    plan.kt_bucket_pack(-1, grads, [slot])
    plan.kt_weighted_reduce(-1, [slot] + peers, K, weights, [slot])
    plan.kt_bucket_unpack_sgd_master(-1, [slot], 0.5, views(mine[0], 3), views(mine[1], 2), views(mine[2], 1), 0.05, 0.9, 5e-4, False)
    torch.cuda.synchronize()
    for got, want in zip(flats[1:], mine):          # whole memory: what lies beside the tensors as well
        kind = torch.int32 if got.dtype == torch.float32 else torch.int16
        assert torch.equal(got.view(kind), want.view(kind))
    assert not torch.equal(flats[1], wl.flat_normal(total + 3, "f32", 2e-2, 51, DEV))

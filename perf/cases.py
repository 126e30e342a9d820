"""What the library is timed on: whole passes of the gradient path through the public entry points.

A case is a gradient set (tensor shapes, element type), the number of peer copies K, the bucket
layout, and the calls that a training program makes on them:

  step       kt_bucket_pack, kt_weighted_reduce in place over slot 0, kt_bucket_unpack_scale
  reduce     kt_weighted_reduce alone (the gradients already live in the buckets)
  fused      kt_fused_step
  sgd        kt_bucket_pack, kt_weighted_reduce in place, kt_bucket_unpack_sgd[_master]
  fused_sgd  kt_fused_step_sgd (with the bf16 model copy where `master` is set)

Keys of a case: `model` (a named set of workloads.py, or "decoder" / "ragged" with sizes of their
own), `dtype`, `K`, `cap_mib` (bucket cap, 0 = one bucket), `align` (bytes; the element size = the
dense layout of DDP's buckets), `views` (the gradients are views into one dense buffer at any
element address, as with DDP's gradient_as_bucket_view), `lists` (the program passes lists of
tensors, whose addresses may be new on every step; otherwise pointer arrays kept from
Plan.marshal), `by_bucket` (one set of calls per bucket, as buckets become ready during backward).
"""
import ctypes
import math
import random

import torch

import paper_2505_10183_amd as kt
from paper_2505_10183_amd import workloads

MIB = 1 << 20
SCALE, LR, MOMENTUM, WEIGHT_DECAY = 1.0, 0.05, 0.9, 5e-4


def listed():
    def case(name, op, model, dtype, K, cap_mib, **more):
        c = {"name": name, "op": op, "model": model, "dtype": dtype, "K": K, "cap_mib": cap_mib,
             "align": 16, "views": False, "lists": False, "by_bucket": False, "master": False}
        c.update(more)
        return c

    return [
        # the smallest real set (an MLP, 6 tensors, one bucket): three launches, latency alone
        case("mlp_step", "step", "mlp", "f32", 2, 0),
        # the paper's own network: 158 small tensors, gradients handed over as lists on every step
        # (optimizers that set gradients to None get new tensors each time)
        case("mobilenetv2_step_lists", "step", "mobilenetv2", "f32", 4, 25, lists=True),
        # the same network, copies to updated parameters in one call
        case("mobilenetv2_fused_sgd", "fused_sgd", "mobilenetv2", "f32", 4, 25),
        # ResNet-18: the one-call gradient step on a middle-sized set
        case("resnet18_fused", "fused", "resnet18", "f32", 4, 25),
        # odd tensor sizes in DDP's dense layout, bf16, gradients as views of the bucket memory
        case("ragged_dense_step_bf16", "step", "ragged", "bf16", 3, 25, align=2, views=True,
             count=400, largest=700001),
        # odd tensor sizes, 16-byte layout, mixed-precision SGD on unpack
        case("ragged_sgd_master_bf16", "sgd", "ragged", "bf16", 5, 25, count=600, largest=1000001, master=True),
        # a transformer of odd width in the dense layout, fp32, one call per step
        case("odd_decoder_dense_fused", "fused", "decoder", "f32", 4, 25, align=4, views=True,
             d=1001, layers=6, vocab=5003),
        # ViT-B/16, all buckets in one batched launch per call
        case("vit_b16_step", "step", "vit_b16", "f32", 8, 25),
        # ViT-B/16, bucket by bucket, as a gradient hook calls it during backward
        case("vit_b16_by_bucket", "step", "vit_b16", "f32", 8, 25, by_bucket=True),
        # many peers: 16 copies of ViT-B/16's buckets
        case("vit_b16_reduce_k16", "reduce", "vit_b16", "f32", 16, 25),
        # the 1.3B decoder in bf16: the chained step and the single pass of mixed-precision training
        case("decoder_1p3b_step", "step", "decoder_1p3b", "bf16", 8, 64),
        case("decoder_1p3b_fused_sgd", "fused_sgd", "decoder_1p3b", "bf16", 8, 64, master=True),
    ]


def draw(rng: random.Random):
    op = rng.choice(["step", "step", "reduce", "fused", "sgd", "fused_sgd"])
    dtype = rng.choice(["f32", "bf16"])
    es = 4 if dtype == "f32" else 2
    K = rng.choice([2, 3, 4, 4, 5, 6, 7, 8, 8, 12, 16])
    dense = rng.random() < 0.3
    c = {"op": op, "dtype": dtype, "K": K, "align": es if dense else 16, "views": dense and rng.random() < 0.7,
         "lists": rng.random() < 0.2, "by_bucket": False, "master": op in ("sgd", "fused_sgd") and dtype == "bf16" and rng.random() < 0.7}
    # elements, spread over their logarithm; the most that all copies and the optimizer state may take is bounded
    most = min(9e8, 14e9 / ((K + 1) * es + (10 if op in ("sgd", "fused_sgd") else 0)))
    n = int(math.exp(rng.uniform(math.log(2e5), math.log(most))))
    if rng.random() < 0.35:
        count = rng.randint(20, 800)
        # sizes are log-uniform between 1 and `largest`: their mean is about largest / log(largest)
        per = max(64, n // count)
        c.update(model="ragged", count=count, largest=int(per * math.log(per) * 1.2) | 1)
    else:
        layers = rng.randint(1, 24)
        d = max(24, int(math.sqrt(n / (12.0 * layers + 6))))
        if rng.random() < 0.6:
            d = max(16, d // 16 * 16)
        c.update(model="decoder", d=d, layers=layers, vocab=max(16, 6 * d + rng.randint(0, 63)))
    # DDP's 25 MiB, larger buckets for larger sets, or one bucket
    total = sum(_numels(c))
    cap = rng.choice([0, 25, 25, 25, 64]) if total * es < 512 * MIB else rng.choice([25, 64, 64, 128])
    c["cap_mib"] = cap
    c["by_bucket"] = 1 < total * es / max(1, cap * MIB) <= 24 and cap > 0 and op != "sgd" and rng.random() < 0.25
    return c


# ---- gradient sets and their layout -----------------------------------------------------------


def _numels(c):
    if c["model"] == "ragged":
        r = random.Random(c["count"] * 7919 + c["largest"])
        sizes = [max(1, int(math.exp(r.uniform(0.0, math.log(c["largest"]))))) for _ in range(c["count"])]
        return sizes
    if c["model"] == "decoder":
        d = c["d"]
        s = [c["vocab"] * d]
        for _ in range(c["layers"]):
            s += [d, d, 3 * d * d, 3 * d, d * d, d, d, d, 4 * d * d, 4 * d, 4 * d * d, d]
        return s + [d, d]
    return workloads.get(c["model"]).numels


def _throughputs(c):
    if c["model"] not in ("ragged", "decoder"):
        w = workloads.get(c["model"])
        if w.K == c["K"]:
            return list(w.throughputs), w.global_batch
    # devices of unequal speed, the fastest first
    return [round(1.0 - 0.6 * k / c["K"], 3) for k in range(c["K"])], 1024


def _torch_dtype(c):
    return torch.float32 if c["dtype"] == "f32" else torch.bfloat16


def _arena(numels, dtype, dense):
    """One allocation holding all tensors, and the tensors: at the 512-byte steps at which torch's
    allocator places tensors of their own, or densely."""
    step = 1 if dense else 512 // torch.empty((), dtype=dtype).element_size()
    offs, at = [], 0
    for n in numels:
        offs.append(at)
        at += -(-n // step) * step
    flat = torch.zeros(at, dtype=dtype, device="cuda")
    return flat, [flat[o:o + n] for o, n in zip(offs, numels)]


def _buckets(c):
    """The documented layout: tensors in order, each at a multiple of `align`; a bucket closes before a
    tensor that would take it over the cap, and its length is rounded up to `align`.
    [(length, [(tensor, offset), ...]), ...]"""
    es = 4 if c["dtype"] == "f32" else 2
    a, cap = c["align"] // es, c["cap_mib"] * MIB // es
    out, end, inside = [], 0, []
    for t, n in enumerate(_numels(c)):
        off = -(-end // a) * a
        if cap and inside and -(-(off + n) // a) * a > cap:
            out.append((-(-end // a) * a, inside))
            off, inside = 0, []
        inside.append((t, off))
        end = off + n
    out.append((-(-end // a) * a, inside))
    return out


def _inputs(c, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    numels, dt, K = _numels(c), _torch_dtype(c), c["K"]
    lens = [n for n, _ in _buckets(c)]

    def normal(n, sigma, dtype):
        return torch.empty(n, dtype=dtype, device="cuda").normal_(0.0, sigma, generator=g)

    s = {}
    if c["op"] == "reduce":
        # in place over the first copy, which is what the gradients' own bucket memory holds
        s["slot0_flat"], s["slot0"] = _arena(lens, dt, False)
        for t in s["slot0"]:
            t.normal_(0.0, 1e-3, generator=g)
    else:
        s["grads_flat"], s["grads"] = _arena(numels, dt, c["views"])
        for t in s["grads"]:
            t.normal_(0.0, 1e-3, generator=g)
        if c["op"] in ("step", "sgd"):
            s["slot0_flat"], s["slot0"] = _arena(lens, dt, False)
    # buckets that arrived from the other devices, each in an allocation of its own
    s["peers"] = [[normal(n, 1e-3, dt) for n in lens] for _ in range(K - 1)]
    if c["op"] in ("step", "fused"):
        s["out_flat"], s["out"] = _arena(numels, dt, c["views"])
    if c["op"] in ("sgd", "fused_sgd"):
        for name, sigma in (("params", 2e-2), ("momenta", 1e-3)):
            s[name + "_flat"], s[name] = _arena(numels, torch.float32, False)
            for t in s[name]:
                t.normal_(0.0, sigma, generator=g)
        s["models_flat"], s["models"] = _arena(numels, torch.bfloat16, False) if c["master"] else (None, None)
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"], K = case, case["K"]
    plan = s["plan"] = kt.Plan(_numels(case), case["dtype"], case["cap_mib"] * MIB, case["align"])
    thr, B = _throughputs(case)
    _, s["weights"] = kt.kt_plan_shares(thr, B)
    nb = plan.num_buckets
    s["others"] = [s["peers"][k][b] for b in range(nb) for k in range(K - 1)]
    if "slot0" in s:
        s["all"] = [s["slot0"][b] if k == 0 else s["peers"][k - 1][b] for b in range(nb) for k in range(K)]
    if not case["lists"]:       # pointer arrays marshalled once, as the binding offers
        for k in ("grads", "slot0", "out", "params", "momenta", "models", "others", "all"):
            if s.get(k) is not None:
                s[k] = plan.marshal(s[k])
        s["weights"] = (ctypes.c_float * K)(*s["weights"])
    s["buckets"] = range(nb) if case["by_bucket"] else (-1,)
    return s


def run(s):
    c, p, K, w = s["case"], s["plan"], s["case"]["K"], s["weights"]
    op = c["op"]
    for b in s["buckets"]:
        if op in ("step", "sgd"):
            p.kt_bucket_pack(b, s["grads"], s["slot0"])
        if op in ("step", "sgd", "reduce"):
            p.kt_weighted_reduce(b, s["all"], K, w, s["slot0"])
        if op == "step":
            p.kt_bucket_unpack_scale(b, s["slot0"], SCALE, s["out"])
        elif op == "fused":
            p.kt_fused_step(b, s["grads"], s["others"], K, w, SCALE, s["out"])
        elif op == "sgd" and c["master"]:
            p.kt_bucket_unpack_sgd_master(b, s["slot0"], SCALE, s["params"], s["momenta"], s["models"], LR, MOMENTUM,
                                          WEIGHT_DECAY, False)
        elif op == "sgd":
            p.kt_bucket_unpack_sgd(b, s["slot0"], SCALE, s["params"], s["momenta"], LR, MOMENTUM, WEIGHT_DECAY, False)
        elif op == "fused_sgd":
            p.kt_fused_step_sgd(b, s["grads"], s["others"], K, w, SCALE, s["params"], s["momenta"], s["models"], LR,
                                MOMENTUM, WEIGHT_DECAY, False)
    return {k: s[k + "_flat"] for k in ("slot0", "out", "params", "momenta", "models") if s.get(k + "_flat") is not None}


def work(case):
    """Inputs read once, outputs written once: the local gradients, the K-1 other copies, and what the
    calls leave behind (reduced buckets, gradients, parameters, momentum, model copy)."""
    e, es, K, op = sum(_numels(case)), 4 if case["dtype"] == "f32" else 2, case["K"], case["op"]
    per = K * es
    per += es if op in ("step", "sgd", "reduce") else 0     # the reduced bucket
    per += es if op in ("step", "fused") else 0             # the gradients
    per += 16 if op in ("sgd", "fused_sgd") else 0          # parameters and momentum, read and written
    per += 2 if case["master"] else 0
    flops = 2 * K - 1 + (1 if op in ("step", "fused") else 7 if op in ("sgd", "fused_sgd") else 0)
    return {"bytes": e * per, "flops": e * flops}


def tolerance(case):
    if case["dtype"] == "f32":
        # against exact(): 4e-8 to 1e-7 (2-norm), 5e-7 at most of an element against the root mean square
        return {"rel": 4e-7, "max": 4e-6}
    # one rounding to bf16 of the sum (2^-9 at most of an element, 1.7e-3 in the 2-norm), two with the model copy
    return {"rel": 7e-3, "max": 2e-2}


def exact(case, seed):
    """The same in 64 bits: the weighted sum, the scale and the update in double, nothing rounded between."""
    s = _inputs(case, seed)
    thr, B = _throughputs(case)
    total = 0.0
    for t in thr:
        total += t
    quota = [t / total * B for t in thr]
    share = [math.floor(q) for q in quota]
    for k in sorted(range(len(thr)), key=lambda k: share[k] - quota[k])[:B - sum(share)]:
        share[k] += 1
    w = [b / B for b in share]
    res = {}
    tens = {}

    def like(name):
        flat = s[name + "_flat"]
        res[name] = torch.zeros(flat.numel(), dtype=torch.float64, device="cuda")
        return [res[name][t.storage_offset():t.storage_offset() + t.numel()] for t in s[name]]

    for name in ("slot0", "out", "params", "momenta", "models"):
        if s.get(name + "_flat") is not None:
            tens[name] = like(name)
    for b, (n, inside) in enumerate(_buckets(case)):
        acc = torch.zeros(n, dtype=torch.float64, device="cuda")
        if case["op"] == "reduce":
            acc += s["slot0"][b]
        else:
            for t, off in inside:
                acc[off:off + s["grads"][t].numel()] = s["grads"][t]
        acc *= w[0]
        for k in range(1, case["K"]):
            acc.add_(s["peers"][k - 1][b], alpha=w[k])
        if "slot0" in tens:
            tens["slot0"][b].copy_(acc)
        if case["op"] == "reduce":
            continue
        for t, off in inside:
            g = acc[off:off + s["grads"][t].numel()]
            if "out" in tens:
                tens["out"][t].copy_(g * SCALE)
            if "params" in tens:
                p = s["params"][t].double()
                v = MOMENTUM * s["momenta"][t].double() + (g * SCALE + WEIGHT_DECAY * p)
                p = p - LR * v
                tens["params"][t].copy_(p)
                tens["momenta"][t].copy_(v)
                if "models" in tens:
                    tens["models"][t].copy_(p)
    return res

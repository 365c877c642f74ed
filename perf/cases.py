"""Workloads by which the speed of the library is followed.

A case is one pass that a user of the framework has it make, through the Python
methods of SSNet (one per C entry point) and the layer-stack harness Chain:

  dense    one dense layer on shares.  packed: the layer-by-layer route with weights
           prepared once (share + limb tiles, product, reduction + truncation +
           opening).  Otherwise the plain calls, both operands fresh share matrices
           (linear_mod, degree_reduce, truncate, reconstruct).
  conv     one convolution layer with ReLU on shares, weights prepared once: limb
           planes where the channel count allows them, the im2col route otherwise.
  stack    a whole network.  opened: every layer's result is opened (the share
           arithmetic of the headline benchmark); otherwise everything stays on
           shares, ReLU and pooling included, and only the logits are opened.
  bulk     sharing a tensor and reconstructing it from the first and the last t+1
           parties.
  reduce   degree reduction with re-randomisation and truncation of product shares.
  pool     ReLU and pooling on shares under the trusted source's masks.

n, t: the scheme (n parties, degree t); prime: 61 or 45 for 2^61 - 1 or 2^45 - 55.
"""
import math

import torch

from paper_2406_02629_amd import P45, P61, SSNet
from paper_2406_02629_amd import fixedpoint as fx
from paper_2406_02629_amd.chain import Chain
from ssnet_inputs import alexnet_chain, lenet_chain, pooling_of, resnet_basic_chain, resnet_chain, vgg16_chain

SCHEMES = [(3, 1), (5, 2), (3, 1), (5, 2), (4, 1), (7, 3)]   # the two that the paper evaluates, and others


def listed():
    return [
        # smallest: the tiny secure matrix product, all steps, bound by launches
        dict(name="dense_tiny", kind="dense", n=3, t=1, prime=61, M=64, K=256, N=128, packed=True),
        # two share matrices that change from call to call, through the five plain calls; ragged sizes
        dict(name="dense_fresh", kind="dense", n=4, t=1, prime=61, M=500, K=1201, N=333, packed=False),
        # one ResNet-style convolution layer on a batch of eight images
        dict(name="conv_layer", kind="conv", n=3, t=1, prime=61, B=8, C=64, H=56, Co=64, k=3, stride=1),
        # a small network at batch 1: latency of many tiny calls
        dict(name="lenet", kind="stack", arch="lenet", image=28, n=3, t=1, prime=61, batch=1, opened=False),
        # large dense layers behind small maps, a few images
        dict(name="vgg16_b4", kind="stack", arch="vgg16", image=32, n=3, t=1, prime=61, batch=4, opened=False),
        # the layer-by-layer stacks of the benchmark, five parties
        dict(name="resnet50_opened", kind="stack", arch="resnet50", image=224, n=5, t=2, prime=61, batch=1, opened=True),
        dict(name="resnet152_opened", kind="stack", arch="resnet152", image=224, n=5, t=2, prime=61, batch=1, opened=True),
        # the paper's own setting: three parties, its prime, one image, everything on shares
        dict(name="resnet50_p45", kind="stack", arch="resnet50", image=224, n=3, t=1, prime=45, batch=1, opened=False),
        # throughput: a batch, everything on shares
        dict(name="resnet50_b8", kind="stack", arch="resnet50", image=224, n=5, t=2, prime=61, batch=8, opened=False),
        # data owner's side at its largest
        dict(name="bulk", kind="bulk", n=5, t=2, prime=61, count=1 << 28),
        # a scheme other than the two of the paper, ragged count
        dict(name="reduce_7_3", kind="reduce", n=7, t=3, prime=61, count=300001),
        # the pooling point after a ResNet stem, three images
        dict(name="pool_stem", kind="pool", n=5, t=2, prime=61, planes=192, H=112, k=3, stride=2, pad=1, mode="max"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


ARCHES = {   # smallest and largest image, largest batch
    "lenet": (24, 64, 64), "vgg16": (32, 64, 8), "resnet18": (64, 224, 8), "resnet50": (64, 224, 8),
    "resnet101": (96, 224, 2), "alexnet": (131, 227, 4),
}
MAX_STACK_MACS = 160e9   # over all parties: below the largest listed case


def draw(rng):
    kind = rng.choice(["dense", "dense", "conv", "conv", "stack", "stack", "stack", "stack", "bulk", "reduce", "pool"])
    n, t = rng.choice(SCHEMES)
    case = dict(kind=kind, n=n, t=t, prime=rng.choice([61, 61, 45]))
    if kind == "dense":
        case.update(M=_log(rng, 1, 2048), K=_log(rng, 48, 4800), N=_log(rng, 10, 4096), packed=rng.random() < 0.6)
    elif kind == "conv":
        case.update(B=_log(rng, 1, 8), C=rng.choice([3, 20, 64, 64, 128, 256, 512]), H=_log(rng, 7, 64),
                    Co=_log(rng, 16, 512), k=rng.choice([1, 3, 3, 5]), stride=rng.choice([1, 1, 2]))
    elif kind == "stack":
        arch = rng.choice(sorted(ARCHES))
        lo, hi, most = ARCHES[arch]
        case.update(arch=arch, image=rng.randint(lo, hi), batch=_log(rng, 1, most), opened=rng.random() < 0.4)
        while case["n"] * case["batch"] * sum(L.macs for L in _layers(case)) > MAX_STACK_MACS:
            case["batch"] -= 1
    elif kind in ("bulk", "reduce"):
        case.update(count=_log(rng, 1000, 1 << (27 if kind == "bulk" else 22)))
    else:
        k = rng.choice([2, 2, 3, 7])
        case.update(planes=_log(rng, 16, 1024), H=rng.randint(max(7, k), 112), k=k, stride=2 if k < 4 else k,
                    pad=1 if k == 3 else 0, mode=rng.choice(["max", "sum"]))
    return case


def _layers(case):
    arch, image = case["arch"], case["image"]
    if arch == "lenet":
        return lenet_chain(image)
    if arch == "vgg16":
        return vgg16_chain(image)
    if arch == "alexnet":
        return alexnet_chain(image)
    if arch == "resnet18":
        return resnet_basic_chain(18, image)
    return resnet_chain(int(arch[6:]), image)


def _prime(case):
    return P45 if case["prime"] == 45 else P61


def _scheme(case, seed):
    # the paper's fraction bits for its prime keep every activation inside the 16 bits of its mask
    return SSNet(case["n"], case["t"], f=12 if case["prime"] == 45 else 13, seed=seed, p=_prime(case))


def _normal(gen, ss, shape, sigma=1.0):
    """fixed-point field elements of N(0, sigma^2)"""
    return fx.encode(torch.randn(shape, generator=gen, dtype=torch.float64, device="cuda") * sigma, ss.f, ss.p)


def _uniform(gen, shape, bound):
    return torch.randint(0, bound, shape, generator=gen, dtype=torch.int64, device="cuda")


def _empty(*shape):
    return torch.empty(shape, dtype=torch.int64, device="cuda")


def _in_one(tensors):
    """(one zeroed buffer, views of it in place of the tensors, each on a 256-byte boundary)"""
    starts, total = [], 0
    for x in tensors:
        starts.append(total)
        total += (x.numel() + 31) // 32 * 32
    flat = torch.zeros(total, dtype=torch.int64, device="cuda")
    return flat, [flat[s:s + x.numel()].view(x.shape) for s, x in zip(starts, tensors)]


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    ss = _scheme(case, seed)
    s = dict(case=case, ss=ss, ids=list(range(1, ss.k + 1)))
    n, kind = ss.n, case["kind"]
    if kind == "dense":
        M, K, N = case["M"], case["K"], case["N"]
        x, w = _normal(gen, ss, (M, K)), ss.share(_normal(gen, ss, (K, N), math.sqrt(2.0 / K)), stream_id=1)
        if case["packed"]:
            s.update(x=x, w=ss.pack_weights_linear(w), xs=_empty(n, M, K),
                     tiles=torch.empty(n * ss.lib.ssnet_packed_weight_bytes(M, K), dtype=torch.uint8, device="cuda"))
        else:
            s.update(xs=ss.share(x, stream_id=2), w=w, reduced=_empty(n, M, N), truncated=_empty(n, M, N))
        s.update(y=_empty(n, M, N), opened=_empty(M, N))
    elif kind == "conv":
        B, C, H, Co, k = case["B"], case["C"], case["H"], case["Co"], case["k"]
        geom = (B, C, H, H, Co, k, k, case["stride"], k // 2)
        Ho = (H + 2 * (k // 2) - k) // case["stride"] + 1
        w = ss.share(_normal(gen, ss, (Co, C, k, k), math.sqrt(2.0 / (C * k * k))), stream_id=1)
        planes = ss.planes_supported(B, C, H, H)
        s.update(x=_normal(gen, ss, (B, C, H, H)), xs=_empty(n, B, C, H, H), y=_empty(n, B, Co, Ho, Ho), geom=geom,
                 w=ss.pack_weights_conv_taps(w) if planes else ss.pack_weights_conv(w), out=_empty(n, B, Co, Ho, Ho),
                 masks=ss.nonlinear_masks((B, Co, Ho, Ho), stream_id=4), planes=None)
        if planes:
            s["planes"] = torch.empty(n * ss.lib.ssnet_conv_planes_bytes(B, C, H, H), dtype=torch.uint8, device="cuda")
    elif kind == "stack":
        chain = Chain(ss, _layers(case), batch=case["batch"], image_seed=seed, weight_seed_base=seed + 1)
        s["shares"], chain.y = _in_one(chain.y)
        if case["opened"]:
            s["opened"], chain.rec = _in_one(chain.rec)
            chain.forward_prepare()
        else:
            chain.secure_prepare(pool_on_shares=True)
        s["chain"] = chain
    elif kind == "bulk":
        s.update(x=_uniform(gen, (case["count"],), ss.p), shares=_empty(n, case["count"]), first=_empty(case["count"]),
                 last=_empty(case["count"]), last_ids=list(range(n - ss.t, n + 1)))
    elif kind == "reduce":
        # degree-2t shares of products of two fixed-point numbers
        v = fx.from_signed(_uniform(gen, (case["count"],), 1 << 34) - (1 << 33), ss.p)
        s.update(c=ss.share(v, stream_id=1, degree=2 * ss.t), out=_empty(n, case["count"]))
    else:
        planes, H, k, st, pad = case["planes"], case["H"], case["k"], case["stride"], case["pad"]
        v = fx.from_signed(_uniform(gen, (planes, H, H), 1 << 14) - (1 << 13), ss.p)
        geom = ((k, k), (st, st), (pad, pad))
        b, bi = ss.pool_masks(planes, H, H, *geom, stream_id=2)
        s.update(x=ss.share(v, stream_id=1), beta=b, betainv=bi, geom=geom, out=torch.empty_like(bi),
                 mode=SSNet.POOL_MAX if case["mode"] == "max" else SSNet.POOL_SUM)
    return s


def run(s):
    case, ss = s["case"], s["ss"]
    kind = case["kind"]
    if kind == "dense":
        if case["packed"]:
            M, K, N = case["M"], case["K"], case["N"]
            ss.share_packed(s["x"], stream_id=2, out=s["xs"], packed=s["tiles"])
            ss.linear_product_prepacked(s["tiles"], s["w"], M, K, N)
            ss.degree_reduce_truncate_reconstruct(None, stream_id=3, ids=s["ids"], out=s["y"], secret=s["opened"])
            return {"input shares": s["xs"], "shares": s["y"], "opened": s["opened"]}
        ss.linear_mod(s["xs"], s["w"], out=s["y"])
        ss.degree_reduce(s["y"], stream_id=3, out=s["reduced"])
        ss.truncate(s["reduced"], stream_id=3, out=s["truncated"])
        ss.reconstruct(s["truncated"], s["ids"], out=s["opened"])
        return {"product": s["y"], "reduced": s["reduced"], "shares": s["truncated"], "opened": s["opened"]}
    if kind == "conv":
        if s["planes"] is not None:
            ss.share_planes(s["x"], stream_id=2, out=s["xs"], planes=s["planes"])
            ss.conv_mod_planes(s["planes"], s["w"], *s["geom"], out=s["y"])
        else:
            ss.share(s["x"], stream_id=2, out=s["xs"])
            ss.conv_mod_packed(s["xs"], s["w"], *s["geom"][4:], out=s["y"])
        ss.reduce_truncate_relu(s["y"], 3, *s["masks"], out=s["out"])
        return {"input shares": s["xs"], "product": s["y"], "shares": s["out"]}
    if kind == "stack":
        chain = s["chain"]
        if case["opened"]:
            chain.forward_timed()
            return {"shares": s["shares"], "opened": s["opened"]}
        chain.secure_timed()
        return {"shares": s["shares"], "pooled": [x for x in chain.pooled if x is not None], "logits": chain.rec[-1]}
    if kind == "bulk":
        ss.share(s["x"], stream_id=1, out=s["shares"])
        ss.reconstruct(s["shares"], s["ids"], out=s["first"])
        ss.reconstruct(s["shares"], s["last_ids"], out=s["last"])
        return {"shares": s["shares"], "first": s["first"], "last": s["last"]}
    if kind == "reduce":
        return ss.degree_reduce_truncate(s["c"], stream_id=3, out=s["out"])
    return ss.relu_pool(s["x"], s["beta"], s["betainv"], *s["geom"], s["mode"], out=s["out"])


def work(case):
    """bytes: operands and weights read once, results written once, 8 bytes per field element (messages between
    the parties not counted).  flops: one multiplication and one addition in the field per multiply-accumulate of
    the linear layers, all parties; element-wise steps are counted by their bytes alone."""
    n, t, kind = case["n"], case["t"], case["kind"]
    if kind == "dense":
        M, K, N = case["M"], case["K"], case["N"]
        words = M * K * (1 + n) + n * K * N + M * N * (n + 1) if case["packed"] else n * (M * K + K * N + 3 * M * N) + M * N
        return {"bytes": 8 * words, "flops": 2 * n * M * K * N}
    if kind == "conv":
        B, C, H, Co, k = case["B"], case["C"], case["H"], case["Co"], case["k"]
        Ho = (H + 2 * (k // 2) - k) // case["stride"] + 1
        words = B * C * H * H * (1 + n) + n * Co * C * k * k + 4 * n * B * Co * Ho * Ho
        return {"bytes": 8 * words, "flops": 2 * n * B * Ho * Ho * C * k * k * Co}
    if kind == "stack":
        words, macs, B = 0, 0, case["batch"]
        for L in _layers(case):
            fan_in, out = B * L.cin * L.hin * L.hin, B * L.cout * L.M
            macs += B * L.macs
            words += n * L.K * L.cout + n * out
            if case["opened"]:
                words += fan_in * (1 + n) + out          # the layer's input shared, its result opened
            elif L.post is not None:
                words += n * out                         # mask shares
                spec = pooling_of(L)
                pooled = out if spec is None else B * L.cout * ((L.hout + 2 * spec[3] - spec[1]) // spec[2] + 1) ** 2
                words += n * pooled * (1 if spec is None else 2)
        return {"bytes": 8 * words, "flops": 2 * n * macs}
    if kind == "bulk":
        return {"bytes": 8 * case["count"] * (1 + n + 2 * (t + 1) + 2), "flops": 0}
    if kind == "reduce":
        return {"bytes": 8 * case["count"] * (2 * t + 1 + n), "flops": 0}
    planes, H, k, st, pad = case["planes"], case["H"], case["k"], case["stride"], case["pad"]
    Ho = (H + 2 * pad - k) // st + 1
    return {"bytes": 8 * planes * (2 * (2 * t + 1) * H * H + 2 * n * Ho * Ho), "flops": 0}


def tolerance(case):
    return "exact"   # field elements

"""Measured workloads of the SqueezeNet forward library: what a program that uses it calls, over the range of sizes it meets.

A case is a plain dict.  Its "kind" names the entry point:
  net         the whole network on kernels packed once (sq_squeezenet_forward_packed, or sq_squeezenet_forward_bf16 for
              "dtype": "bf16"), 224 x 224 RGB images, 1000 class probabilities per image
  fire        one fire layer on fp32 NCHW maps: sq_fire_forward, or sq_fire_forward_packed with "packed"
  fire_blocked  one fire layer of the reduced-precision network: blocked bfloat16 map in and out
  conv        one convolution with bias and ReLU, scratch given (sq_conv2d_forward_ws), fp32 or bfloat16 operands
  stem        the 7x7 stride-2 layer on an image and the 3x3 stride-2 max pooling behind it, as two calls
  classifier  1x1 convolution, global average pooling and softmax as one call
Workspaces, packed kernels and output buffers are made once, as a serving program keeps them.
"""
import math

import torch

import paper_1611_07151_amd as sq

# Cin, squeeze layers, expand layers (of each of the two expands), extent of the map: the network's eight fire layers.
FIRES = ((96, 16, 64, 55), (128, 16, 64, 55), (128, 32, 128, 55), (256, 32, 128, 27),
         (256, 48, 192, 27), (384, 48, 192, 27), (384, 64, 256, 27), (512, 64, 256, 13))
POOL_BEHIND = (2, 6)          # fire layers (by position) that a 3x3 stride-2 max pooling follows


def listed():
    return [
        # one photograph, the latency of a whole prediction
        {"name": "net_f32_b1", "kind": "net", "dtype": "f32", "n": 1},
        # the throughput benchmark: 64 photographs at a time
        {"name": "net_f32_b64", "kind": "net", "dtype": "f32", "n": 64},
        # the same in the reduced-precision mode
        {"name": "net_bf16_b64", "kind": "net", "dtype": "bf16", "n": 64},
        # a fire layer alone, one image, kernels as they lie: the smallest call a program makes
        {"name": "fire2_f32_b1", "kind": "fire", "packed": False, "n": 1, "cin": 96, "csq": 16, "ce": 64, "h": 55, "w": 55},
        # a middle fire layer at an ordinary serving batch, kernels packed
        {"name": "fire6_f32_b16", "kind": "fire", "packed": True, "n": 16, "cin": 256, "csq": 48, "ce": 192, "h": 27, "w": 27},
        # the fire layer with the most arithmetic at the benchmark's batch, kernels packed
        {"name": "fire8_f32_b64", "kind": "fire", "packed": True, "n": 64, "cin": 384, "csq": 64, "ce": 256, "h": 27, "w": 27},
        # the reduced-precision fire layer with the largest maps
        {"name": "fire4_bf16_b64", "kind": "fire_blocked", "n": 64, "cin": 128, "csq": 32, "ce": 128, "h": 55, "w": 55},
        # convolutions of another network: 5x5 on 27 x 27 maps and 3x3 on 13 x 13 maps
        {"name": "conv5x5_f32_b16", "kind": "conv", "dtype": "f32", "n": 16, "cin": 96, "cout": 256, "k": 5, "h": 27, "w": 27},
        {"name": "conv3x3_f32_b7", "kind": "conv", "dtype": "f32", "n": 7, "cin": 256, "cout": 384, "k": 3, "h": 13, "w": 13},
        # the reduced-precision layer sweep at its batch of 256: bfloat16 operands, fp32 results
        {"name": "conv3x3_bf16_b256", "kind": "conv", "dtype": "bf16", "n": 256, "cin": 32, "cout": 128, "k": 3, "h": 55, "w": 55},
        # the first layer and the pooling behind it on a ragged image
        {"name": "stem_f32_b8", "kind": "stem", "n": 8, "h": 227, "w": 227, "pad": 0},
        # the classifier end at an ordinary batch
        {"name": "classifier_f32_b32", "kind": "classifier", "n": 32, "cin": 512, "cout": 1000, "h": 13, "w": 13},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


MOST_WORK = 1.1e9     # of a drawn case, in the unit of _cost: below the batch-64 network's 2.1e9


def _cost(case):
    w = work(case)
    return max(w["bytes"], w["flops"] / 50)


def draw(rng):
    kind = rng.choice(("net", "net", "fire", "fire", "fire_blocked", "conv", "conv", "conv_bf16", "stem", "classifier"))
    n = _log(rng, 1, 64)
    if kind == "net":
        case = {"kind": "net", "dtype": rng.choice(("f32", "bf16")), "n": n}
    elif kind in ("fire", "fire_blocked"):
        cin, csq, ce, h = rng.choice(FIRES)
        h = rng.randint(max(7, h - 20), h + 1)
        case = {"kind": kind, "n": n, "cin": cin, "csq": csq, "ce": ce, "h": h, "w": max(7, h + rng.randint(-5, 5))}
        if kind == "fire":
            case["packed"] = rng.random() < 0.5
    elif kind == "conv":
        h = _log(rng, 7, 56)
        case = {"kind": "conv", "dtype": "f32", "n": n, "cin": rng.choice((16, 24, 32, 48, 64, 96, 128, 256, 384)),
                "cout": rng.choice((16, 40, 64, 96, 128, 192, 256, 384)), "k": rng.choice((1, 3, 3, 5)), "h": h,
                "w": max(7, h + rng.randint(-4, 4))}
    elif kind == "conv_bf16":
        cin, csq, ce, h = rng.choice(FIRES)
        a, b, k = rng.choice(((cin, csq, 1), (csq, ce, 1), (csq, ce, 3), (csq, ce, 3)))
        case = {"kind": "conv", "dtype": "bf16", "n": _log(rng, 16, 256), "cin": a, "cout": b, "k": k, "h": h, "w": h}
    elif kind == "stem":
        h = rng.randint(96, 256)
        case = {"kind": "stem", "n": n, "h": h, "w": h + rng.randint(-20, 20), "pad": rng.choice((0, 2, 3))}
    else:
        h = rng.randint(6, 15)
        case = {"kind": "classifier", "n": n, "cin": rng.choice((128, 256, 512)), "cout": rng.choice((10, 100, 1000)), "h": h, "w": h}
    while _cost(case) > MOST_WORK:
        case["n"] = max(1, case["n"] // 2)
    return case


# ------------------------------------------------------------------------------------------------ what a pass is worth
def _conv_work(n, cin, cout, k, ho, wo, hi, wi, size_in=4, size_out=4):
    return (size_in * (n * cin * hi * wi + cout * cin * k * k) + 4 * cout + size_out * n * cout * ho * wo,
            2.0 * n * cout * cin * k * k * ho * wo)


def _fire_work(n, cin, csq, ce, h, w, size):
    weights = csq * cin + ce * csq * 10
    return (size * (n * h * w * (cin + 2 * ce) + weights) + 4 * (csq + 2 * ce),
            2.0 * n * h * w * weights)


def work(case):
    n, kind = case["n"], case["kind"]
    if kind == "net":
        # image, the 1 248 424 parameters and the probabilities; the multiply-accumulates of the layer definitions
        kernel_bytes = 4 if case["dtype"] == "f32" else 2
        return {"bytes": 4.0 * n * 3 * 224 * 224 + kernel_bytes * 1248424.0 + 4.0 * n * 1000, "flops": 2.0 * 832667936 * n}
    if kind in ("fire", "fire_blocked"):
        b, f = _fire_work(n, case["cin"], case["csq"], case["ce"], case["h"], case["w"], 4 if kind == "fire" else 2)
    elif kind == "conv":
        h, w = case["h"], case["w"]
        b, f = _conv_work(n, case["cin"], case["cout"], case["k"], h, w, h, w, 4 if case["dtype"] == "f32" else 2)
    elif kind == "stem":
        ho, wo = _stem_extent(case)
        b, f = _conv_work(n, 3, 96, 7, ho, wo, case["h"], case["w"])
        b += 4 * n * 96 * ((ho - 3) // 2 + 1) * ((wo - 3) // 2 + 1)      # both maps are results
    else:
        hw = case["h"] * case["w"]
        b = 4 * (n * case["cin"] * hw + case["cout"] * (case["cin"] + 1) + n * case["cout"])
        f = 2.0 * n * hw * case["cin"] * case["cout"]
    return {"bytes": float(b), "flops": float(f)}


def _stem_extent(case):
    return tuple((case[d] + 2 * case["pad"] - 7) // 2 + 1 for d in ("h", "w"))


# ----------------------------------------------------------------------------------------------------- inputs and state
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _kernels(g, cout, cin, k):
    """He-normal kernels and small biases, which keep activations of order one through a network."""
    w = torch.randn((cout, cin, k, k), generator=g, device="cuda") * math.sqrt(2.0 / (cin * k * k))
    return w, torch.rand(cout, generator=g, device="cuda") * 0.2 - 0.1


def _activations(g, shape):
    """What a layer inside the network reads: the results of a ReLU."""
    return torch.randn(shape, generator=g, device="cuda").clamp_(min=0)


def _net_params(g):
    params = list(_kernels(g, 96, 3, 7))
    for cin, csq, ce, _ in FIRES:
        params += [*_kernels(g, csq, cin, 1), *_kernels(g, ce, csq, 1), *_kernels(g, ce, csq, 3)]
    return params + list(_kernels(g, 1000, 512, 1))


def _inputs(case, seed):
    """The tensors of a case, from the seed alone (exact() makes the same ones)."""
    g, n, kind = _gen(seed), case["n"], case["kind"]
    if kind == "net":
        return [torch.rand((n, 3, 224, 224), generator=g, device="cuda")] + _net_params(g)
    if kind in ("fire", "fire_blocked"):
        cin, csq, ce = case["cin"], case["csq"], case["ce"]
        t = [_activations(g, (n, cin, case["h"], case["w"])), *_kernels(g, csq, cin, 1), *_kernels(g, ce, csq, 1), *_kernels(g, ce, csq, 3)]
        # reduced precision: map and kernels are bfloat16 values, biases stay fp32
        return t if kind == "fire" else [x.bfloat16() if x.dim() == 4 else x for x in t]
    if kind == "conv":
        t = [_activations(g, (n, case["cin"], case["h"], case["w"])), *_kernels(g, case["cout"], case["cin"], case["k"])]
        return t if case["dtype"] == "f32" else [t[0].bfloat16(), t[1].bfloat16(), t[2]]
    if kind == "stem":
        return [torch.rand((n, 3, case["h"], case["w"]), generator=g, device="cuda"), *_kernels(g, 96, 3, 7)]
    return [_activations(g, (n, case["cin"], case["h"], case["w"])), *_kernels(g, case["cout"], case["cin"], 1)]


def _scratch(nbytes):
    return torch.empty(max(int(nbytes), 256), device="cuda", dtype=torch.uint8)


def _block(x):
    """NCHW -> [N][C/8][H][W][8]."""
    n, c, h, w = x.shape
    return x.view(n, c // 8, 8, h, w).permute(0, 1, 3, 4, 2).contiguous()


def prepare(case, seed):
    t, n, kind = _inputs(case, seed), case["n"], case["kind"]
    s = {"case": case}
    if kind == "net":
        s["x"], s["params"] = t[0], t[1:]
        if case["dtype"] == "f32":
            s["packed"] = sq.sq_pack_weights(s["params"], sq.SQ_F32)
            s["ws"] = _scratch(sq.sq_squeezenet_workspace_bytes(n))
        else:
            s["packed"] = sq.sq_squeezenet_bf16_pack_params(s["params"])
            s["ws"] = _scratch(sq.sq_squeezenet_bf16_workspace_bytes(n))
        s["probs"] = torch.empty((n, 1000), device="cuda")
    elif kind == "fire":
        s["args"] = t
        if case["packed"]:
            s["packed"] = sq.sq_fire_pack_weights(t[5])
        s["ws"] = _scratch(sq.sq_fire_workspace_bytes(n, case["h"], case["w"], case["csq"], case["ce"]))
        s["out"] = torch.empty((n, 2 * case["ce"], case["h"], case["w"]), device="cuda")
    elif kind == "fire_blocked":
        s["x"] = _block(t[0])
        s["packed"] = [sq.sq_blocked_pack_kernels(t[i]) for i in (1, 3, 5)]
        s["bias"] = [t[2], t[4], t[6]]
        s["ws"] = _scratch(sq.sq_blocked_map_bytes(n, case["csq"], case["h"], case["w"]))
    elif kind == "conv":
        s["args"] = t
        k, pad = case["k"], (case["k"] - 1) // 2
        need = sq.sq_conv2d_workspace_bytes(case["cin"], case["cout"], k, 1, pad)
        if case["dtype"] == "bf16":
            need = max(need, sq.sq_conv2d_bf16_workspace_bytes(n, case["cin"], case["h"], case["w"], case["cout"], k, 1, pad))
        s["ws"] = _scratch(need)
        s["out"] = torch.empty((n, case["cout"], case["h"], case["w"]), device="cuda")
    elif kind == "stem":
        s["args"] = t
    else:
        s["args"] = t
        s["ws"] = _scratch(sq.lib.sq_classifier_workspace_bytes(n, case["cin"], case["h"], case["w"], case["cout"]))
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "net":
        call = sq.sq_squeezenet_forward_packed if case["dtype"] == "f32" else sq.sq_squeezenet_forward_bf16
        return call(s["x"], s["params"], s["packed"], workspace=s["ws"], probs=s["probs"])
    if kind == "fire":
        if case["packed"]:
            return sq.sq_fire_forward_packed(*s["args"], s["packed"], workspace=s["ws"], out=s["out"])
        return sq.sq_fire_forward(*s["args"], workspace=s["ws"], out=s["out"])
    if kind == "fire_blocked":
        p, b = s["packed"], s["bias"]
        return sq.sq_blocked_fire_forward(s["x"], case["cin"], p[0], b[0], p[1], b[1], p[2], b[2], case["csq"], case["ce"], case["ce"],
                                          workspace=s["ws"])
    if kind == "conv":
        x, w, b = s["args"]
        return sq.sq_conv2d_forward_ws(x, w, b, 1, (case["k"] - 1) // 2, True, out=s["out"], workspace=s["ws"])
    if kind == "stem":
        full = sq.sq_conv2d_forward(*s["args"], stride=2, pad=case["pad"], relu=True)
        return full, sq.sq_maxpool(full, 3, 2)
    probs, means = sq.sq_classifier_forward(*s["args"], want_means=True, workspace=s["ws"])
    return probs, means


# ------------------------------------------------------------------------------------------------------ the same in 64 bits
def _conv64(x, w, b, stride=1, pad=0):
    """relu(conv) by one matrix product per kernel tap."""
    n, cin, h, wd = x.shape
    cout, _, k, _ = w.shape
    ho, wo = (h + 2 * pad - k) // stride + 1, (wd + 2 * pad - k) // stride + 1
    if pad:
        x = torch.nn.functional.pad(x, (pad, pad, pad, pad))
    out = b.double().view(1, cout, 1).expand(n, cout, ho * wo).clone()
    w = w.double()
    for i in range(k):
        for j in range(k):
            tap = x[:, :, i:i + (ho - 1) * stride + 1:stride, j:j + (wo - 1) * stride + 1:stride].reshape(n, cin, ho * wo)
            out += torch.matmul(w[:, :, i, j].contiguous(), tap)
    return out.clamp_(min=0).view(n, cout, ho, wo)


def _pool64(x):
    return torch.nn.functional.max_pool2d(x, 3, 2)


def _fire64(x, w_sq, b_sq, w_e1, b_e1, w_e3, b_e3):
    s = _conv64(x, w_sq, b_sq)
    return torch.cat([_conv64(s, w_e1, b_e1), _conv64(s, w_e3, b_e3, 1, 1)], 1)


def exact(case, seed):
    t, kind = _inputs(case, seed), case["kind"]
    x, p = t[0].double(), t[1:]
    if kind == "net":
        x = _pool64(_conv64(x, p[0], p[1], 2, 2))
        for f in range(8):
            x = _fire64(x, *p[2 + 6 * f:8 + 6 * f])
            if f in POOL_BEHIND:
                x = _pool64(x)
        return torch.softmax(_conv64(x, p[50], p[51]).mean((2, 3)), 1)
    if kind == "fire":
        return _fire64(x, *p)
    if kind == "fire_blocked":
        return _block(_fire64(x, *p))
    if kind == "conv":
        return _conv64(x, p[0], p[1], 1, (case["k"] - 1) // 2)
    if kind == "stem":
        full = _conv64(x, p[0], p[1], 2, case["pad"])
        return full, _pool64(full)
    means = _conv64(x, p[0], p[1]).mean((2, 3))
    return torch.softmax(means, 1), means


def tolerance(case):
    """About four times the error against exact() that the first measured state of the library showed over the listed and drawn cases."""
    kind = case["kind"]
    if kind == "net":
        return {"rel": 1.3e-2} if case["dtype"] == "bf16" else {"rel": 1.5e-6}
    if kind == "fire_blocked":
        return {"rel": 9e-3}      # squeeze map and results are rounded to bfloat16 (2^-9 each)
    return {"rel": 2.5e-6}

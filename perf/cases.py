"""Performance cases of the integrated fixed-point quantized conv library.

A case is one call that a program using this library makes once its network
is converted: a whole layer chain (DeviceStack.run), a single quantized conv
layer (ifq_conv_forward), a max-pool on codes (ifq_maxpool_codes) or a code
layout conversion (ifq_convert_codes). Conversion (packing weights, folding
thresholds) is done once by prepare(), as such a program does.

Network shapes are the repository's own: the AlexNet body, the VGG-16 convs,
the ResNet-18 body and the Tiny-YOLOv2-shaped detector. All outputs are codes
or int32 sums, which have one correct value each.
"""
import math
from types import SimpleNamespace as NS

import numpy as np
import torch

import paper_1911_08076_amd as P

LAYOUT = {"i8": P.IFQ_LAYOUT_I8_NHWC, "u2": P.IFQ_LAYOUT_U2_NHWC_PACKED,
          "b64": P.IFQ_LAYOUT_U2_BLOCK64, "i32": P.IFQ_LAYOUT_I32_NHWC}


# -- networks ----------------------------------------------------------------
def _conv(name, src, dst, h, w, cin, cout, k, s, p, inb, outb, join=None):
    return NS(name=name, src=src, dst=dst, h=h, w=w, cin=cin, cout=cout, k=k, stride=s,
              pad=p, in_bits=inb, out_bits=outb, join=join)


def _pool(name, src, dst, h, w, c, k, s, mode, bits):
    return NS(name=name, src=src, dst=dst, h=h, w=w, c=c, k=k, stride=s, mode=mode, bits=bits)


def _chain(rows, b, in_bits):
    """Layers of a plain chain from rows ("c", hw, cin, cout, k, pad) and
    ("p", hw, c, k, stride, mode); a head row is ("h", hw, cin, cout)."""
    out, src = [], "x"
    for i, r in enumerate(rows):
        dst = "y" if i == len(rows) - 1 else "t%d" % i
        name = "%s%d" % (r[0], i)
        if r[0] == "p":
            out.append(_pool(name, src, dst, r[1], r[1], r[2], r[3], r[4], r[5], b))
        elif r[0] == "h":
            out.append(_conv(name, src, dst, r[1], r[1], r[2], r[3], 1, 1, 0, b, 0))
        else:
            out.append(_conv(name, src, dst, r[1], r[1], r[2], r[3], r[4], 1, r[5],
                             in_bits if i == 0 else b, b))
        src = dst
    return out


def _alexnet(b):
    return _chain([("c", 27, 96, 256, 5, 2), ("p", 27, 256, 3, 2, "valid"),
                   ("c", 13, 256, 384, 3, 1), ("c", 13, 384, 384, 3, 1),
                   ("c", 13, 384, 256, 3, 1), ("p", 13, 256, 3, 2, "valid")], b, b)


def _vgg16(b):
    rows, cin = [("c", 224, 64, 64, 3, 1), ("p", 224, 64, 2, 2, "valid")], 64
    for hw, cout, n in ((112, 128, 2), (56, 256, 3), (28, 512, 3), (14, 512, 3)):
        for _ in range(n):
            rows.append(("c", hw, cin, cout, 3, 1))
            cin = cout
        rows.append(("p", hw, cout, 2, 2, "valid"))
    return _chain(rows, b, b)


def _yolo(b):
    rows, cin, hw = [], 3, 416
    for cout in (16, 32, 64, 128, 256):
        rows += [("c", hw, cin, cout, 3, 1), ("p", hw, cout, 2, 2, "valid")]
        cin, hw = cout, hw // 2
    rows += [("c", 13, 256, 512, 3, 1), ("p", 13, 512, 2, 1, "same"),
             ("c", 13, 512, 512, 3, 1), ("c", 13, 512, 512, 3, 1), ("h", 13, 512, 30)]
    return _chain(rows, b, 8)


def _resnet18(b):
    out, cur, cin, hw, t = [], "x", 64, 56, 0
    for si, cout in enumerate((64, 128, 256, 512)):
        for bi in range(2):
            pre, down = "l%d.%d" % (si + 1, bi), bi == 0 and si > 0
            s, join = (2 if down else 1), ("identity", cur)
            mid, dst = "t%d" % t, "y" if (si, bi) == (3, 1) else "t%d" % (t + 2)
            out.append(_conv(pre + ".conv1", cur, mid, hw, hw, cin, cout, 3, s, 1, b, b))
            if down:
                out.append(_conv(pre + ".down", cur, "t%d" % (t + 1), hw, hw, cin, cout, 1, 2,
                                 0, b, 0))
                join = ("conv", "t%d" % (t + 1), pre + ".down")
            hw //= s
            out.append(_conv(pre + ".conv2", mid, dst, hw, hw, cout, cout, 3, 1, 1, b, b, join))
            cur, cin, t = dst, cout, t + 3
    return out


NETS = {"alexnet": _alexnet, "vgg16": _vgg16, "yolo": _yolo, "resnet18": _resnet18}


def _layers(c):
    if c["kind"] == "stack":
        return NETS[c["net"]](c["bits"])
    if c["kind"] == "conv":
        return [_conv("conv", "x", "y", c["h"], c["w"], c["cin"], c["cout"], c["k"], c["stride"],
                      c["pad"], c["in_bits"], c["out_bits"])]
    return [_pool("pool", "x", "y", c["h"], c["w"], c["c"], c["k"], c["stride"], c["mode"],
                  c["bits"])]


def _out_hw(L):
    if hasattr(L, "cin") or L.mode == "valid":
        p = L.pad if hasattr(L, "cin") else 0
        return ((v + 2 * p - L.k) // L.stride + 1 for v in (L.h, L.w))
    return (-(-v // L.stride) for v in (L.h, L.w))


# -- inputs ------------------------------------------------------------------
def _step(bits):
    """Step between code levels: 8-bit pixels, or k-bit codes over the range
    that the 2-bit network's step 0.5 covers."""
    return 1.0 / 255.0 if bits == 8 else 2.0 ** (1 - bits)


def _params(L, seed, i):
    """+-1 weights and the float parameters of a conv, its batch norm scaled
    to the spread of the sums so that all code levels occur."""
    r = np.random.default_rng([seed, i])
    w = r.integers(0, 2, (L.cout, L.cin, L.k, L.k), dtype=np.int8) * 2 - 1
    levels = np.arange(1 << L.in_bits, dtype=np.float64)
    alpha = r.uniform(0.01, 0.1, L.cout)
    spread = alpha * _step(L.in_bits) * math.sqrt(L.k * L.k * L.cin * np.mean(levels ** 2))
    gamma = r.uniform(0.5, 1.5, L.cout) * np.where(r.random(L.cout) < 0.1, -1.0, 1.0)
    ob = L.out_bits or 2
    return dict(w=w.astype(np.int8), alpha=alpha, bias=np.zeros(L.cout),
                mean=r.normal(0.0, 0.5, L.cout) * spread,
                var=r.uniform(0.5, 2.0, L.cout) * spread ** 2, gamma=gamma,
                bn_beta=r.normal(0.0, 1.0, L.cout), eps=1e-5, beta_in=_step(L.in_bits),
                q_thr=(np.arange(1, 1 << ob) - 0.5) * _step(ob))


def _codes(shape, bits, layout, seed):
    """Uniform random codes on the GPU, as the flat byte tensor of a layout."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    n = math.prod(shape)
    if layout != "i8":  # every byte holds four 2-bit codes
        return torch.randint(0, 256, (n // 4,), generator=g, device="cuda", dtype=torch.uint8)
    return torch.randint(0, 1 << bits, (n,), generator=g, device="cuda", dtype=torch.uint8)


def _stack_layout(c, bits, ch):
    if bits == 2 and c["layout"] == "b64" and ch % 64 == 0:
        return "b64"
    return "u2" if bits == 2 and c["layout"] != "i8" and ch % 16 == 0 else "i8"


def _x(c, seed):
    """(shape, bits, layout, device codes) of a case's input."""
    if c["kind"] == "convert":
        shape, bits, lay = (c["n"], c["h"], c["w"], c["c"]), 2, c["src"]
    else:
        L = _layers(c)[0]
        bits, ch = (L.in_bits, L.cin) if hasattr(L, "cin") else (L.bits, L.c)
        shape = (c["n"], L.h, L.w, ch)
        lay = _stack_layout(c, bits, ch) if c["kind"] == "stack" else c["layout"]
    return shape, bits, lay, _codes(shape, bits, lay, seed)


def _bytes(n, h, w, ch, layout):
    return P.ifq_tensor_bytes(n, h, w, ch, LAYOUT[layout])


def prepare(case, seed):
    c = case
    shape, _, lay, x = _x(c, seed)
    if c["kind"] == "convert":
        return NS(kind="convert", dims=shape, src=LAYOUT[lay], dst=LAYOUT[c["dst"]], x=x,
                  y=torch.empty(_bytes(*shape, c["dst"]), dtype=torch.uint8, device="cuda"))
    layers = _layers(c)
    if c["kind"] == "pool":
        L = layers[0]
        ho, wo = _out_hw(L)
        d = P.pool_desc(c["n"], L.h, L.w, L.c, L.k, L.stride,
                        P.IFQ_POOL_VALID if L.mode == "valid" else P.IFQ_POOL_SAME, L.bits,
                        LAYOUT[lay])
        return NS(kind="pool", desc=d, x=x,
                  y=torch.empty(_bytes(c["n"], ho, wo, L.c, lay), dtype=torch.uint8,
                                device="cuda"))
    params = [_params(L, seed, i) if hasattr(L, "cin") else None for i, L in enumerate(layers)]
    if c["kind"] == "stack":
        dev = P.DeviceStack(layers, params, c["n"], code_layout=c["layout"],
                            fuse_down=c["fuse"], fuse_pool=c["fuse"], fp4=c["fp4"])
        return NS(kind="stack", dev=dev, x=x, y=dev.alloc_output())
    L, p = layers[0], params[0]
    ob = c["out_layout"]
    d = P.conv_desc(c["n"], L.h, L.w, L.cin, L.cout, L.k, L.stride, L.pad, L.in_bits, L.out_bits,
                    LAYOUT[lay], LAYOUT[ob])
    ho, wo = _out_hw(L)
    thr = join = keep = None
    if c["join"]:  # residual: the shortcut's codes have the output's shape and layout
        table = P.ifq_fold_join_table(p, _step(2), L.in_bits, L.k * L.k * L.cin, L.out_bits,
                                      p["q_thr"])
        keep = (torch.from_numpy(table).cuda(), _codes((c["n"], ho, wo, L.cout), 2, ob, seed + 1))
        join = P.make_join(P.IFQ_JOIN_IDENTITY, LAYOUT[ob], keep[1], None, p["q_thr"],
                           table=keep[0])
    elif L.out_bits:
        thr = torch.from_numpy(P.ifq_fold_thresholds(
            L.cout, L.in_bits, L.out_bits, L.k * L.k * L.cin, p["alpha"], p["beta_in"],
            p["q_thr"], bias=p["bias"], mean=p["mean"], var=p["var"], gamma=p["gamma"],
            bn_beta=p["bn_beta"], eps=p["eps"])).cuda()
    need = P.ifq_conv_workspace_bytes(d)
    return NS(kind="conv", desc=d, x=x, w=torch.from_numpy(P.ifq_pack_weights(d, p["w"])).cuda(),
              thr=thr, join=join, keep=keep,
              ws=torch.zeros(need, dtype=torch.uint8, device="cuda") if need else None,
              y=torch.empty(_bytes(c["n"], ho, wo, L.cout, ob), dtype=torch.uint8, device="cuda"))


def run(state):
    s = state
    if s.kind == "stack":
        s.dev.run(s.x, s.y)
    elif s.kind == "conv":
        P.ifq_conv_forward(s.desc, s.x, s.w, s.thr, s.y, join=s.join, ws=s.ws)
    elif s.kind == "pool":
        P.ifq_maxpool_codes(s.desc, s.x, s.y)
    else:
        P.ifq_convert_codes(*s.dims, s.src, s.dst, s.x, s.y)
    return s.y


# -- work, tolerance, reference ------------------------------------------------
def work(case):
    """Input, weights at one bit each, one threshold record per channel and the
    output; two operations per product, padding included."""
    c = case
    if c["kind"] == "convert":
        d = (c["n"], c["h"], c["w"], c["c"])
        return {"bytes": _bytes(*d, c["src"]) + _bytes(*d, c["dst"]), "flops": 0}
    layers = _layers(c)
    L0, L1 = layers[0], layers[-1]
    conv0, conv1 = hasattr(L0, "cin"), hasattr(L1, "cin")
    ib, ic = (L0.in_bits, L0.cin) if conv0 else (L0.bits, L0.c)
    ob, oc = (L1.out_bits, L1.cout) if conv1 else (L1.bits, L1.c)
    if c["kind"] == "stack":
        il, ol = _stack_layout(c, ib, ic), "i32" if ob == 0 else _stack_layout(c, ob, oc)
    else:
        il, ol = c["layout"], c.get("out_layout", c["layout"])
    ho, wo = _out_hw(L1)
    b, f = _bytes(c["n"], L0.h, L0.w, ic, il) + _bytes(c["n"], ho, wo, oc, ol), 0
    if c.get("join"):
        b += _bytes(c["n"], ho, wo, oc, ol)
    for L in layers:
        if hasattr(L, "cin"):
            ho, wo = _out_hw(L)
            k = L.k * L.k * L.cin
            b += L.cout * k // 8 + (L.cout * 4 << L.out_bits if L.out_bits else 0)
            f += 2 * c["n"] * ho * wo * L.cout * k
    return {"bytes": b, "flops": f}


def tolerance(case):
    return "exact"  # codes and integer sums


def _unpack(x, shape, layout):
    """Device bytes of a layout -> NHWC float64 codes."""
    n, h, w, ch = shape
    if layout == "i8":
        return x.view(shape).double()
    sh = torch.tensor([0, 2, 4, 6], device=x.device, dtype=torch.uint8)
    v = (x.view(-1, 1) >> sh) & 3
    if layout == "b64":
        return v.view(n, ch // 64, h, w, 64).permute(0, 2, 3, 1, 4).reshape(shape).double()
    return v.view(shape).double()


def _pack(v, layout):
    """NHWC float64 values -> the flat byte tensor of a layout."""
    n, h, w, ch = v.shape
    if layout == "i32":
        return v.to(torch.int32).contiguous().view(-1).view(torch.uint8)
    u = v.to(torch.uint8)
    if layout == "b64":
        u = u.view(n, h, w, ch // 64, 64).permute(0, 3, 1, 2, 4)
    if layout != "i8":
        u = u.reshape(-1, 4)
        u = u[:, 0] | (u[:, 1] << 2) | (u[:, 2] << 4) | (u[:, 3] << 6)
    return u.reshape(-1).contiguous()


def _bn(a, p):
    t = {k: torch.from_numpy(np.asarray(p[k])).cuda() for k in ("alpha", "mean", "var", "gamma",
                                                                 "bn_beta")}
    return (t["gamma"] * (t["alpha"] * p["beta_in"] * a - t["mean"]) /
            torch.sqrt(t["var"] + p["eps"]) + t["bn_beta"])


def _sums(x, L, w):
    """Integer sums of a conv, in 64 bits, one filter tap at a time."""
    ho, wo = _out_hw(L)
    xp = torch.nn.functional.pad(x, (0, 0, L.pad, L.pad, L.pad, L.pad))
    wt = torch.from_numpy(w).cuda().double()
    a = 0
    for r in range(L.k):
        for s in range(L.k):
            v = xp[:, r:r + (ho - 1) * L.stride + 1:L.stride, s:s + (wo - 1) * L.stride + 1:L.stride]
            a = a + v.reshape(-1, L.cin) @ wt[:, :, r, s].t().contiguous()
    return a.view(x.shape[0], ho, wo, L.cout)


def exact(case, seed):
    """The float chain of each layer (conv, batch norm, join, quantizer) and
    the pools, in 64 bits."""
    c = case
    shape, bits, lay, x = _x(c, seed)
    v = _unpack(x, shape, lay)
    if c["kind"] == "convert":
        return _pack(v, c["dst"])
    layers, t, by = _layers(c), {"x": v}, {}
    for i, L in enumerate(layers):
        v = t[L.src]
        if not hasattr(L, "cin"):
            ho, wo = _out_hw(L)
            q = torch.nn.functional.pad(v, (0, 0, 0, max(0, (wo - 1) * L.stride + L.k - L.w), 0,
                                            max(0, (ho - 1) * L.stride + L.k - L.h)))
            t[L.dst] = torch.nn.functional.max_pool2d(q.permute(0, 3, 1, 2), L.k,
                                                      L.stride).permute(0, 2, 3, 1).contiguous()
            continue
        p = _params(L, seed, i)
        by[L.name] = p
        a = _sums(v, L, p["w"])
        if L.out_bits == 0:
            t[L.dst] = a
            continue
        z = _bn(a, p)
        if L.join and L.join[0] == "identity":
            z = z + p["beta_in"] * t[L.join[1]]
        elif L.join:
            z = z + _bn(t[L.join[1]], by[L.join[2]])
        elif c.get("join"):
            sc = _codes((c["n"], *z.shape[1:]), 2, c["out_layout"], seed + 1)
            z = z + _step(2) * _unpack(sc, tuple(z.shape), c["out_layout"])
        t[L.dst] = sum((z > q).double() for q in p["q_thr"])
    L = layers[-1]
    if c["kind"] == "stack":
        ob, ch = (L.out_bits, L.cout) if hasattr(L, "cin") else (L.bits, L.c)
        ol = "i32" if ob == 0 else _stack_layout(c, ob, ch)
    else:
        ol = c.get("out_layout", c["layout"])
    return _pack(t["y"], ol)


# -- cases -------------------------------------------------------------------
def _stack_case(net, n, layout="b64", bits=2, fuse=True, fp4=False):
    return dict(kind="stack", net=net, n=n, layout=layout, bits=bits, fuse=fuse, fp4=fp4)


def _conv_case(n, h, w, cin, cout, k, stride, pad, in_bits=2, out_bits=2, layout="b64",
               out_layout=None, join=False):
    return dict(kind="conv", n=n, h=h, w=w, cin=cin, cout=cout, k=k, stride=stride, pad=pad,
                in_bits=in_bits, out_bits=out_bits, layout=layout,
                out_layout=out_layout or ("i32" if out_bits == 0 else layout), join=join)


def listed():
    return [
        # one image through one 3x3 layer: the smallest call, launch-bound
        dict(name="conv3x3_b1", **_conv_case(1, 28, 28, 64, 64, 3, 1, 1)),
        # a classifier body at serving batch with every fusion: the benchmark's stack
        dict(name="resnet18_b64", **_stack_case("resnet18", 64)),
        # the same network as DeviceStack takes it by default: one byte per
        # code, downsamples and pools as layers of their own, a small batch
        dict(name="resnet18_bytes_b8", **_stack_case("resnet18", 8, "i8", fuse=False)),
        # the largest call: 224x224 maps, 488 G operations
        dict(name="vgg16_b16", **_stack_case("vgg16", 16)),
        # detection on raw 8-bit pixels: narrow first layers, int32 head
        dict(name="yolo_b8", **_stack_case("yolo", 8)),
        # the paper's classifier at 2 bits: a 5x5 layer on 96 channels, overlapping pools
        dict(name="alexnet_b32", **_stack_case("alexnet", 32)),
        # the same network at 4 bits, the widest codes the paper evaluates
        dict(name="alexnet_4bit_b32", **_stack_case("alexnet", 32, "i8", 4, False)),
        # its first fully connected layer, as a 6x6 conv over the last pool
        dict(name="fc6_b32", **_conv_case(32, 6, 6, 256, 4096, 6, 1, 0, layout="u2")),
        # a strided layer at an odd size on NHWC packed codes
        dict(name="conv3x3_s2_odd_u2", **_conv_case(6, 75, 57, 128, 160, 3, 2, 1, layout="u2")),
        # the 3x3 layers on the fp4 matrix instructions, at a small serving batch
        dict(name="resnet18_fp4_b16", **_stack_case("resnet18", 16, fp4=True)),
        # the classifier's overlapping pool on its first layer's codes
        dict(name="pool3x3_s2_b64", kind="pool", n=64, h=55, w=55, c=96, k=3, stride=2,
             mode="valid", bits=2, layout="u2"),
        # a batch of byte codes laid out for the packed network input
        dict(name="convert_i8_b64", kind="convert", n=64, h=56, w=56, c=64, src="i8", dst="b64"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["conv"] * 5 + ["stack"] * 3 + ["pool", "convert"])
    if kind == "stack":
        net = rng.choice(list(NETS))
        how = rng.choice(["b64", "b64", "b64 fp4", "u2", "i8", "bits"])
        top = {"alexnet": 48, "vgg16": 12, "yolo": 12, "resnet18": 64}[net]
        if how in ("i8", "bits", "u2"):
            top = {"alexnet": 32, "vgg16": 2, "yolo": 8, "resnet18": 12}[net]
        if how == "bits":
            # residual shortcuts are 2-bit: k-bit codes run in the plain chains
            net = "alexnet" if net == "resnet18" else net
            return _stack_case(net, _log(rng, 1, min(top, 12)), "i8", rng.choice([3, 4]), False)
        return _stack_case(net, _log(rng, 1, top), how[:3].strip(), 2,
                           how[:3] == "b64" and rng.random() < 0.8, how.endswith("fp4"))
    if kind == "conv":
        while True:
            lay = rng.choice(["b64", "b64", "u2", "i8"])
            k = rng.choice([3, 3, 3, 3, 1, 5])
            first = lay == "i8" and rng.random() < 0.25
            cin = 3 if first else (64 * _log(rng, 1, 8) if lay == "b64" else
                                   16 * _log(rng, 1, 32))
            cout = (64 * _log(rng, 1, 8) if lay == "b64" else 16 * _log(rng, 1, 32))
            ib = 8 if first else rng.choice([2, 3, 4]) if lay == "i8" else 2
            ob = ib if lay == "i8" and not first else 2
            if k == 1 and rng.random() < 0.4:
                ob = 0
            hw = _log(rng, 7, 224)
            c = _conv_case(_log(rng, 1, 64), hw, max(7, hw - rng.randrange(0, 1 + hw // 4)), cin,
                           cout, k, rng.choice([1, 1, 1, 2]), k // 2, ib, ob, lay,
                           join=k == 3 and ib == 2 and ob == 2 and rng.random() < 0.25)
            w = work(c)
            if w["flops"] <= (4e10 if lay == "b64" else 1e10) and w["bytes"] <= 6e7:
                return c
    while True:
        hw, lay = _log(rng, 7, 224), rng.choice(["b64", "u2", "i8"])
        c = dict(n=_log(rng, 1, 64), h=hw, w=max(7, hw - rng.randrange(0, 1 + hw // 4)),
                 c=(64 * _log(rng, 1, 8) if lay == "b64" else 16 * _log(rng, 1, 32)))
        if kind == "pool":
            k, s, mode = rng.choice([(2, 2, "valid"), (3, 2, "valid"), (2, 1, "same")])
            c.update(kind="pool", k=k, stride=s, mode=mode, layout=lay,
                     bits=rng.choice([2, 4]) if lay == "i8" else 2)
        else:
            to = [v for v in ("i8", "u2", "b64") if v != lay and (v != "b64" or c["c"] % 64 == 0)]
            c.update(kind="convert", src=lay, dst=rng.choice(to))
        if work(c)["bytes"] <= 6e7:
            return c

"""What a training job has this library do, as cases that can be timed and compared.

A case names a network shape (`net` and its sizes), what is asked for every layer of it (`op`) and the element type of
activations and output gradients (`dtype`).  The shapes are the layer geometries of the networks the paper trains
(section 6.1) at the sizes of the benchmark's workloads, and `draw` varies every size of them: channel counts and map
sizes that fill no tile, batches from a few examples up, fewer blocks.

op:
  layer         one layer through the per-layer calls: factors with running average, damped inverses, preconditioning
  update        a whole second-order update, one batched call for each of these three stages
  update_pi     the same with the damping split of Eq. 12
  eigen         the same with eigen-decompositions and the preconditioner of Eq. 13 (the paper's default)
  factors       the factor update alone: what most iterations that touch the factors do when inverses are refreshed
                less often (section 6.5 refreshes factors every 50 iterations and inverses every 500)
  precondition  preconditioning alone: what every iteration does

Buffers that live as long as the model (running factors, inverses, preconditioned gradients, workspace) and the layer
descriptions are converted to C arrays once, as the binding offers for training loops; what autograd hands over anew
in every iteration (activations, output gradients, layer gradients) goes in as lists of tensors.
"""
from __future__ import annotations

import math
from dataclasses import dataclass

import torch

import paper_2206_15143_amd as kf

DEV = "cuda:0"
DECAY = 0.95


@dataclass(frozen=True)
class Layer:
    conv: bool
    c_in: int
    c_out: int
    rows: int                # linear: samples or tokens; conv: images
    h: int = 1
    w: int = 1
    kh: int = 1
    kw: int = 1
    stride: int = 1
    ph: int = 0
    pw: int = 0

    @property
    def h_out(self):
        return (self.h + 2 * self.ph - self.kh) // self.stride + 1

    @property
    def w_out(self):
        return (self.w + 2 * self.pw - self.kw) // self.stride + 1

    @property
    def d_A(self):
        return self.c_in * self.kh * self.kw + 1

    @property
    def d_G(self):
        return self.c_out

    @property
    def R(self):
        return self.rows * self.h_out * self.w_out if self.conv else self.rows

    def desc(self, bf16):
        dt = kf.KFAC_BF16 if bf16 else kf.KFAC_F32
        if self.conv:
            return kf.LayerDesc.conv2d(self.c_in, self.c_out, self.kh, self.stride, self.ph, True, dt, kw=self.kw,
                                       pad_w=self.pw)
        return kf.LayerDesc.linear(self.c_in, self.c_out, True, dt)


def _conv(n, cin, cout, k, h, stride=1):
    p = (k - 1) // 2
    return Layer(True, cin, cout, n, h, h, k, k, stride, p, p)


def _fc(rows, cin, cout):
    return Layer(False, cin, cout, rows)


# ---- network shapes -------------------------------------------------------------------------------------------


def _single_fc(c):
    return [_fc(c["batch"], c["d_in"], c["d_out"])]


def _single_conv(c):
    return [_conv(c["batch"], c["d_in"], c["d_out"], c["k"], c["image"])]


def _resnet_cifar(c):
    """A stem and three stages of equal 3x3 convolutions on maps halved twice, a classifier."""
    n, w, h = c["batch"], c["width"], c["image"]
    layers = [_conv(n, 3, w, 3, h)]
    for s in range(3):
        layers += [_conv(n, w << s, w << s, 3, h >> s)] * c["depth"]
    return layers + [_fc(n, 4 * w, 10)]


def _bottleneck(c):
    """ResNet-50-shaped: 7x7 stem, four stages of 1x1 / 3x3 / 1x1 blocks with projection shortcuts, a classifier."""
    n, w, size = c["batch"], c["width"], c["image"]
    layers = [_conv(n, 3, w, 7, size, 2)]
    h, cin = (size + 3) // 4, w
    for s, reps in enumerate(int(x) for x in c["blocks"].split(",")):
        mid = w << s
        for b in range(reps):
            st = 2 if s and not b else 1
            ho = (h - 1) // st + 1
            layers += [_conv(n, cin, mid, 1, h), _conv(n, mid, mid, 3, h, st), _conv(n, mid, 4 * mid, 1, ho)]
            if not b:
                layers.append(_conv(n, cin, 4 * mid, 1, h, st))
            cin, h = 4 * mid, ho
    return layers + [_fc(n, cin, c["classes"])]


def _encoder(c):
    """Transformer encoder blocks: four projections and the two feed-forward layers each."""
    d, f, rows = c["hidden"], c["ffn"], c["rows"]
    return ([_fc(rows, d, d)] * 4 + [_fc(rows, d, f), _fc(rows, f, d)]) * c["blocks"]


def _dense(c):
    """DenseNet-201-shaped: a dense layer sees all channels so far; widths grow in steps, few are powers of two."""
    n, g, size = c["batch"], c["growth"], c["image"]
    ch, h = 2 * g, (size + 3) // 4
    layers = [_conv(n, 3, ch, 7, size, 2)]
    blocks = [int(x) for x in c["blocks"].split(",")]
    for s, reps in enumerate(blocks):
        for j in range(reps):
            layers += [_conv(n, ch + g * j, 4 * g, 1, h), _conv(n, 4 * g, g, 3, h)]
        ch += g * reps
        if s + 1 < len(blocks):
            layers.append(_conv(n, ch, ch // 2, 1, h))
            ch //= 2
            h //= 2
    return layers + [_fc(n, ch, c["classes"])]


def _vgg(c):
    """VGG-16-shaped: thirteen 3x3 convolutions in five groups on halving maps, three fully connected layers."""
    n, w, h, cin, layers = c["batch"], c["width"], c["image"], 3, []
    for mul, reps in ((1, 2), (2, 2), (4, 3), (8, 3), (8, 3)):
        for _ in range(reps):
            layers.append(_conv(n, cin, w * mul, 3, h))
            cin = w * mul
        h //= 2
    return layers + [_fc(n, cin, cin), _fc(n, cin, cin), _fc(n, cin, 10)]


def _factorised(c):
    """Inception-style 1x7 / 7x1 and 1x3 / 3x1 convolutions padded along the long side, one of each stage on a map
    that is not square, one layer unpadded."""
    n, u, m, s = c["batch"], c["unit"], c["map"], c["map2"]

    def ns(cin, cout, kh, kw, h, w, same=True):
        return Layer(True, cin * u // 2, cout * u // 2, n, h, w, kh, kw, 1, (kh - 1) // 2 if same else 0,
                     (kw - 1) // 2 if same else 0)
    return [ns(6, 6, 1, 7, m, m), ns(6, 7, 7, 1, m, m), ns(7, 8, 1, 7, m, m + 6), ns(12, 8, 1, 3, s, s),
            ns(12, 8, 3, 1, s, s), ns(14, 16, 3, 1, s, s + 4), ns(6, 7, 1, 7, m, m, same=False)]


# net -> (layers of a case, damping, std of the output gradients, activations pass a ReLU)
NETS = {
    "fc": (_single_fc, 0.03, 0.1, False),
    "conv": (_single_conv, 0.03, 0.1, True),
    "resnet_cifar": (_resnet_cifar, 0.03, 1e-3 ** 0.5, True),
    "bottleneck": (_bottleneck, 0.001, 1e-3 ** 0.5, True),
    "encoder": (_encoder, 0.003, 1e-2, False),
    "dense": (_dense, 0.001, 1e-3 ** 0.5, True),
    "vgg": (_vgg, 0.03, 1e-3 ** 0.5, True),
    "factorised": (_factorised, 0.001, 1e-3 ** 0.5, True),
}

_RESNET110 = dict(net="resnet_cifar", width=16, depth=36, image=32, batch=128, dtype="f32")
_RESNET50 = dict(net="bottleneck", width=64, blocks="3,4,6,3", image=224, classes=1000, batch=32, dtype="f32")


def listed():
    return [
        # one small fully connected layer, call by call: nothing but latency (smallest workload of the benchmark)
        dict(name="fc_layer", op="layer", net="fc", d_in=64, d_out=32, batch=32, dtype="f32"),
        # 110 narrow layers, the whole update in three batched calls
        dict(name="resnet110_update", op="update", **_RESNET110),
        # the same layers in an ordinary iteration, between refreshes
        dict(name="resnet110_precondition", op="precondition", **_RESNET110),
        # the same layers with the paper's default variant (Eq. 13)
        dict(name="resnet110_eigen", op="eigen", **_RESNET110),
        # the benchmark's headline workload
        dict(name="resnet50_update", op="update", **_RESNET50),
        # the same layers in an ordinary iteration
        dict(name="resnet50_precondition", op="precondition", **_RESNET50),
        # mixed-precision training of the same network, twice the batch
        dict(name="resnet50_bf16_update", op="update", **dict(_RESNET50, dtype="bf16", batch=64)),
        # 24 transformer blocks in mixed precision: the largest
        dict(name="encoder_bf16_update", op="update", net="encoder", hidden=1024, ffn=4096, rows=4096, blocks=24,
             dtype="bf16"),
        # fine-tuning with a handful of sequences: fewer rows than columns, every factor rank-deficient, Eq. 12 damping
        dict(name="bert_small_batch_update_pi", op="update_pi", net="encoder", hidden=768, ffn=3072, rows=512,
             blocks=12, dtype="f32"),
        # 201 layers of 107 different shapes, hardly one of them a power of two wide
        dict(name="densenet201_update", op="update", net="dense", growth=32, blocks="6,12,48,32", image=224,
             classes=1000, batch=16, dtype="f32"),
        # a refresh of the factors alone; maps down to 2x2
        dict(name="vgg16_factors", op="factors", net="vgg", width=64, image=32, batch=128, dtype="f32"),
        # kernels and maps that are not square, odd map sizes
        dict(name="factorised_update", op="update", net="factorised", unit=64, map=17, map2=8, batch=32, dtype="f32"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _candidate(rng):
    op = rng.choice(["layer", "update", "update", "update", "update_pi", "eigen", "factors", "precondition"])
    if op == "layer":
        if rng.random() < 0.5:
            return dict(op=op, net="fc", d_in=_log(rng, 16, 2048), d_out=_log(rng, 10, 1024), batch=_log(rng, 8, 4096),
                        dtype=rng.choice(["f32", "bf16"]))
        return dict(op=op, net="conv", d_in=_log(rng, 3, 256), d_out=_log(rng, 8, 512), k=rng.choice([1, 3]),
                    image=_log(rng, 4, 64), batch=_log(rng, 4, 128), dtype=rng.choice(["f32", "bf16"]))
    if op == "eigen":
        return dict(op=op, net="resnet_cifar", width=rng.randint(8, 16), depth=rng.randint(4, 36),
                    image=rng.choice([28, 32]), batch=rng.randint(48, 128), dtype="f32")
    net = rng.choice(["resnet_cifar", "bottleneck", "encoder", "dense", "vgg", "factorised"])
    c = dict(op=op, net=net)
    if net == "resnet_cifar":
        c.update(width=rng.choice([8, 12, 16, 16, 20, 24, 32]), depth=rng.randint(3, 36), image=rng.choice([24, 28, 32]),
                 batch=_log(rng, 24, 128), dtype=rng.choice(["f32", "f32", "bf16"]))
    elif net == "bottleneck":
        c.update(width=rng.choice([24, 32, 40, 48, 64]), blocks=rng.choice(["1,1,1,1", "2,2,2,2", "3,4,6,3"]),
                 image=rng.randint(96, 224), classes=rng.randint(10, 1000), batch=rng.randint(8, 32),
                 dtype=rng.choice(["f32", "f32", "bf16"]))
    elif net == "encoder":
        d = 8 * rng.randint(24, 128)
        c.update(hidden=d, ffn=4 * d, rows=_log(rng, 200, 4096), blocks=rng.randint(1, 12),
                 dtype=rng.choice(["f32", "bf16"]))
    elif net == "dense":
        c.update(growth=rng.choice([12, 24, 32]), blocks=rng.choice(["4,8,12,8", "6,12,24,16", "6,12,48,32"]),
                 image=rng.randint(112, 224), classes=rng.randint(10, 1000), batch=rng.randint(6, 16), dtype="f32")
    elif net == "vgg":
        c.update(width=rng.choice([24, 32, 48, 56, 64]), image=rng.choice([32, 40, 48]), batch=_log(rng, 24, 128),
                 dtype=rng.choice(["f32", "f32", "bf16"]))
    else:
        c.update(unit=2 * rng.randint(8, 32), map=rng.randint(9, 23), map2=rng.randint(5, 12), batch=_log(rng, 8, 64),
                 dtype=rng.choice(["f32", "f32", "bf16"]))
    return c


def draw(rng):
    """A case of the ranges above.  None costs more than the largest listed one (which has 1e13 operations)."""
    while True:
        c = _candidate(rng)
        w = work(c)
        if w["flops"] <= 6e12 and w["bytes"] <= 1e10:
            return c


# ---- one case ---------------------------------------------------------------------------------------------------


def _layers(case):
    return NETS[case["net"]][0](case)


def _views(shapes, fill=None):
    """One zeroed buffer that holds a matrix of each shape, every matrix on a 256-byte boundary, and the matrices."""
    offs, n = [], 0
    for s in shapes:
        offs.append(n)
        n += -(-math.prod(s) // 64) * 64
    flat = torch.zeros(n, device=DEV)
    views = [flat[o:o + math.prod(s)].view(s) for o, s in zip(offs, shapes)]
    if fill is not None:
        for v in views:
            fill(v)
    return flat, views


def prepare(case, seed):
    make, damping, gout_std, relu = NETS[case["net"]]
    layers, bf16, op = make(case), case["dtype"] == "bf16", case["op"]
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    s = dict(op=op, damping=damping)
    descs = [l.desc(bf16) for l in layers]
    b = [l.rows for l in layers]
    h, w = [l.h for l in layers], [l.w for l in layers]
    scale = [1.0 / l.rows for l in layers]                # conv: summed over positions, averaged over the examples
    if op == "layer":
        s["work"] = torch.empty(kf.kfac_workspace_bytes(descs[0], b[0], h[0], w[0]), dtype=torch.uint8, device=DEV)
        s.update(descs=descs, b=b, h=h, w=w, scale=scale)
    else:
        s["work"] = torch.empty(kf.kfac_workspace_bytes_batched(descs, b, h, w), dtype=torch.uint8, device=DEV)
        s.update(descs=kf.marshal_descs(descs), b=kf.marshal_ints(b), h=kf.marshal_ints(h), w=kf.marshal_ints(w),
                 scale=kf.marshal_floats(scale))
    ptrs = (lambda v: v) if op == "layer" else kf.marshal_ptrs

    def buffer(name, shapes, fill=None):
        s[name + "_flat"], views = _views(shapes, fill)
        s[name + "_views"] = views                        # the C arrays hold addresses only
        s[name] = ptrs(views)

    sq_A, sq_G = [(l.d_A, l.d_A) for l in layers], [(l.d_G, l.d_G) for l in layers]
    if op != "precondition":
        s["acts"], s["gouts"] = [], []
        for l in layers:
            a = torch.randn((l.rows, l.c_in, l.h, l.w) if l.conv else (l.rows, l.c_in), generator=g, device=DEV)
            o = torch.randn((l.rows, l.c_out, l.h_out, l.w_out) if l.conv else (l.rows, l.c_out), generator=g, device=DEV)
            a = a.relu_() if relu else a
            o.mul_(gout_std)
            s["acts"].append(a.bfloat16() if bf16 else a)
            s["gouts"].append(o.bfloat16() if bf16 else o)
        eye = lambda v: v.fill_diagonal_(1.0)  # noqa: E731
        buffer("A_run", sq_A, eye)
        buffer("G_run", sq_G, eye)
    if op != "factors":
        s["grads"] = [torch.randn((l.d_G, l.d_A), generator=g, device=DEV) for l in layers]
        buffer("out", [(l.d_G, l.d_A) for l in layers])

        def inverse(v):                                   # symmetric, dominated by its diagonal
            r = torch.randn(v.shape, generator=g, device=DEV)
            v.copy_((r + r.T) * (0.05 / math.sqrt(v.shape[0])))
            v.diagonal().add_(torch.rand(v.shape[0], generator=g, device=DEV) + 0.5)
        fill = inverse if op == "precondition" else None
        buffer("A_inv", sq_A, fill)                       # eigen: the eigenvectors
        buffer("G_inv", sq_G, fill)
    if op == "eigen":
        buffer("v_A", [(l.d_A,) for l in layers])
        buffer("v_G", [(l.d_G,) for l in layers])
    s["info"] = torch.zeros(2 * len(layers), dtype=torch.int32, device=DEV)
    return s


def run(s):
    op, lam = s["op"], s["damping"]
    if op == "layer":
        d = s["descs"][0]
        A, G, Ai, Gi, out = (s[k][0] for k in ("A_run", "G_run", "A_inv", "G_inv", "out"))
        kf.kfac_update_factors(d, s["acts"][0], s["gouts"][0], s["b"][0], s["h"][0], s["w"][0], s["scale"][0],
                               s["scale"][0], DECAY, A, G, s["work"])
        kf.kfac_invert(d, A, G, lam, lam, Ai, Gi, s["info"], s["work"])
        kf.kfac_precondition(d, Ai, Gi, s["grads"][0], out, s["work"])
    else:
        d = s["descs"]
        if op != "precondition":
            kf.kfac_update_factors_batched(d, s["acts"], s["gouts"], s["b"], s["h"], s["w"], s["scale"], s["scale"],
                                           DECAY, s["A_run"], s["G_run"], s["work"])
        if op == "update":
            kf.kfac_invert_batched(d, s["A_run"], s["G_run"], lam, lam, s["A_inv"], s["G_inv"], s["info"], s["work"])
        elif op == "update_pi":
            kf.kfac_invert_pi_batched(d, s["A_run"], s["G_run"], lam, s["A_inv"], s["G_inv"], s["info"], None, s["work"])
        elif op == "eigen":
            kf.kfac_eigen_batched(d, s["A_run"], s["G_run"], s["A_inv"], s["v_A"], s["G_inv"], s["v_G"], s["info"],
                                  s["work"])
            kf.kfac_precondition_eigen_batched(d, s["A_inv"], s["v_A"], s["G_inv"], s["v_G"], lam, s["grads"], s["out"],
                                               s["work"])
        if op in ("update", "update_pi", "precondition"):
            kf.kfac_precondition_batched(d, s["A_inv"], s["G_inv"], s["grads"], s["out"], s["work"])
    # eigenvectors are unique up to sign and order only: Eq. 13's result, made of all of them, stands for them
    names = {"factors": ("A_run", "G_run"), "precondition": ("out",), "eigen": ("A_run", "G_run", "out")}.get(
        op, ("A_run", "G_run", "A_inv", "G_inv", "out"))
    got = {k: s[k + "_flat"] for k in names}
    if op not in ("factors", "precondition"):
        got["info"] = s["info"]
    return got


def work(case):
    op, e = case["op"], 2 if case["dtype"] == "bf16" else 4
    nbytes = flops = 0.0
    for l in _layers(case):
        A, G = l.d_A, l.d_G
        if op != "precondition":
            ins = l.rows * l.c_in * l.h * l.w + l.R * l.c_out
            nbytes += ins * e + 4.0 * (A * (A + 1) / 2 + G * (G + 1) / 2 + A * A + G * G)
            flops += 1.0 * l.R * (A * (A + 1) + G * (G + 1))
        if op in ("layer", "update", "update_pi"):
            nbytes += 4.0 * (A * A + G * G)
            flops += 1.0 * A ** 3 + 1.0 * G ** 3
        if op == "eigen":                                 # reduction to tridiagonal form and the vectors back from it
            nbytes += 4.0 * (A * A + G * G + A + G)
            flops += 4.0 * (A ** 3 + G ** 3)
        if op == "precondition":
            nbytes += 4.0 * (A * A + G * G)
        if op != "factors":
            nbytes += 8.0 * A * G
            flops += (2.0 if op != "eigen" else 4.0) * A * G * (A + G)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Factors and products are 32-bit sums.  An inverse at 32 bits carries the condition number of the damped factor
    (1e3 to 1e4 here) times 2^-24, and so does what is computed from it."""
    return {"rel": 1e-5 if case["op"] in ("factors", "precondition") else 1e-4}

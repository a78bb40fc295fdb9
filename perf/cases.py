"""The work a user of the library has it do, as cases that can be timed and checked.

Every case is one pass through the public entry points of ``paper_1504_04343_amd.binding`` on
tensors that already live on the GPU, with the descriptors and workspaces a program keeps between
calls.  The kinds:

  ``conv``   one convolutional layer: a forward pass alone (inference), or a training step of the
             layer (forward, backward-weights with the bias gradient, backward-data);
  ``fc``     the same for a fully connected layer, which the library takes as a convolution whose
             kernel covers the whole input;
  ``glue``   what CaffeNet puts between two convolutions: ReLU, max pooling and local response
             normalisation, forward and backward;
  ``head``   the end of a classifier in training: dropout, a fully connected layer, the softmax
             loss, and the gradients back to the features;
  ``net``    the inference pass of a whole CaffeNet-shaped network: five convolutions with their
             glue layers and three fully connected layers, up to the logits.

Shapes are CaffeNet's layers, the small configuration, the channel-ratio sweep and generic layers
of the same ranges: 3 to 512 channels, 6 to 227 pixels, kernels of 1 to 11 pixels, batches of 1 to
1024 images.
"""
import math

import torch
import torch.nn.functional as F

from paper_1504_04343_amd import binding as B


def conv(name, N, C, H, O, K, stride=1, pad=0, groups=1, train=True, bf16=False, x="relu"):
    return dict(name=name, kind="conv", N=N, C=C, H=H, O=O, K=K, stride=stride, pad=pad,
                groups=groups, train=train, bf16=bf16, x=x)


def listed():
    return [
        # one small layer called alone (batch 4 of 3 x 32 x 32 images, 16 kernels of 5 x 5): what
        # counts is launches and latency
        conv("small_forward", 4, 3, 32, 16, 5, 1, 2, train=False, x="uniform"),
        # answering one request: a CaffeNet-shaped network on a single image; most of its layers
        # are too small to fill the chip, and its fully connected weights are read for one image
        dict(name="net_one_image", kind="net", N=1),
        # CaffeNet's first layer in training: 3 channels, 11 x 11 kernels, stride 4, 227 x 227 images
        conv("conv1_train", 256, 3, 227, 96, 11, 4, 0, x="uniform"),
        # the layer with the most work: 5 x 5 kernels, two groups
        conv("conv2_train", 256, 96, 27, 256, 5, 1, 2, 2),
        # a deep 3 x 3 layer at the largest batch that the library is benchmarked with
        conv("conv3_train_large_batch", 1024, 256, 13, 384, 3, 1, 1),
        # the same kind of layer at a small batch that is no multiple of anything
        conv("conv5_train_small_batch", 50, 384, 13, 256, 3, 1, 1, 2),
        # training with bf16 operands and fp32 accumulation
        conv("conv4_train_bf16", 256, 384, 13, 384, 3, 1, 1, 2, bf16=True),
        # 1 x 1 kernels that reduce the channels of a 28 x 28 plane
        conv("pointwise_forward", 128, 256, 28, 64, 1, train=False, x="uniform"),
        # many channels in, few out: the end of the channel-ratio sweep where the lowering on the
        # output side is the cheapest
        conv("narrow_forward", 128, 512, 28, 16, 3, 1, 1, train=False, x="uniform"),
        # CaffeNet's first fully connected layer in training (256 x 6 x 6 features, 4096 outputs)
        dict(name="fc6_train", kind="fc", N=256, C=256, H=6, O=4096),
        # what follows conv1 in training: ReLU, 3 x 3 max pooling with stride 2, normalisation
        dict(name="relu_pool_norm_train", kind="glue", N=256, C=96, H=55, K=3, stride=2),
        # the classifier's end in training: dropout on 4096 features, 1000 classes, softmax loss
        dict(name="head_train", kind="head", N=256, F=4096, classes=1000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_conv(rng):
    """A CaffeNet layer at another batch, or a generic layer of the same ranges."""
    train = rng.random() < 0.7
    bf16 = rng.random() < 0.25
    if rng.random() < 0.45:
        N = _log_int(rng, 1, 700)
        C, H, O, K, stride, pad, groups = rng.choice([
            (3, 227, 96, 11, 4, 0, 1), (96, 27, 256, 5, 1, 2, 2), (256, 13, 384, 3, 1, 1, 1),
            (384, 13, 384, 3, 1, 1, 2), (384, 13, 256, 3, 1, 1, 2)])
        return conv("", N, C, H, O, K, stride, pad, groups, train, bf16,
                    "uniform" if C == 3 else "relu")
    K = rng.choice([1, 1, 3, 3, 3, 5, 7])
    groups = rng.choice([1, 1, 1, 2])
    stride = rng.choice([1, 1, 1, 2])
    H = rng.randint(max(7, K), 56)
    pad = rng.choice([0, K // 2])
    Cg = _log_int(rng, 3, 512 // groups)
    Og = _log_int(rng, 16, 512 // groups)
    if rng.random() < 0.5:   # channel counts in use are mostly round, but not all
        Cg, Og = max(8, Cg // 8 * 8), max(16, Og // 16 * 16)
    return conv("", _log_int(rng, 1, 256), Cg * groups, H, Og * groups, K, stride, pad, groups,
                train, bf16, rng.choice(["uniform", "relu"]))


def draw(rng):
    u = rng.random()
    while True:
        if u < 0.60:
            case = _draw_conv(rng)
        elif u < 0.72:
            case = dict(name="", kind="fc", N=_log_int(rng, 1, 512), C=_log_int(rng, 16, 512),
                        H=rng.choice([1, 1, 5, 6, 7]), O=_log_int(rng, 10, 4096))
        elif u < 0.84:
            K, stride = rng.choice([(3, 2), (3, 2), (2, 2)])
            case = dict(name="", kind="glue", N=_log_int(rng, 1, 256), C=_log_int(rng, 16, 384),
                        H=rng.randint(7, 60), K=K, stride=stride)
        elif u < 0.92:
            case = dict(name="", kind="head", N=_log_int(rng, 1, 512), F=_log_int(rng, 64, 4096),
                        classes=_log_int(rng, 10, 1000))
        else:
            case = dict(name="", kind="net", N=_log_int(rng, 1, 16))
        del case["name"]
        w = work(case)
        # no more than the largest listed case, whose work is 918 GFLOP; traffic no more than
        # that of the glue layers after conv1
        if w["flops"] <= 9.0e11 and w["bytes"] <= 2.4e9:
            return case


# ---- shapes -------------------------------------------------------------------------------------

def _out(H, K, stride, pad):
    return (H + 2 * pad - K) // stride + 1


def _pool_out(H, K, stride):
    return -(-(H - K) // stride) + 1


# CaffeNet: conv (C, O, K, stride, pad, groups), pooled / normalised after it or not
_NET = [(3, 96, 11, 4, 0, 1, True, True), (96, 256, 5, 1, 2, 2, True, True),
        (256, 384, 3, 1, 1, 1, False, False), (384, 384, 3, 1, 1, 2, False, False),
        (384, 256, 3, 1, 1, 2, True, False)]
_NET_H = 227
_NET_FC = [(256, 6, 4096), (4096, 1, 4096), (4096, 1, 1000)]


def _net_layers():
    """(kind, shape parameters) of every layer, with the plane size it sees."""
    H = _NET_H
    for C, O, K, s, p, g, pool, norm in _NET:
        Ho = _out(H, K, s, p)
        yield "conv", (C, H, O, K, s, p, g, Ho)
        H = Ho
        if pool:
            Hp = _pool_out(H, 3, 2)
            yield "pool", (O, H, Hp)
            H = Hp
        if norm:
            yield "norm", (O, H)
    for i, (C, Hf, O) in enumerate(_NET_FC):
        yield "fc", (C, Hf, O, i + 1 < len(_NET_FC))


# ---- what a program has in hand before the call -------------------------------------------------

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _randn(g, *shape, std=1.0):
    return torch.randn(shape, generator=g, device="cuda").mul_(std)


def _activations(g, dist, *shape):
    """relu: outputs of a ReLU layer, about half of them zero; uniform: an image in [-1, 1]."""
    if dist == "relu":
        return torch.randn(shape, generator=g, device="cuda").relu_()
    return torch.rand(shape, generator=g, device="cuda").mul_(2.0).sub_(1.0)


def _conv_state(case, seed):
    g = _gen(seed)
    fc = case["kind"] == "fc"
    N, C, H, O = case["N"], case["C"], case["H"], case["O"]
    K, stride, pad, groups = (H, 1, 0, 1) if fc else (case["K"], case["stride"], case["pad"],
                                                      case["groups"])
    train = True if fc else case["train"]
    bf16 = (not fc) and case["bf16"]
    Ho = _out(H, K, stride, pad)
    fan_in = C // groups * K * K
    s = dict(x=_activations(g, "relu" if fc else case["x"], N, C, H, H),
             w=_randn(g, O, C // groups, K, K, std=(2.0 / fan_in) ** 0.5),
             b=_randn(g, O, std=0.1))
    d = B.make_desc(N, C, H, H, O, K, stride, pad, groups,
                    precision=B.PREC_BF16_IN_F32_ACC if bf16 else B.PREC_F32)
    s["desc"] = d
    s["y"] = torch.empty(N, O, Ho, Ho, device="cuda")
    s["ws_f"] = B.alloc_workspace(d, B.PASS_FORWARD)
    if train:
        s["dy"] = _randn(g, N, O, Ho, Ho)
        s["dx"], s["dw"], s["db"] = (torch.empty_like(s[k]) for k in ("x", "w", "b"))
        s["ws_d"] = B.alloc_workspace(d, B.PASS_BACKWARD_DATA)
        s["ws_w"] = B.alloc_workspace(d, B.PASS_BACKWARD_WEIGHTS)
    return s


def _glue_state(case, seed):
    g = _gen(seed)
    N, C, H, K, stride = (case[k] for k in ("N", "C", "H", "K", "stride"))
    Ho = _pool_out(H, K, stride)
    s = dict(x=_randn(g, N, C, H, H, std=4.0), dy=_randn(g, N, C, Ho, Ho),
             pool=B.make_pool_desc(N, C, H, H, K, stride), lrn=B.make_lrn_desc(N, C, Ho, Ho))
    s["a"], s["da"], s["dx"] = (torch.empty_like(s["x"]) for _ in range(3))
    s["p"], s["n"], s["dp"] = (torch.empty_like(s["dy"]) for _ in range(3))
    s["arg"] = torch.empty(N, C, Ho, Ho, dtype=torch.int32, device="cuda")
    return s


def _head_state(case, seed):
    g = _gen(seed)
    N, Fe, cl = case["N"], case["F"], case["classes"]
    s = dict(x=_activations(g, "relu", N, Fe, 1, 1), w=_randn(g, cl, Fe, 1, 1, std=Fe ** -0.5),
             b=_randn(g, cl, std=0.1),
             mask=(torch.rand(N, Fe, 1, 1, generator=g, device="cuda") < 0.5).to(torch.uint8),
             label=torch.randint(0, cl, (N,), generator=g, device="cuda", dtype=torch.int32),
             desc=B.make_desc(N, Fe, 1, 1, cl, 1))
    s["h"], s["dh"], s["dx"] = (torch.empty_like(s["x"]) for _ in range(3))
    s["score"] = torch.empty(N, cl, 1, 1, device="cuda")
    s["prob"], s["dscore"] = (torch.empty(N, cl, device="cuda") for _ in range(2))
    s["image_loss"], s["loss"] = torch.empty(N, device="cuda"), torch.empty(1, device="cuda")
    s["dw"], s["db"] = torch.empty_like(s["w"]), torch.empty_like(s["b"])
    s["ws_f"] = B.alloc_workspace(s["desc"], B.PASS_FORWARD)
    s["ws_d"] = B.alloc_workspace(s["desc"], B.PASS_BACKWARD_DATA)
    s["ws_w"] = B.alloc_workspace(s["desc"], B.PASS_BACKWARD_WEIGHTS)
    return s


def _net_state(case, seed):
    g = _gen(seed)
    N = case["N"]
    steps = []
    for kind, p in _net_layers():
        if kind in ("conv", "fc"):
            if kind == "conv":
                C, H, O, K, s, pad, gr, Ho = p
                relu = True
            else:
                C, H, O, relu = p
                K, s, pad, gr, Ho = H, 1, 0, 1, 1
            d = B.make_desc(N, C, H, H, O, K, s, pad, gr)
            fan_in = C // gr * K * K
            steps.append(dict(kind="conv", desc=d, relu=relu, shape=(N, C, H, H),
                              w=_randn(g, O, C // gr, K, K, std=(2.0 / fan_in) ** 0.5),
                              b=_randn(g, O, std=0.05), ws=B.alloc_workspace(d, B.PASS_FORWARD),
                              y=torch.empty(N, O, Ho, Ho, device="cuda")))
        elif kind == "pool":
            O, H, Hp = p
            steps.append(dict(kind="pool", desc=B.make_pool_desc(N, O, H, H, 3, 2),
                              y=torch.empty(N, O, Hp, Hp, device="cuda")))
        else:
            O, H = p
            steps.append(dict(kind="norm", desc=B.make_lrn_desc(N, O, H, H),
                              y=torch.empty(N, O, H, H, device="cuda")))
    return dict(x=_activations(g, "uniform", N, 3, _NET_H, _NET_H), steps=steps)


def prepare(case, seed):
    make = {"conv": _conv_state, "fc": _conv_state, "glue": _glue_state, "head": _head_state,
            "net": _net_state}[case["kind"]]
    return dict(kind=case["kind"], **make(case, seed))


# ---- one pass -----------------------------------------------------------------------------------

def _run_conv(s):
    B.cct_conv_forward(s["desc"], s["x"], s["w"], s["b"], s["y"], s["ws_f"])
    if "dy" not in s:
        return dict(y=s["y"])
    B.cct_conv_backward_weights(s["desc"], s["x"], s["dy"], s["dw"], s["db"], s["ws_w"])
    B.cct_conv_backward_data(s["desc"], s["w"], s["dy"], s["dx"], s["ws_d"])
    return dict(y=s["y"], dw=s["dw"], db=s["db"], dx=s["dx"])


def _run_glue(s):
    B.cct_relu_forward(s["x"], s["a"])
    B.cct_maxpool_forward(s["pool"], s["a"], s["p"], s["arg"])
    B.cct_lrn_forward(s["lrn"], s["p"], s["n"])
    B.cct_lrn_backward(s["lrn"], s["p"], s["dy"], s["dp"])
    B.cct_maxpool_backward(s["pool"], s["dp"], s["arg"], s["da"])
    B.cct_relu_backward(s["a"], s["da"], s["dx"])
    return dict(a=s["a"], p=s["p"], arg=s["arg"], n=s["n"], dp=s["dp"], da=s["da"], dx=s["dx"])


def _run_head(s):
    scale = 2.0
    B.cct_dropout_forward(s["x"], s["mask"], scale, s["h"])
    B.cct_conv_forward(s["desc"], s["h"], s["w"], s["b"], s["score"], s["ws_f"])
    N, cl = s["prob"].shape
    B.cct_softmax_loss_forward(s["score"].view(N, cl), s["label"], s["prob"], s["image_loss"],
                               s["loss"])
    B.cct_softmax_loss_backward(s["prob"], s["label"], s["dscore"])
    ds = s["dscore"].view(N, cl, 1, 1)
    B.cct_conv_backward_weights(s["desc"], s["h"], ds, s["dw"], s["db"], s["ws_w"])
    B.cct_conv_backward_data(s["desc"], s["w"], ds, s["dh"], s["ws_d"])
    B.cct_dropout_backward(s["dh"], s["mask"], scale, s["dx"])
    return dict(score=s["score"], prob=s["prob"], loss=s["loss"], dscore=s["dscore"], dw=s["dw"],
                db=s["db"], dx=s["dx"])


def _run_net(s):
    t = s["x"]
    for st in s["steps"]:
        if st["kind"] == "conv":
            B.cct_conv_forward(st["desc"], t.view(st["shape"]), st["w"], st["b"], st["y"], st["ws"])
            if st["relu"]:
                B.cct_relu_forward(st["y"], st["y"])
        elif st["kind"] == "pool":
            B.cct_maxpool_forward(st["desc"], t, st["y"])
        else:
            B.cct_lrn_forward(st["desc"], t, st["y"])
        t = st["y"]
    return dict(logits=t)


def run(state):
    return {"conv": _run_conv, "fc": _run_conv, "glue": _run_glue, "head": _run_head,
            "net": _run_net}[state["kind"]](state)


# ---- what a pass cannot do without: every call reads its inputs once and writes its outputs once --

def _conv_work(N, C, H, O, K, stride, pad, groups, train):
    Ho = _out(H, K, stride, pad)
    x, y, w = N * C * H * H, N * O * Ho * Ho, O * (C // groups) * K * K
    flops = 2 * y * (C // groups) * K * K
    once = 4 * (x + y + w + O)
    return (3 * once, 3 * flops + y) if train else (once, flops)


def work(case):
    k = case["kind"]
    N = case["N"]
    if k == "conv":
        by, fl = _conv_work(*(case[i] for i in ("N", "C", "H", "O", "K", "stride", "pad", "groups",
                                                "train")))
    elif k == "fc":
        by, fl = _conv_work(N, case["C"], case["H"], case["O"], case["H"], 1, 0, 1, True)
    elif k == "glue":
        Ho = _pool_out(case["H"], case["K"], case["stride"])
        x, y = N * case["C"] * case["H"] ** 2, N * case["C"] * Ho * Ho
        by = 4 * ((2 + 3) * x + (x + 2 * y) * 2 + (2 + 3) * y)
        fl = 2 * x + 2 * case["K"] ** 2 * y + 40 * y
    elif k == "head":
        Fe, cl = case["F"], case["classes"]
        by, fl = _conv_work(N, Fe, 1, cl, 1, 1, 0, 1, True)
        by += 2 * 9 * N * Fe + 16 * N * cl
        fl += 2 * N * Fe + 6 * N * cl
    else:
        by = fl = 0
        for kind, p in _net_layers():
            if kind == "conv":
                C, H, O, K, s, pad, gr, Ho = p
                b1, f1 = _conv_work(N, C, H, O, K, s, pad, gr, False)
                b1 += 8 * N * O * Ho * Ho
            elif kind == "fc":
                b1, f1 = _conv_work(N, p[0], p[1], p[2], p[1], 1, 0, 1, False)
                b1 += 8 * N * p[2] if p[3] else 0
            elif kind == "pool":
                b1, f1 = 4 * N * p[0] * (p[1] ** 2 + p[2] ** 2), 9 * N * p[0] * p[2] ** 2
            else:
                b1, f1 = 8 * N * p[0] * p[1] ** 2, 15 * N * p[0] * p[1] ** 2
            by, fl = by + b1, fl + f1
    return dict(bytes=by, flops=fl)


def tolerance(case):
    """About four times the error that the fp32 path shows against 64 bits over these ranges."""
    if case["kind"] == "conv" and case["bf16"]:
        return {"rel": 1e-2, "max": 6e-2}   # the operands' rounding to 8 bits (measured 2.4e-3, 1.3e-2)
    if case["kind"] == "glue":
        return {"rel": 5e-7, "max": 1e-5}   # a power and short sums (measured 5e-8, 1.4e-6)
    return {"rel": 5e-6, "max": 4e-5}       # sums of up to 260 000 products (measured 1.4e-6, 9.4e-6)


# ---- the same in 64 bits, plain torch -----------------------------------------------------------

def _conv64(x, w, b, stride, pad, groups, dy=None):
    """y, and for a given dy also dw, db, dx, by unfolding a few images at a time."""
    N, C, H, _ = x.shape
    O, Cg, K, _ = w.shape
    Ho = _out(H, K, stride, pad)
    w2 = w.double().view(groups, O // groups, Cg * K * K)
    y = torch.empty(N, O, Ho, Ho, dtype=torch.float64, device=x.device)
    dx = torch.empty(x.shape, dtype=torch.float64, device=x.device) if dy is not None else None
    dw = torch.zeros_like(w2)
    step = max(1, int(2.5e8 // (C * K * K * Ho * Ho)))
    for n in range(0, N, step):
        xc = x[n:n + step].double()
        m = xc.shape[0]
        cols = F.unfold(xc, K, padding=pad, stride=stride).view(m, groups, Cg * K * K, Ho * Ho)
        cols = cols.permute(1, 2, 0, 3).reshape(groups, Cg * K * K, m * Ho * Ho)
        yc = [w2[q] @ cols[q] for q in range(groups)]
        y[n:n + step] = torch.cat(yc).view(O, m, Ho, Ho).transpose(0, 1)
        if dy is None:
            continue
        g = dy[n:n + step].double().transpose(0, 1).reshape(groups, O // groups, m * Ho * Ho)
        dcols = torch.empty_like(cols)
        for q in range(groups):
            dw[q] += g[q] @ cols[q].t().contiguous()
            dcols[q] = w2[q].t().contiguous() @ g[q]
        dcols = dcols.view(C * K * K, m, Ho * Ho).transpose(0, 1).contiguous()
        dx[n:n + step] = F.fold(dcols, (H, H), K, padding=pad, stride=stride)
    y += b.double().view(1, O, 1, 1)
    if dy is None:
        return y
    return y, dw.view(w.shape), dy.double().sum((0, 2, 3)), dx


def _lrn64(x, size=5, alpha=1e-4, beta=0.75, k=1.0):
    sq = F.pad(x * x, (0, 0, 0, 0, size // 2, size // 2))
    C = x.shape[1]
    win = sum(sq[:, i:i + C] for i in range(size))
    return x * (k + alpha / size * win) ** -beta


def exact(case, seed):
    s = prepare(case, seed)
    k = case["kind"]
    if k in ("conv", "fc"):
        st, pad, gr = (1, 0, 1) if k == "fc" else (case["stride"], case["pad"], case["groups"])
        if "dy" not in s:
            return dict(y=_conv64(s["x"], s["w"], s["b"], st, pad, gr))
        y, dw, db, dx = _conv64(s["x"], s["w"], s["b"], st, pad, gr, s["dy"])
        return dict(y=y, dw=dw, db=db, dx=dx)
    if k == "glue":
        K, stride = case["K"], case["stride"]
        a = s["x"].double().relu().requires_grad_()
        p, arg = F.max_pool2d(a, K, stride, ceil_mode=True, return_indices=True)
        pl = p.detach().requires_grad_()
        n = _lrn64(pl)
        dp, = torch.autograd.grad(n, pl, s["dy"].double())
        da, = torch.autograd.grad(p, a, dp)
        return dict(a=a.detach(), p=p.detach(), arg=arg.to(torch.int32), n=n.detach(), dp=dp, da=da,
                    dx=da * (s["x"] > 0))
    if k == "head":
        N, cl = case["N"], case["classes"]
        keep = s["mask"].double().view(N, -1) * 2.0
        h = s["x"].double().view(N, -1) * keep
        w = s["w"].double().view(cl, -1)
        score = h @ w.t().contiguous() + s["b"].double()
        prob = torch.softmax(score, 1)
        label = s["label"].long()
        loss = F.cross_entropy(score, label).view(1)
        ds = (prob - F.one_hot(label, cl).double()) / N
        dx = (ds @ w) * keep
        return dict(score=score.view(N, cl, 1, 1), prob=prob, loss=loss, dscore=ds,
                    dw=(ds.t().contiguous() @ h).view(s["w"].shape), db=ds.sum(0),
                    dx=dx.view(s["x"].shape))
    t = s["x"].double()
    for st in s["steps"]:
        if st["kind"] == "conv":
            d = st["desc"]
            t = _conv64(t.view(st["shape"]), st["w"], st["b"], d.stride, d.pad, d.groups)
            t = t.relu() if st["relu"] else t
        elif st["kind"] == "pool":
            t = F.max_pool2d(t, 3, 2, ceil_mode=True)
        else:
            t = _lrn64(t)
    return dict(logits=t)

"""The work that performance is measured on: one worker's calls into this framework, over the range of networks, batches
and images that its configurations, tests and benchmark use.

A case is one call sequence of a user's program ("do"):
  attack    dat_attack + dat_make_xadv: the inner maximisation, the larger part of every training iteration and all of an
            evaluation; `losses` asks for the loss at every iterate (an evaluation or a monitored run), which ends on the host
  step      the outer gradient at an adversarial batch
  trades    the same for the semi-supervised objective, TRADES regulariser + clean loss (two forward, two backward sweeps)
  worker    the whole iteration of the fp32 toy model: FGSM, gradient, update, quantizer and its inverse
  exchange  dat_quantize + dat_dequantize of a gradient with a real tensor table
  server    dat_aggregate of M workers' packed gradients

Networks start near the identity: the last batch-norm scale of every residual branch is 0.001, the start of large-batch
training.  Every tensor carries ordinary non-zero values then, and the outputs can be compared: with unit scales two
correct bf16 implementations of these networks differ by 10 to 100 % in the gradients (a rounding that falls the other
way moves a ReLU or a sign, and the deep network amplifies it), near the identity by less than 1 %.
"""
import math

import torch

import paper_2206_06257_amd as dat

MEAN, STD = (0.485, 0.456, 0.406), (0.229, 0.224, 0.225)
NETS = {   # architecture, classes, normalised input, eps, layers' table
    "tinycnn": (0, 10, False, 8 / 255),
    "resnet18": (1, 10, False, 8 / 255),
    "preact_resnet18": (4, 10, False, 8 / 255),
    "wrn28_10": (5, 10, False, 8 / 255),
    "wrn34_10": (2, 10, False, 8 / 255),
    "resnet50": (3, 1000, True, 2 / 255),
}
BRANCH_GAMMA = 0.001


def listed():
    return [
        # the smallest call: the fp32 toy configuration, every launch of an iteration a few microseconds long
        {"name": "worker_tinycnn_b32", "do": "worker", "net": "tinycnn", "B": 32, "H": 32, "bits": 8},
        # an odd handful of images against a small network (evaluation of a few samples): latency and launch count
        {"name": "attack_preact18_b13", "do": "attack", "net": "preact_resnet18", "B": 13, "H": 32, "K": 10, "losses": True},
        # CIFAR training, the inner maximisation at the configured batch
        {"name": "attack_resnet18_b512", "do": "attack", "net": "resnet18", "B": 512, "H": 32, "K": 10, "losses": False},
        # ... and its outer step on a last, odd-sized batch of an epoch
        {"name": "step_resnet18_b391", "do": "step", "net": "resnet18", "B": 391, "H": 32},
        # the widest CIFAR network
        {"name": "attack_wrn34_b256", "do": "attack", "net": "wrn34_10", "B": 256, "H": 32, "K": 10, "losses": False},
        # semi-supervised training: TRADES objective with a clean-loss term
        {"name": "trades_wrn28_b128", "do": "trades", "net": "wrn28_10", "B": 128, "H": 32, "lam": 1.0},
        # ImageNet training at the benchmark's configuration: the largest call
        {"name": "attack_resnet50_b256", "do": "attack", "net": "resnet50", "B": 256, "H": 224, "K": 10, "losses": False},
        # 85 images per GPU and four PGD steps, with the losses watched
        {"name": "attack_resnet50_b85", "do": "attack", "net": "resnet50", "B": 85, "H": 224, "K": 4, "losses": True},
        # the outer step of the benchmark's configuration
        {"name": "step_resnet50_b256", "do": "step", "net": "resnet50", "B": 256, "H": 224},
        # the outer step at a small share of a batch, smaller images
        {"name": "step_resnet50_b50_160", "do": "step", "net": "resnet50", "B": 50, "H": 160},
        # gradient compression of a 25.6 M parameter network
        {"name": "exchange_resnet50_8bit", "do": "exchange", "net": "resnet50", "bits": 8},
        # averaging eight workers' gradients
        {"name": "server_resnet50_m8", "do": "server", "net": "resnet50", "bits": 8, "M": 8},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    do = rng.choice(["attack"] * 9 + ["step"] * 5 + ["trades"] * 2 + ["exchange"] * 2 + ["server", "worker"])
    if do == "worker":
        return {"do": do, "net": "tinycnn", "B": _log_int(rng, 8, 128), "H": rng.randint(24, 40), "bits": rng.choice([4, 8])}
    if do == "exchange":
        return {"do": do, "net": rng.choice(["resnet18", "wrn28_10", "resnet50"]), "bits": rng.choice([2, 4, 8, 16]), "shift": rng.randint(0, 99999)}
    if do == "server":
        return {"do": do, "net": rng.choice(["resnet18", "resnet50"]), "bits": rng.choice([4, 8, 16]), "M": rng.randint(2, 16)}
    net = rng.choice(["resnet18", "preact_resnet18", "wrn28_10", "wrn34_10"] + ["resnet50"] * 3)
    if do == "trades" and net == "resnet50":
        net = "preact_resnet18"
    if net == "resnet50":
        H = rng.choice([96, 128, 160, 161, 192, 224, 224, 224])
        B = _log_int(rng, 8, 256)
        if do == "step":   # small sums over few pixels make the gradients of the deepest layers ill-conditioned
            B, H = max(B, 32), max(H, 128)
    else:
        H = rng.choice([24, 28, 32, 32, 32, 33])
        B = _log_int(rng, 8, 480 if "18" in net else 230 if do == "attack" else 128)
    case = {"do": do, "net": net, "B": B, "H": H}
    if do == "attack":
        case.update(K=rng.choice([1, 2, 3, 4, 7, 10]), losses=rng.random() < 0.3)
    elif do == "trades":
        case.update(lam=rng.choice([0.5, 1.0]))
    return case


def _model(case, g):
    arch, classes, norm, _ = NETS[case["net"]]
    dtype = dat.F32 if case["net"] == "tinycnn" else dat.BF16
    m = dat.Model(arch, dtype, case["B"], case["H"], case["H"], classes, MEAN if norm else None, STD if norm else None)
    theta = torch.zeros(m.d, device="cuda")
    for t in range(m.num_tensors):
        part, kind = theta[int(m.offsets[t]):int(m.offsets[t + 1])], int(m.kind[t])
        if kind in (0, 4):
            part.normal_(0.0, math.sqrt(2.0 / int(m.fan_in[t])), generator=g)
        elif kind in (2, 6):
            part.fill_(BRANCH_GAMMA if kind == 6 else 1.0)
    m.set_params(theta.cpu().numpy())
    return m


def _gradient(offsets, g):
    """Per-tensor normal values of very different scales, as a network's layers have them."""
    v = torch.randn(int(offsets[-1]), device="cuda", generator=g)
    scale = (10.0 ** (-4.0 * torch.rand(len(offsets) - 1, device="cuda", generator=g))).tolist()
    for t in range(len(offsets) - 1):
        v[int(offsets[t]):int(offsets[t + 1])] *= scale[t]
    return v


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    do, net = case["do"], case["net"]
    arch, classes, norm, eps = NETS[net]
    s = {"case": dict(case), "seed": int(seed), "it": 0}
    if do in ("exchange", "server"):
        table = dat.Model(arch, dat.BF16, 1, 32, 32, classes)   # the tensor table a program takes from its model
        d, T = table.d, table.num_tensors
        offsets = table.offsets.copy()
        shift = case.get("shift", 0)
        if shift:   # another network's table: the first tensor cut short, every later offset ragged
            cut = shift % max(1, int(offsets[1]) - 1)
            offsets[1:] -= cut
            d -= cut
        offs = torch.from_numpy(offsets).cuda()
        bits = case["bits"]
        s.update(offs=offs, d=d)
        if do == "exchange":
            s.update(grads=_gradient(offsets, g), q=torch.empty(dat.quantized_bytes(d, bits), dtype=torch.uint8, device="cuda"),
                     scales=torch.empty(T, device="cuda"), out=torch.empty(d, device="cuda"))
        else:
            pairs = [dat.quantize(_gradient(offsets, g), offs, bits, int(seed) + w) for w in range(case["M"])]
            s.update(q=[p[0] for p in pairs], scales=[p[1] for p in pairs], out=torch.empty(d, device="cuda"))
        return s
    B, H = case["B"], case["H"]
    m = _model(case, g)
    x = torch.rand(B, H, H, 3, device="cuda", generator=g)
    y = torch.randint(0, classes, (B,), device="cuda", dtype=torch.int32, generator=g)
    s.update(m=m, x=x, y=y, xadv=torch.empty_like(x), eps=eps)
    if do in ("attack", "worker"):
        s.update(delta=torch.empty_like(x))
    if do in ("step", "trades"):   # the batch as an attack leaves it: most pixels at the border of the ball
        torch.clamp(x + eps * torch.sign(torch.randn(x.shape, device="cuda", generator=g)), 0.0, 1.0, out=s["xadv"])
    if do != "attack":
        s.update(grads=torch.empty(m.d, device="cuda"))
    if do == "worker":
        s.update(q=torch.empty(dat.quantized_bytes(m.d, case["bits"]), dtype=torch.uint8, device="cuda"),
                 scales=torch.empty(m.num_tensors, device="cuda"), out=torch.empty(m.d, device="cuda"),
                 offs=torch.from_numpy(m.offsets.copy()).cuda())
    return s


def run(s):
    case, do = s["case"], s["case"]["do"]
    s["it"] += 1
    seed = s["seed"] * 65536 + s["it"]
    if do == "exchange":
        dat.quantize(s["grads"], s["offs"], case["bits"], seed, q=s["q"], scales=s["scales"])
        dat.dequantize(s["q"], s["scales"], s["offs"], s["d"], case["bits"], out=s["out"])
        return s["q"], s["scales"], s["out"]
    if do == "server":
        return dat.aggregate(s["q"], s["scales"], s["offs"], s["d"], case["bits"], out=s["out"])
    m, x, y = s["m"], s["x"], s["y"]
    if do == "attack":
        K = case["K"]
        alpha = 2.5 * s["eps"] / K if K > 1 else 1.25 * s["eps"]
        got = m.attack(x, y, s["eps"], alpha, K, dat.INIT_UNIFORM, seed=seed, delta=s["delta"], want_losses=case["losses"])
        dat.make_xadv(x, s["delta"], out=s["xadv"])
        return (s["xadv"], got[1]) if case["losses"] else s["xadv"]
    if do == "worker":
        m.attack(x, y, s["eps"], 1.25 * s["eps"], 1, dat.INIT_ZERO, delta=s["delta"])
        dat.make_xadv(x, s["delta"], out=s["xadv"])
        m.step(s["xadv"], y, grads=s["grads"])
        dat.quantize(s["grads"], s["offs"], case["bits"], seed, q=s["q"], scales=s["scales"])
        dat.dequantize(s["q"], s["scales"], s["offs"], m.d, case["bits"], out=s["out"])
        m.sgd_update(s["out"], 0.01)
        return s["xadv"], s["grads"], s["out"]
    if do == "step":
        m.step(s["xadv"], y, grads=s["grads"])
    else:
        m.step_reg(x, s["xadv"], y, case["lam"], dat.PHI_TRADES_KL, grads=s["grads"])
    return s["grads"]


# ---- the least work of a case --------------------------------------------------------------------------------------
def _convs(net, H):
    """(output pixels, Cout, k*k*Cin) of every convolution for one image, and (inputs, outputs) of the classifier."""
    out = []

    def conv(h, cin, cout, k, stride):
        h = (h - 1) // stride + 1        # the paddings used keep ceil(h / stride)
        out.append((h * h, cout, k * k * cin))
        return h

    if net == "tinycnn":
        conv(conv(H, 3, 16, 3, 1), 16, 32, 3, 2)
        return out, (32, 10)
    if net == "resnet50":
        h, c = (conv(H, 3, 64, 7, 2) - 1) // 2 + 1, 64
        for w, depth, stride in ((64, 3, 1), (128, 4, 2), (256, 6, 2), (512, 3, 2)):
            for b in range(depth):
                st = stride if b == 0 else 1
                conv(h, c, w, 1, 1)
                ho = conv(h, w, w, 3, st)
                conv(ho, w, 4 * w, 1, 1)
                if b == 0:
                    conv(h, c, 4 * w, 1, st)
                h, c = ho, 4 * w
        return out, (c, 1000)
    if "18" in net:
        c, widths, depth = 64, (64, 128, 256, 512), 2
    else:
        c, widths, depth = 16, (160, 320, 640), 5 if net == "wrn34_10" else 4
    h = conv(H, 3, c, 3, 1)
    for i, w in enumerate(widths):
        for b in range(depth):
            st = 2 if b == 0 and i > 0 else 1
            ho = conv(h, c, w, 3, st)
            conv(ho, w, w, 3, 1)
            if st != 1 or c != w:
                conv(h, c, w, 1, st)
            h, c = ho, w
    return out, (c, 10)


def work(case):
    do, net = case["do"], case["net"]
    convs, (fi, fo) = _convs(net, case.get("H", 32))
    weights = sum(co * kk for _, co, kk in convs) + fi * fo
    if do == "exchange":
        return {"bytes": weights * (4 + case["bits"] / 8 + 4), "flops": 0}
    if do == "server":
        return {"bytes": weights * (case["M"] * case["bits"] / 8 + 4), "flops": 2 * weights * case["M"]}
    B = case["B"]
    sweep = B * (2.0 * sum(p * co * kk for p, co, kk in convs) + 2.0 * fi * fo)   # one direction through the network
    image = 12 * B * case["H"] ** 2
    if do == "attack":      # pixels in, perturbed pixels and perturbation out; weights once
        return {"bytes": 3 * image + 2 * weights, "flops": sweep * (2 * case["K"] + (1 if case["losses"] else 0))}
    if do == "worker":
        return {"bytes": 3 * image + 20 * weights, "flops": 5 * sweep}
    if do == "trades":
        return {"bytes": 2 * image + 14 * weights, "flops": 6 * sweep}
    return {"bytes": image + 14 * weights, "flops": 3 * sweep}


def tolerance(case):
    """Measured by running the same samples in another order within the batch, which reorders every sum over pixels and
    images: adversarial pixels 0.005 to 0.02 (eps 8/255) and 0.006 (eps 2/255), single pixels by up to the width of the
    ball; gradients 0.0001 to 0.0002 (wide networks), 0.003 (18 layers), 0.004 to 0.008 (50 layers), single elements by
    0.1 to 0.9 of the root mean square (the first layer's are the largest, and the mean runs over millions of small ones)."""
    do = case["do"]
    if do in ("exchange", "server"):
        return "exact"
    if do == "worker":        # fp32 throughout; a code of the quantizer may fall the other way
        return {"rel": 2e-3, "max": 0.2}
    if do == "attack":
        return {"rel": 0.03 if NETS[case["net"]][3] > 0.02 else 0.02, "max": 0.25}
    return {"rel": 0.03 if case["net"] == "resnet50" else 0.012, "max": 0.99}

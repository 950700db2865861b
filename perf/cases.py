"""Timing cases of the ResIST hot path: what a user of the library has it do, through its public entry points.

Four kinds of work, each over a range of sizes, data types and options:

  step      one local SGD iteration of one sub-ResNet (forward, backward, momentum update): `local_step`
  predict   the test-time forward pass of the reassembled global model, residual branches scaled by 1/S: `forward`
  exchange  the end of a synchronisation round: reassembly of the global model from S sub-ResNets, plain (`aggregate`)
            or with every communicated parameter compressed to b bits in both directions (`compress_blocks`,
            `aggregate_compressed`, `decompress_blocks`)
  conv      one convolution layer on its own: forward, data gradient and weight gradient

Networks are the three shapes the repository's configurations use: "tiny" (two basic blocks at 16 channels on 16x16
images), "cifar" (basic blocks [3, 4, 23, 3] on 32x32 images) and "imagenet" (bottleneck blocks [3, 4, 6, 3] behind a 7x7
stem and a max-pool), as post- or pre-activation blocks.  Values: images N(0, 1), Kaiming-normal (fan-out) filters, BN scale
near 1, uniform labels -- those of the repository's seeded inputs, drawn on the GPU.
"""
import math

import torch

import paper_2107_00961_amd as R

_NETS = {
    "tiny": dict(block_kind=0, stem_kind=0, widths=[16], blocks=[2]),
    "cifar": dict(block_kind=0, stem_kind=0, widths=[64, 128, 256, 512], blocks=[3, 4, 23, 3]),
    "imagenet": dict(block_kind=1, stem_kind=1, widths=[64, 128, 256, 512], blocks=[3, 4, 6, 3]),
}


def listed():
    return [
        # the smallest training call: two blocks at 16 channels, batch 4 -- latency and launches are all there is
        dict(name="step_tiny_f32", kind="step", net="tiny", preact=False, dtype="f32", hw=16, classes=10, batch=4, S=1, lr=0.1),
        # the repository's headline workload: one of four CIFAR-shaped sub-ResNets, batch 128, fp32
        dict(name="step_cifar_sub_f32", kind="step", net="cifar", preact=False, dtype="f32", hw=32, classes=10, batch=128, S=4, lr=0.01),
        # the paper's preferred pre-activation blocks, 100 classes, on the ragged last batch of an epoch
        dict(name="step_cifar_preact_ragged_f32", kind="step", net="cifar", preact=True, dtype="f32", hw=32, classes=100, batch=77, S=4, lr=0.01),
        # the full model (S = 1), fp32: the largest training call
        dict(name="step_cifar_full_f32", kind="step", net="cifar", preact=False, dtype="f32", hw=32, classes=10, batch=128, S=1, lr=0.01),
        # the same with bf16 storage and matrix operands
        dict(name="step_cifar_full_bf16", kind="step", net="cifar", preact=False, dtype="bf16", hw=32, classes=10, batch=128, S=1, lr=0.001),
        # an ImageNet-shaped bottleneck sub-ResNet of S = 2, batch 64, bf16: the memory-heavy training call
        dict(name="step_imagenet_sub_bf16", kind="step", net="imagenet", preact=False, dtype="bf16", hw=224, classes=1000, batch=64, S=2, lr=0.001),
        # evaluation of the reassembled model between rounds, one test batch, branches scaled by 1/S
        dict(name="predict_cifar_f32", kind="predict", net="cifar", preact=False, dtype="f32", hw=32, classes=10, batch=128, S=4),
        # one image through the bottleneck model: a serving call, bound by latency
        dict(name="predict_one_imagenet_bf16", kind="predict", net="imagenet", preact=False, dtype="bf16", hw=224, classes=1000, batch=1, S=2),
        # end of a round with four workers, fp32 parameters
        dict(name="aggregate_cifar", kind="exchange", net="cifar", preact=False, hw=32, classes=100, S=4, bits=0),
        # the same with every communicated parameter as an 8-bit code, in both directions
        dict(name="exchange_cifar_8bit", kind="exchange", net="cifar", preact=False, hw=32, classes=100, S=4, bits=8),
        # the layer most of the CIFAR-shaped model's time goes to, on its own
        dict(name="conv3x3_f32", kind="conv", dtype="f32", n=128, h=8, w=8, c=256, k=256, r=3, stride=1),
        # a bottleneck's widening 1x1 layer in bf16, odd batch: more memory than arithmetic
        dict(name="conv1x1_bf16", kind="conv", dtype="bf16", n=61, h=14, w=14, c=256, k=1024, r=1, stride=1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "predict", "predict", "exchange", "conv", "conv"])
    if kind in ("step", "predict"):
        net = rng.choice(["tiny", "cifar", "cifar", "imagenet"])
        if net == "tiny":
            c = dict(hw=rng.choice([8, 12, 16, 20, 32]), classes=rng.randint(2, 40), batch=_log_int(rng, 1, 64), S=1)
        elif net == "cifar":
            c = dict(hw=32, classes=rng.choice([10, 100]), batch=_log_int(rng, 1, 128), S=rng.choice([1, 2, 4, 8]))
        else:
            c = dict(hw=rng.choice([96, 128, 160, 192, 224]), classes=rng.choice([100, 1000]), batch=_log_int(rng, 1, 64), S=rng.choice([2, 4]))
        # fp32 for either; bf16 as the larger networks are run in it
        c.update(kind=kind, net=net, preact=net == "cifar" and rng.random() < 0.3,
                 dtype="f32" if net == "tiny" else rng.choice(["f32", "bf16"]) if net == "cifar" else "bf16")
        if kind == "step":
            # training batches; the step sizes are those of a learning-rate schedule after its decays
            c["batch"] = max(c["batch"], {"tiny": 1, "cifar": 16, "imagenet": 8}[net])
            c["lr"] = 0.1 if net == "tiny" else 0.001 if c["dtype"] == "bf16" else 0.01
        return c
    if kind == "exchange":
        net = rng.choice(["tiny", "cifar", "imagenet"])
        return dict(kind=kind, net=net, preact=False, hw=32 if net != "imagenet" else 224, classes=rng.choice([10, 37, 100]),
                    S=rng.choice([1, 2, 3, 4, 8] if net != "tiny" else [1]), bits=rng.choice([0, 0, 4, 5, 8]))
    dtype, r, stride = rng.choice(["f32", "bf16"]), rng.choice([1, 3, 3]), rng.choice([1, 1, 1, 2])
    h = rng.choice([4, 7, 8, 14, 16, 28, 32, 56] if stride == 1 else [8, 14, 16, 28, 32, 56])
    c = 16 * _log_int(rng, 1, 32)
    k = rng.choice([c, c, 16 * _log_int(rng, 1, 32)])
    # at most 128 images, at most 40 GFLOP forward and 64 M elements a tensor
    most = min(128, int(40e9 * stride * stride / (2.0 * h * h * r * r * c * k)), (64 << 20) // (h * h * max(c, k)))
    return dict(kind=kind, dtype=dtype, n=_log_int(rng, 1, max(2, most)), h=h, w=h, c=c, k=k, r=r, stride=stride)


# ---- networks ---------------------------------------------------------------------------------------------------
def _model(case):
    net = _NETS[case["net"]]
    # pre-activation networks start with the bare 3x3 stem
    return dict(block_kind=net["block_kind"] + (2 if case["preact"] else 0), stem_kind=net["stem_kind"], in_c=3,
                in_h=case["hw"], in_w=case["hw"], widths=list(net["widths"]), blocks=list(net["blocks"]), num_classes=case["classes"],
                compute_dtype=1 if case.get("dtype") == "bf16" else 0, bn_eps=1e-5, bn_momentum=0.1)


def _blocks_of(case, model):
    """Block list of the network a call runs: sub-ResNet 0 of the partition for a step, all blocks otherwise."""
    if case["kind"] == "step" and case["S"] > 1:
        return R.partition(model, case["S"], 0, 1, 0)[0][0]
    return list(range(R.num_blocks(model)))


def _conv_table(model, blocks):
    """(block, layer, H_out, W_out, C, K, R) of every convolution, stem first, with its shortcut as layer 3."""
    bott = model["block_kind"] in (1, 3)
    exp = 4 if bott else 1
    h, w = model["in_h"], model["in_w"]
    rows = []
    if model["stem_kind"] == 1:
        h, w = (h + 1) // 2, (w + 1) // 2
    rows.append((-1, 0, h, w, model["in_c"], model["widths"][0], 7 if model["stem_kind"] else 3))
    if model["stem_kind"] == 1:
        h, w = (h + 1) // 2, (w + 1) // 2
    c, b = model["widths"][0], 0
    for si, (wd, nb) in enumerate(zip(model["widths"], model["blocks"])):
        for bi in range(nb):
            st = 2 if (si > 0 and bi == 0) else 1
            ho, wo = h // st, w // st
            if b in blocks:
                if bott:
                    rows += [(b, 0, h, w, c, wd, 1), (b, 1, ho, wo, wd, wd, 3), (b, 2, ho, wo, wd, wd * exp, 1)]
                else:
                    rows += [(b, 0, ho, wo, c, wd, 3), (b, 1, ho, wo, wd, wd * exp, 3)]
                if bi == 0 and (st != 1 or c != wd * exp):
                    rows.append((b, 3, ho, wo, c, wd * exp, 1))
            h, w, c, b = ho, wo, wd * exp, b + 1
    return rows


class _Flat:
    """One device buffer holding a list of block buffers (views of it, each at a multiple of 256 bytes)."""

    def __init__(self, counts, dtype, make=torch.zeros):
        size = torch.empty(0, dtype=dtype).element_size()
        at, total = [], 0
        for n in counts:
            at.append(total)
            total += (n * size + 255) // 256 * 256 // size
        self.all = make(total, dtype=dtype, device="cuda")
        self.views = [self.all[o:o + n] for o, n in zip(at, counts)]


def _fill_block(model, key, buf, gen, nb, trained):
    """Weights of one block in the library's layout; `trained` = BN parameters and running statistics as after training
    (the variance a convolution of unit-variance inputs with these filters has), otherwise as at the start of it."""
    std = {}
    for t in R.block_layout(model, key):
        v = buf[t["offset"]:t["offset"] + t["count"]]
        kind, layer, dims = t["kind"], t["layer"], t["dims"]
        if kind == 0:
            v.normal_(0.0, math.sqrt(2.0 / (dims[0] * dims[1] * dims[2])), generator=gen)
            std[layer] = math.sqrt(dims[3] / dims[0]) * (math.sqrt(2.0) if layer in (0, 3) else 1.0)
        elif kind == 1:
            v.fill_(1.0)
            if trained:
                v.add_(torch.randn(v.shape, generator=gen, device="cuda"), alpha=0.1)
        elif kind == 2 and trained:
            v.normal_(0.0, 0.1, generator=gen)
        elif kind == 3 and trained:
            v.normal_(0.0, 0.1 * std.get(layer, 1.0), generator=gen)
        elif kind == 4:
            v.fill_(1.0)
            if trained:
                v.uniform_(0.8, 1.2, generator=gen).mul_(std.get(layer, 1.0) ** 2)
        elif kind in (5, 6):
            fan_in = next(i["dims"][1] for i in R.block_layout(model, nb) if i["kind"] == 5)
            v.uniform_(-1.0 / math.sqrt(fan_in), 1.0 / math.sqrt(fan_in), generator=gen)


def _params(model, keys, gen, trained=False):
    nb = R.num_blocks(model)
    flat = _Flat([R.block_param_count(model, k)[0] for k in keys], torch.float32)
    for k, v in zip(keys, flat.views):
        _fill_block(model, k, v, gen, nb, trained)
    return flat


# ---- prepare / run ----------------------------------------------------------------------------------------------
def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return {"step": _prepare_step, "predict": _prepare_predict, "exchange": _prepare_exchange, "conv": _prepare_conv}[case["kind"]](case, gen)


def run(state):
    return {"step": _run_step, "predict": _run_predict, "exchange": _run_exchange, "conv": _run_conv}[state["case"]["kind"]](state)


def _prepare_step(case, gen):
    model = _model(case)
    blocks = _blocks_of(case, model)
    keys = [-1] + blocks + [R.num_blocks(model)]
    n = case["batch"]
    return dict(case=case, model=model, blocks=blocks, params=_params(model, keys, gen),
                momentum=_Flat([R.block_param_count(model, k)[1] for k in keys], torch.float32),
                x=torch.randn(n, 3, case["hw"], case["hw"], generator=gen, device="cuda"),
                labels=torch.randint(0, case["classes"], (n,), generator=gen, device="cuda", dtype=torch.int32),
                workspace=torch.empty(R.workspace_bytes(model, blocks, n), dtype=torch.uint8, device="cuda"),
                loss=torch.zeros(1, device="cuda"))


def _run_step(s):
    R.local_step(s["model"], s["blocks"], s["params"].views, s["momentum"].views, None, s["x"], s["labels"], s["case"]["lr"], 0.9,
                 5e-4, s["workspace"], s["loss"])
    out = {"loss": s["loss"], "params": s["params"].all}
    if s["case"]["net"] == "tiny":
        # momentum = the gradients.  Deep networks return the updated parameters only: a ReLU decision of a value that is zero
        # to rounding falls either way, and single gradients of the layers below move by their own size (bf16: all of them do)
        out["momentum"] = s["momentum"].all
    return out


def _prepare_predict(case, gen):
    model = _model(case)
    blocks = _blocks_of(case, model)
    first, n = set(), 0
    for nb in model["blocks"]:
        first.add(n)
        n += nb
    return dict(case=case, model=model, blocks=blocks, params=_params(model, [-1] + blocks + [len(blocks)], gen, trained=True),
                scale=[1.0 if b in first else 1.0 / case["S"] for b in blocks],
                x=torch.randn(case["batch"], 3, case["hw"], case["hw"], generator=gen, device="cuda"),
                workspace=torch.empty(R.forward_workspace_bytes(model, blocks, case["batch"]), dtype=torch.uint8, device="cuda"),
                logits=torch.empty(case["batch"], case["classes"], device="cuda"))


def _run_predict(s):
    R.forward(s["model"], s["blocks"], s["params"].views, s["x"], s["logits"], s["workspace"], s["scale"])
    return {"logits": s["logits"]}


def _prepare_exchange(case, gen):
    model = _model(case)
    nb = R.num_blocks(model)
    subs = R.partition(model, case["S"], 0, 1, 0)[0]
    keys = [-1] + list(range(nb)) + [nb]
    glob = _params(model, keys, gen, trained=True)
    workers = []
    for sub in subs:   # every worker's copy after its local steps: the global parameters, moved a little
        f = _Flat([R.block_param_count(model, k)[0] for k in [-1] + list(sub) + [nb]], torch.float32)
        for k, v in zip([-1] + list(sub) + [nb], f.views):
            v.copy_(glob.views[k + 1])
        f.all.add_(torch.randn(f.all.shape, generator=gen, device="cuda"), alpha=0.01)
        workers.append(f)
    s = dict(case=case, model=model, subs=subs, keys=keys, glob=glob, workers=workers)
    if case["bits"]:
        def compressed(ks):
            sizes = [R.compressed_block_size(model, k, case["bits"]) for k in ks]
            ranges = _Flat([4 * nt for _, nt in sizes], torch.int32)
            return _Flat([n for n, _ in sizes], torch.uint8), ranges
        s["sub_keys"] = [[-1] + list(sub) + [nb] for sub in subs]
        s["up"] = [compressed(ks) for ks in s["sub_keys"]]
        s["down"] = compressed(keys)
        s["received"] = [_Flat([v.numel() for v in f.views], torch.float32) for f in workers]
    return s


def _run_exchange(s):
    model, bits = s["model"], s["case"]["bits"]
    if not bits:
        R.aggregate(model, s["subs"], [f.views for f in s["workers"]], s["glob"].views)
        return {"glob": s["glob"].all}
    for ks, f, (codes, ranges) in zip(s["sub_keys"], s["workers"], s["up"]):
        R.compress_blocks(model, ks, bits, f.views, codes.views, ranges.views)
    R.aggregate_compressed(model, s["subs"], bits, [c.views for c, _ in s["up"]], [r.views for _, r in s["up"]], s["glob"].views)
    codes, ranges = s["down"]
    R.compress_blocks(model, s["keys"], bits, s["glob"].views, codes.views, ranges.views)
    for ks, f in zip(s["sub_keys"], s["received"]):
        R.decompress_blocks(model, ks, bits, [codes.views[k + 1] for k in ks], [ranges.views[k + 1] for k in ks], f.views)
    return {"glob": s["glob"].all, "up": [c.all for c, _ in s["up"]], "down": codes.all, "received": [f.all for f in s["received"]]}


def _prepare_conv(case, gen):
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    pad = case["r"] // 2
    p, q = (case["h"] + 2 * pad - case["r"]) // case["stride"] + 1, (case["w"] + 2 * pad - case["r"]) // case["stride"] + 1
    w = torch.randn(case["k"], case["r"], case["r"], case["c"], generator=gen, device="cuda") * math.sqrt(2.0 / (case["k"] * case["r"] ** 2))
    return dict(case=case, pad=pad, w=w.to(dt),
                x=torch.randn(case["n"], case["h"], case["w"], case["c"], generator=gen, device="cuda").relu_().to(dt),   # behind a ReLU
                dy=torch.randn(case["n"], p, q, case["k"], generator=gen, device="cuda").mul_(1e-3).to(dt))


def _run_conv(s):
    st, pad = s["case"]["stride"], s["pad"]
    return {"y": R.conv2d_forward(s["x"], s["w"], st, pad),
            "dx": R.conv2d_dgrad(s["dy"], s["w"], tuple(s["x"].shape), st, pad),
            "dw": R.conv2d_wgrad(s["dy"], s["x"], tuple(s["w"].shape), st, pad)}


# ---- what a pass cannot do without, and how close two correct results are ----------------------------------------
def work(case):
    if case["kind"] == "conv":
        pad, es = case["r"] // 2, 2 if case["dtype"] == "bf16" else 4
        p, q = (case["h"] + 2 * pad - case["r"]) // case["stride"] + 1, (case["w"] + 2 * pad - case["r"]) // case["stride"] + 1
        x, y, w = case["n"] * case["h"] * case["w"] * case["c"], case["n"] * p * q * case["k"], case["k"] * case["c"] * case["r"] ** 2
        # forward reads x, w and writes y; the gradients read dy, w, x and write dx, dw
        return dict(bytes=es * (2.0 * x + 2.0 * y + w) + 4.0 * w, flops=3 * 2.0 * case["n"] * p * q * case["k"] * case["c"] * case["r"] ** 2)
    model = _model(case)
    nb = R.num_blocks(model)
    if case["kind"] == "exchange":
        subs = R.partition(model, case["S"], 0, 1, 0)[0]
        size = [R.block_param_count(model, k)[0] for k in range(-1, nb + 1)]
        sent = sum(size[0] + size[-1] + sum(size[b + 1] for b in sub) for sub in subs)
        if not case["bits"]:
            return dict(bytes=4.0 * (sent + sum(size)), flops=0.0)
        code = 1.0 if case["bits"] > 4 else 0.5
        # workers read fp32 and write codes; the server reads codes, writes fp32 and codes; workers read codes, write fp32
        return dict(bytes=sent * (4 + code) + sent * code + sum(size) * (4 + code) + sent * (code + 4), flops=0.0)
    blocks = _blocks_of(case, model)
    conv = sum(2.0 * case["batch"] * h * w * c * k * r * r for _, _, h, w, c, k, r in _conv_table(model, set(blocks)))
    stem = 2.0 * case["batch"] * math.prod(_conv_table(model, set(blocks))[0][2:6]) * _conv_table(model, set(blocks))[0][6] ** 2
    image = 4.0 * case["batch"] * 3 * case["hw"] ** 2
    params = sum(R.block_param_count(model, k)[0] for k in [-1] + blocks + [nb])
    if case["kind"] == "predict":
        return dict(bytes=4.0 * params + image + 4.0 * case["batch"] * case["classes"], flops=conv)
    # parameters and momentum read and written; the stem has no data gradient
    return dict(bytes=16.0 * params + image, flops=3 * conv - stem)


def tolerance(case):
    """Measured: each path against itself with its input moved by half an fp32 ulp, and with the sums of the BN backward taken
    in the other of the library's two orders; a single convolution against float64.  About four times the largest seen."""
    bf16 = case.get("dtype") == "bf16"
    if case["kind"] == "exchange":
        return "exact"   # order and rounding of every sum, division and code are part of the interface
    if case["kind"] == "conv":
        # fp32: 8e-7 / 6e-6 over up to 4608 terms.  bf16: the rounding of the output itself (1.7e-3 / one ulp)
        return {"rel": 4e-3, "max": 1.6e-2} if bf16 else {"rel": 5e-6, "max": 5e-5}
    if case["kind"] == "predict":
        # up to 66 layers: 7e-7 in fp32; in bf16 1.5e-3 / 1.3e-2 (stored activations move across rounding boundaries)
        return {"rel": 1e-2, "max": 0.1} if bf16 else {"rel": 1e-5, "max": 1e-4}
    if case["net"] == "tiny":
        return {"rel": 1e-5, "max": 1e-4}
    # Deep training steps flip ReLU decisions of values that are zero to rounding, and a second step amplifies it: after two
    # steps the updated parameters differ by 2e-4 (33 blocks, batch 128) to 1e-3 (batch 8), single ones by a quarter of the
    # RMS; in bf16 by up to 3.4e-3 with the loss by 3.8e-3
    return {"rel": 1.5e-2, "max": 0.5} if bf16 else {"rel": 4e-3, "max": 0.5}

"""Workloads on which the local-update step is measured.

A case describes a network, its local-training scheme and one minibatch; one pass is one call of
`LocalTrainer.step` (or of `LocalTrainer.eval` where the case says so) on device buffers that the
caller keeps, as a training program makes it.
"""
import math

import paper_2012_03837_amd as lp
import lp_inputs as LI
from lp_inputs import configs as CF

MLP = dict(family="mlp", layers=4, in_dim=64, width=256, hidden=256, classes=10, batch=128, scheme="greedy", chunk=1,
           combine="sum", opt="sgd", pass_="step", schedule="sync")
RESNET = dict(family="resnet", stages=4, channels=64, image=32, image_channels=3, classes=10, batch=256, blocks=2,
              head="pool_linear_ce", scheme="greedy", chunk=1, combine="sum", opt="sgdm", pass_="step", schedule="sync")
DECODER = dict(family="decoder", layers=12, width=768, heads=12, hidden=3072, seq=1024, batch=8, vocab=32000, act="gelu",
               scheme="greedy", chunk=1, combine="sum", opt="adam", pass_="step", schedule="sync")


def listed():
    return [
        # The residual MLP of the paper's block-size study, one block per layer, fp32: about a hundred small launches,
        # so latency and launches are what a user waits for.
        dict(MLP, name="mlp_greedy"),
        # A wider MLP at sizes that no tile divides, overlapping windows averaged (the paper's combination), Adam.
        dict(MLP, name="mlp_overlap_ragged", layers=6, in_dim=100, width=520, hidden=1000, batch=333, scheme="overlap",
             combine="mean", opt="adam"),
        # The CIFAR-shaped four-stage residual CNN, one block per stage, bf16: the vision workload.
        dict(RESNET, name="resnet_greedy"),
        # Small single-channel images in a narrow network with the paper's normalised auxiliary head and a short batch:
        # odd feature maps (28, 14, 7), channel counts off the tile sizes, overlapping windows.
        dict(RESNET, name="resnet_ragged", stages=3, channels=24, image=28, image_channels=1, batch=50, blocks=1,
             head="bn_pool_linear_ce", scheme="overlap"),
        # A decoder of test size: ragged sequence and vocabulary, every launch short.
        dict(DECODER, name="decoder_tiny", layers=3, width=128, heads=2, hidden=320, seq=200, batch=3, vocab=1000),
        # The paper's small transformer (eight heads of 16, width 128, 8k vocabulary): heads below 64 wide.
        dict(DECODER, name="decoder_small_heads", layers=4, width=128, heads=8, hidden=256, seq=128, batch=64, vocab=8000),
        # The twelve-layer decoder, one block per layer: a vocabulary head behind every layer.
        dict(DECODER, name="decoder_greedy"),
        # The same with windows of two layers, contributions summed.
        dict(DECODER, name="decoder_overlap", scheme="overlap"),
        # The largest configuration: 24 layers in six chunks of four.
        dict(DECODER, name="decoder_chunk", layers=24, width=1024, heads=16, hidden=4096, seq=2048, batch=4, scheme="chunk",
             chunk=4),
        # Ordinary backpropagation (one head, full window) at odd sizes: a vocabulary that is not a multiple of 8, an odd
        # sequence length, ReLU.
        dict(DECODER, name="decoder_backprop_ragged", layers=6, width=448, heads=7, hidden=1200, seq=511, batch=5,
             vocab=10003, act="relu", scheme="backprop"),
        # The pipelined schedule (blocks work on each other's previous outputs) at a middling size.
        dict(DECODER, name="decoder_pipelined", layers=8, width=512, heads=8, hidden=2048, seq=256, batch=8, vocab=16000,
             scheme="chunk", chunk=2, schedule="pipelined"),
        # Validation: the forward pass and every head's loss of the twelve-layer decoder.
        dict(DECODER, name="decoder_eval", pass_="eval"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _scheme(rng, layers):
    kind = rng.choice(["greedy", "overlap", "chunk", "backprop"])
    return dict(scheme=kind, chunk=rng.randint(2, max(2, layers // 2)) if kind == "chunk" else 1)


def draw(rng):
    most = max(work(c)["flops"] for c in listed())
    while True:
        family = rng.choice(["mlp", "resnet", "decoder", "decoder"])
        if family == "mlp":
            n = rng.randint(2, 8)
            c = dict(MLP, layers=n, in_dim=_log_int(rng, 16, 512), width=_log_int(rng, 64, 1024),
                     hidden=_log_int(rng, 64, 1024), batch=_log_int(rng, 16, 1024), classes=rng.choice([2, 10, 100]),
                     combine=rng.choice(["sum", "mean"]), opt=rng.choice(["sgd", "sgdm", "adam"]), **_scheme(rng, n))
        elif family == "resnet":
            n = rng.randint(2, 4)
            s = _scheme(rng, n)
            if s["scheme"] == "chunk":
                s["chunk"] = 2
            c = dict(RESNET, stages=n, channels=rng.choice([16, 24, 32, 40, 48, 64, 64, 96]), image=rng.choice([16, 24, 32, 40]),
                     image_channels=rng.choice([1, 3]), batch=_log_int(rng, 8, 256), blocks=rng.randint(1, 2),
                     head=rng.choice(["pool_linear_ce", "bn_pool_linear_ce"]), classes=rng.choice([10, 100]), **s)
        else:
            n = _log_int(rng, 2, 24)
            heads = _log_int(rng, 2, 16)
            size = rng.choice([64, 64, 64, 32, 16])
            seq = _log_int(rng, 64, 2048)
            batch = _log_int(rng, 1, max(1, 8192 // seq))
            if size != 64:
                seq = min(seq, 512)
            vocab = _log_int(rng, 500, 32000)
            if rng.random() < 0.3:            # any vocabulary; up to 2048 tokens
                n, batch = min(n, 8), max(1, min(batch, 2048 // seq))
            else:
                vocab = (vocab + 7) // 8 * 8
            c = dict(DECODER, layers=n, heads=heads, width=heads * size, hidden=heads * size * rng.choice([2, 3, 4]),
                     seq=seq, batch=batch, vocab=vocab, act=rng.choice(["gelu", "relu"]),
                     pass_="eval" if rng.random() < 0.15 else "step", **_scheme(rng, n))
            if c["scheme"] in ("greedy", "chunk") and c["pass_"] == "step" and rng.random() < 0.25:
                c["schedule"] = "pipelined"
        if 1e7 < work(c)["flops"] <= most:
            return c


def config(case, seed=0):
    opt = {"sgd": CF.OptCfg("sgd", lr=0.1), "sgdm": CF.OptCfg("sgdm", lr=0.1, momentum=0.9),
           "adam": CF.OptCfg("adam", lr=1e-3)}[case["opt"]]
    common = dict(scheme=case["scheme"], chunk=case["chunk"], combine=case["combine"], opt=opt, batch=case["batch"], seed=seed)
    if case["family"] == "mlp":
        return CF.mlp_config("mlp", n_layers=case["layers"], in_dim=case["in_dim"], width=case["width"],
                             hidden=case["hidden"], n_classes=case["classes"], **common)
    if case["family"] == "resnet":
        return CF.resnet_config("resnet", channels=tuple(case["channels"] << i for i in range(case["stages"])),
                                in_hw=case["image"], in_ch=case["image_channels"], n_classes=case["classes"],
                                n_basic_blocks=case["blocks"], head=case["head"], **common)
    return CF.decoder_config("decoder", n_layers=case["layers"], width=case["width"], n_heads=case["heads"],
                             hidden=case["hidden"], seq_len=case["seq"], vocab=case["vocab"], act=case["act"], **common)


def prepare(case, seed):
    """A trainer with weights initialised from the seed, a minibatch on the device, and views of what a step updates."""
    cfg = config(case, seed)
    tr = lp.LocalTrainer(cfg, n_streams=lp.default_side_streams(cfg), schedule=case["schedule"])
    x, y = LI.make_batch(cfg, seed)
    xd, yd = tr.stage(x, y)
    out = {"losses": tr.losses}
    if case["pass_"] == "step":
        import torch
        # parameters are stored one after another, each on a 64-element boundary: fp32 weights first in `params`,
        # the optimizer's moments in `state` in the same order
        n = sum((math.prod(s) + 63) // 64 * 64 for s in LI.param_shapes(cfg).values())
        out["weights"] = tr.params[:4 * n].view(torch.float32)
        # A ResNet's momentum is left out: after a step it is the change of the weights over the learning rate, and by
        # itself it is ill conditioned (see `tolerance`).  Its running batch statistics follow the momentum in `state`.
        if case["opt"] != "sgd" and case["family"] != "resnet":
            out["m"] = tr.state[:4 * n].view(torch.float32)
        if case["opt"] == "adam":
            out["v"] = tr.state[4 * n:8 * n].view(torch.float32)
        if case["family"] == "resnet":
            running, at = tr.state[4 * n:].view(torch.float32), 0
            out["running"] = []
            for name, (channels,) in ((k, s) for k, s in LI.param_shapes(cfg).items() if len(s) == 1):
                if name.endswith(".g") and name.split(".")[-2].startswith("bn"):
                    out["running"].append(running[at:at + 2 * channels])
                    at += 2 * ((channels + 63) // 64 * 64)
    return {"trainer": tr, "x": xd, "y": yd, "step": case["pass_"] == "step", "out": out}


def run(state):
    tr = state["trainer"]
    if state["step"]:
        tr.step(state["x"], state["y"])
    else:
        tr.eval(state["x"], state["y"])
    return state["out"]


def _layer_flops(l, batch):
    """(dense products, attention) of one forward pass."""
    if l.kind == "resmlp":
        return 2.0 * batch * (2 * l.width * l.hidden + (l.in_dim * l.width if l.in_dim != l.width else 0)), 0.0
    if l.kind == "decoder":
        t = batch * l.seq_len
        return 2.0 * t * l.width * (4 * l.width + 2 * l.hidden), 2.0 * t * l.seq_len * l.width
    hw = (l.in_hw // l.stride) ** 2
    f = 2.0 * batch * l.in_hw ** 2 * l.out_ch * 9 * l.in_ch if l.has_stem else 0.0
    for b in range(l.n_basic_blocks):
        cin = l.in_ch if b == 0 and not l.has_stem else l.out_ch
        f += 2.0 * batch * hw * l.out_ch * 9 * (cin + l.out_ch)
        if b == 0 and not l.has_stem and (l.stride != 1 or cin != l.out_ch):
            f += 2.0 * batch * hw * l.out_ch * cin
    return f, 0.0


def work(case):
    """Products: each layer forward once, its input gradient once per head whose window holds it and is not the window's
    first layer, its weight gradient once; each head forward, and both its gradients.  Bytes: the minibatch, and the
    weights and optimizer state of a step read and written once (with a bf16 working copy written in bf16 networks)."""
    cfg = config(case)
    B, step = cfg.batch, case["pass_"] == "step"
    flops = sum(sum(_layer_flops(l, B)) for l in cfg.layers)
    covered = set()
    for h, (s, e) in zip(cfg.heads, LI.head_windows(cfg)):
        l = cfg.layers[e - 1]
        flops += (3 if step else 1) * 2.0 * B * (l.seq_len if l.kind == "decoder" else 1) * h.in_dim * h.n_classes
        if step:
            for i in range(s, e):
                dense, attn = _layer_flops(cfg.layers[i], B)
                if l.kind == "decoder":
                    # every product but the one that leads out of the window, and attention's five instead of two
                    first = 2.0 * B * l.seq_len * l.width * 3 * l.width if i == s else 0.0
                    flops += dense - first + 2.5 * attn
                elif l.kind == "resmlp":
                    flops += dense / 2 if i == s else dense
                else:
                    lay = cfg.layers[i]
                    hw = (lay.in_hw // lay.stride) ** 2
                    lead = 0.0
                    if i == s:
                        lead = (2.0 * B * lay.in_hw ** 2 * lay.out_ch * 9 * lay.in_ch if lay.has_stem
                                else 2.0 * B * hw * lay.out_ch * 10 * lay.in_ch)
                    flops += dense - lead
                covered.add(i)
    flops += sum(_layer_flops(cfg.layers[i], B)[0] for i in covered)
    n = 0
    for name, shape in LI.param_shapes(cfg).items():
        if not step or name[0] == "H" or int(name.split(".")[0][1:]) - 1 in covered:
            n += math.prod(shape)
    l0 = cfg.layers[0]
    if l0.kind == "decoder":
        data = 8.0 * B * l0.seq_len
    elif l0.kind == "resmlp":
        data = 4.0 * B * (l0.in_dim + 1)
    else:
        data = B * (2.0 * l0.in_hw ** 2 * l0.in_ch + 4)
    low = cfg.dtype == "bf16"
    if step:
        per = {"sgd": 8, "sgdm": 16, "adam": 24}[case["opt"]] + (2 if low else 0)
    else:
        per = 2 if low else 4
    return {"bytes": data + per * n + 4.0 * len(cfg.heads), "flops": flops}


def tolerance(case):
    """Measured after one and two steps, against another order of every sum (other kernels for the same products,
    convolutions and attention) or against float64, over the listed and some forty drawn cases.

    Adam divides the gradient by its own magnitude: where a gradient is rounding noise, so is the sign of a whole update,
    and the largest difference is that of such elements (twice the learning rate against weights of about 0.02).
    fp32 MLP: SGD weights 4e-7 (max 2e-5) from float64; Adam's moments 4e-4 (max 0.07).
    bf16 decoder: 1e-4 to 9e-3 (max 0.16, moments up to 0.9).
    bf16 ResNet: a pre-activation that rounds to the other side of zero flips a ReLU, and normalisation spreads it over
    the batch: weights and running statistics 1e-5 to 6e-3 (max 0.1), momentum itself 2e-3 to 0.3."""
    if case["family"] == "mlp":
        return {"rel": 2e-3, "max": 0.3} if case["opt"] == "adam" else {"rel": 1e-5, "max": 1e-3}
    if case["family"] == "resnet":
        return {"rel": 0.02, "max": 0.4}
    return {"rel": 0.02, "max": 0.9}

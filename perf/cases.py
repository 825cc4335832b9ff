"""What the optimizer step is timed on: calls through the public entry points, with the sizes of this repository's own
workloads and, between and around them, generic ones.

Three kinds of call:
  stepper   one ``MuonStepper.step`` (workspace owned by the caller), the way a training loop steps a parameter list
  static    one ``muon_step_static`` (nothing is allocated), the way a captured or allocation-free loop steps a short list
  adamw     one ``muon_adamw_step`` over the parameters that stay off Muon
Shapes are written "ROWSxCOLS*COUNT" separated by blanks; W, G and M have the distributions of training: W ~ N(0, 0.02^2),
G ~ N(0, (1e-3)^2), momentum of the size it settles at, optionally 1 % of the gradient entries multiplied by 100.
"""
from __future__ import annotations

import math

import torch

from paper_2502_16982_amd import binding

DEV = "cuda:0"
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
NS_COEFF = (3.4445, -4.7750, 2.0315)
LR, WD, MU, RMS_SCALE, EPS = 0.02, 0.1, 0.95, 0.2, 1e-7
ADAM = {"lr": 4.2e-4, "weight_decay": 0.1, "beta1": 0.9, "beta2": 0.95, "eps": 1e-8, "step": 100}
STATIC_NS_BYTES = 40 << 20        # Newton-Schulz temporaries that surely fit muon_step_static's 64 MiB


def muon(name, shapes, *, kind="stepper", ns="bf16", buf="bf16", steps=5, nesterov=True, mode=0, rms=False, outliers=False,
         ws_mib=0):
    return {"name": name, "kind": kind, "shapes": shapes, "ns": ns, "buf": buf, "steps": steps, "nesterov": nesterov,
            "mode": mode, "rms": rms, "outliers": outliers, "ws_mib": ws_mib}


def adamw(name, sizes, *, buf="bf16"):
    return {"name": name, "kind": "adamw", "shapes": sizes, "buf": buf}


def listed():
    return [
        # the smallest call: one small fp32 matrix, bound by the number of dependent launches
        muon("single_128x256_f32", "128x256", ns="f32", buf="f32"),
        # accurate arithmetic of a small model on the fp32 path, fp32 master weights
        muon("list_f32", "512x512*4 512x1536*2 1536x512", ns="f32", buf="f32"),
        # an allocation-free step of a short list (a captured loop), update RMS logged
        muon("static_bf16", "256x384*4 384x256*2 512x768 768x512 200x333", kind="static", rms=True),
        # one layer of the width-1024 model: stepped as its gradients arrive, or the share of one of many ranks
        muon("layer_w1024", "1024x1024*4 1024x4096*2 4096x1024"),
        # the whole width-1024 model
        muon("dense12_w1024", " ".join(["1024x1024*4 1024x4096*2 4096x1024"] * 12)),
        # one block of a 4096-wide model, gradients with outliers, update RMS logged
        muon("block_w4096", "4096x4096*4 4096x11008*2 11008x4096", outliers=True, rms=True),
        # one layer of the 66-expert mixture with its attention, in a workspace that holds half of it
        muon("moe_layer_chunked", "2048x1408*132 1408x2048*66 2048x2048*4", ws_mib=2560),
        # odd and ragged sizes, both orientations, fp32 buffers, plain momentum, the "Update Norm" scaling
        muon("ragged_f32buf", "1000x3001 777x777 2049x513 63x4097 4097x130 1500x1111", buf="f32", nesterov=False, mode=2),
        # the accurate arithmetic on one layer: two planes, and three planes with ten iterations on a smaller one
        muon("accurate_x2_layer", "1024x1024*4 1024x4096*2 4096x1024", ns="bf16x2", mode=1),
        muon("accurate_x3_n10", "512x512*4 512x1536*2 1500x500", ns="bf16x3", buf="f32", steps=10),
        # parameters off Muon: embedding, LM head and gains of a width-2048 model; the gains alone
        adamw("adamw_embeddings", "67108864*2 2048*55"),
        adamw("adamw_gains", "1024*25", buf="f32"),
    ]


MAX_FLOPS = 12e12                 # below one mixture layer
MAX_ELEMS = 120_000_000


def draw(rng):
    """One more call of the same ranges: lists of 1 to 100 matrices, sides from 16 to 4096 with odd ones among them."""
    if rng.random() < 0.15:
        sizes = " ".join(str(int(2 ** rng.uniform(6, 24))) for _ in range(rng.randint(1, 40)))
        return {"kind": "adamw", "shapes": sizes, "buf": rng.choice(["bf16", "f32"])}
    ns = rng.choice(["bf16"] * 6 + ["f32"] * 2 + ["bf16x2", "bf16x3"])
    top = {"bf16": 4096, "f32": 1024, "bf16x2": 2048, "bf16x3": 1024}[ns]
    budget = {"bf16": MAX_FLOPS, "f32": 0.2e12, "bf16x2": 3e12, "bf16x3": 1.5e12}[ns]

    def side():
        v = 2 ** rng.uniform(4, math.log2(top))
        grain = rng.choice([1, 1, 8, 64, 128])
        return max(16, min(top, int(round(v / grain)) * grain))

    while True:
        groups = [(side(), side(), int(2 ** rng.uniform(0, 5))) for _ in range(rng.randint(1, 4))]
        steps = rng.choice([5, 5, 5, 10]) if ns != "bf16" else 5
        flops = sum(k * steps * (3 * min(a, b) ** 2 * max(a, b) + min(a, b) ** 3) for a, b, k in groups)
        if flops <= budget and sum(k * a * b for a, b, k in groups) <= MAX_ELEMS:
            break
    case = muon("", " ".join(f"{a}x{b}*{k}" for a, b, k in groups), ns=ns, buf=rng.choice(["bf16", "f32"]), steps=steps,
                nesterov=rng.random() < 0.7, mode=rng.choice([0, 0, 1, 2]), rms=rng.random() < 0.4,
                outliers=rng.random() < 0.2)
    del case["name"]
    planes = {"bf16": 2, "f32": 4, "bf16x2": 4, "bf16x3": 6}[ns]
    pad = lambda v: -(-v // 128) * 128
    temp = sum(k * planes * (3 * pad(a) * pad(b) + 2 * pad(min(a, b)) ** 2) for a, b, k in groups)
    if temp <= STATIC_NS_BYTES and sum(k for _, _, k in groups) <= 64 and rng.random() < 0.5:
        case["kind"] = "static"
    return case


def parse(text):
    out = []
    for item in text.split():
        size, _, count = item.partition("*")
        out += [tuple(int(v) for v in size.split("x"))] * int(count or 1)
    return out


def flat_parts(shapes, dtype):
    """One buffer with room for every shape, each on a 256-byte boundary (how a program keeps its parameters together),
    and the views of it."""
    starts, end = [], 0
    for shape in shapes:
        starts.append(end)
        end += -(-math.prod(shape) // 128) * 128
    flat = torch.zeros(end, dtype=dtype, device=DEV)
    return flat, [flat[s:s + math.prod(shape)].view(shape) for s, shape in zip(starts, shapes)]


def make_inputs(case, seed):
    """Flat buffers [w, g, m] (adamw: [p, g, m, v]) and the tuple of views per parameter, from the seed alone."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed * 7919 + 17)
    dt = DTYPES[case["buf"]]
    shapes = parse(case["shapes"])
    adam = case["kind"] == "adamw"
    parts = [flat_parts(shapes, t) for t in ([dt, dt, torch.float32, torch.float32] if adam else [dt, dt, torch.float32])]

    def normal(shape, std):
        return torch.empty(shape, dtype=torch.float32, device=DEV).normal_(0.0, std, generator=gen)

    tensors = list(zip(*(views for _, views in parts)))
    for shape, views in zip(shapes, tensors):
        views[0].copy_(normal(shape, 0.02))
        g = normal(shape, 1e-3)
        if case.get("outliers"):
            hit = torch.empty(shape, dtype=torch.float32, device=DEV).uniform_(0.0, 1.0, generator=gen) < 0.01
            g = torch.where(hit, g * 100.0, g)
        views[1].copy_(g)
        views[2].copy_(normal(shape, 3e-4 if adam else 3e-3))
        if adam:
            views[3].copy_(normal(shape, 1e-3).square_())
    return [flat for flat, _ in parts], tensors


def hidden_size(shapes):
    return float(max(min(s) for s in shapes))


def prepare(case, seed):
    flats, tensors = make_inputs(case, seed)
    state = {"case": case, "tensors": tensors, "out": [flats[0]] + flats[2:]}
    if case["kind"] == "adamw":
        return state
    shapes = parse(case["shapes"])
    over = dict(lr=LR, weight_decay=WD, momentum=MU, rms_scale=RMS_SCALE, eps=EPS, ns_steps=case["steps"],
                nesterov=int(case["nesterov"]), scale_mode=case["mode"])
    if case["mode"] == 1:
        over["hidden_size"] = hidden_size(shapes)
    state["hp"] = binding.default_hparams(**over)
    state["rms"] = torch.zeros(len(tensors), dtype=torch.float32, device=DEV) if case["rms"] else None
    if case["rms"]:
        state["out"].append(state["rms"])
    if case["kind"] == "static":
        params = binding.param_array(shapes, [binding.dtype_code(w.dtype) for w, _, _ in tensors],
                                     [binding.dtype_code(g.dtype) for _, g, _ in tensors])
        for p, (w, g, m) in zip(params, tensors):
            p.w, p.g, p.m = w.data_ptr(), g.data_ptr(), m.data_ptr()
        state["params"] = params
    else:
        state["stepper"] = binding.MuonStepper(tensors, ns_dtype=case["ns"], max_workspace_bytes=case["ws_mib"] << 20)
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "adamw":
        binding.muon_adamw_step(state["tensors"], stream_ptr=torch.cuda.current_stream().cuda_stream, **ADAM)
    elif case["kind"] == "static":
        rms = state["rms"]
        binding.muon_step_static(state["params"], len(state["tensors"]), binding.NS_DTYPES[case["ns"]], state["hp"],
                                 torch.cuda.current_stream().cuda_stream, 0 if rms is None else rms.data_ptr())
    else:
        state["stepper"].step(state["hp"], update_rms=state["rms"])
    return state["out"]


def work(case):
    """Each buffer once in and, where it is updated, once out; the multiply-adds of Eq. 2 with the two symmetric products
    from one triangle (whatever the number of planes a matrix is kept in)."""
    e = 2 if case["buf"] == "bf16" else 4
    if case["kind"] == "adamw":
        n = sum(s[0] for s in parse(case["shapes"]))
        return {"bytes": n * (3 * e + 16), "flops": n * 16}
    n, flops = 0, 0
    for a, b in parse(case["shapes"]):
        n += a * b
        flops += case["steps"] * (3 * min(a, b) ** 2 * max(a, b) + min(a, b) ** 3)
    return {"bytes": n * (3 * e + 8), "flops": flops}


def tolerance(case):
    """Whole-output bars, four times what is seen: bf16 storage of the weights rounds at 1.7e-3 (2-norm), fp32 at 3e-8; a
    weight carries the error of the Newton-Schulz result (1.0e-2 in bf16 at these sides, 2.5e-5 with two planes, below
    3e-6 otherwise) times the size of the update relative to the weight."""
    stored = 1.7e-3 if case["buf"] == "bf16" else 6e-8
    if case["kind"] == "adamw":
        return {"rel": 4 * max(stored, 2e-7)}
    shapes = parse(case["shapes"])
    widest = max(math.sqrt(hidden_size(shapes) / max(s)) for s in shapes) if case["mode"] == 1 else 1.0
    ratio = LR * RMS_SCALE * max(1.0, widest) / 0.02
    seen = {"bf16": 1.2e-2, "bf16x2": 3e-5, "bf16x3": 3e-6, "f32": 3e-6}[case["ns"]] * ratio / math.hypot(1.0, ratio)
    return {"rel": 4 * math.hypot(stored, seen)}


def exact(case, seed):
    _, tensors = make_inputs(case, seed)
    shapes = parse(case["shapes"])
    adam = case["kind"] == "adamw"
    parts = [flat_parts(shapes, torch.float64) for _ in range(3 if adam else 2)]
    rms = []
    if adam:
        b1, b2, t = ADAM["beta1"], ADAM["beta2"], ADAM["step"]
        for (p, g, m, v), outs in zip(tensors, zip(*(views for _, views in parts))):
            p, g, m, v = p.double(), g.double(), m.double(), v.double()
            m = b1 * m + (1 - b1) * g
            v = b2 * v + (1 - b2) * g * g
            upd = (m / (1 - b1 ** t)) / ((v / (1 - b2 ** t)).sqrt() + ADAM["eps"])
            for out, value in zip(outs, (p - ADAM["lr"] * (upd + ADAM["weight_decay"] * p), m, v)):
                out.copy_(value)
        return [flat for flat, _ in parts]
    a, b, c = NS_COEFF
    hidden = hidden_size(shapes)
    for (w, g, m), outs in zip(tensors, zip(*(views for _, views in parts))):
        w, g, m = w.double(), g.double(), m.double()
        m = MU * m + g
        u = MU * m + g if case["nesterov"] else m
        x = u / (u.norm() + EPS)
        flip = x.shape[0] > x.shape[1]
        x = x.T.contiguous() if flip else x
        for _ in range(case["steps"]):
            gram = x @ x.T
            x = a * x + (b * gram + c * (gram @ gram)) @ x
        o = x.T if flip else x
        r = o.square().mean().sqrt()
        factor = (RMS_SCALE * math.sqrt(max(w.shape)), RMS_SCALE * math.sqrt(hidden), RMS_SCALE / r)[case["mode"]]
        outs[0].copy_(w - LR * (factor * o + WD * w))
        outs[1].copy_(m)
        rms.append(r)
    return [flat for flat, _ in parts] + ([torch.stack(rms)] if case["rms"] else [])

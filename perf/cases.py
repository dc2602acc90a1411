"""The work that the performance of this library is judged by.

A case is a dict of plain values; its "path" names what one pass does:

  codec     encode a boundary tensor, then decode it (sender and receiver of one message)
  stage     a pipeline stage on one microbatch: "forward", "backward" (recomputes the forward) or "train" (both, as a
            peer does for every microbatch); with "coded" the boundary tensors travel as int8 messages
  boundary  both halves of a compression-aware boundary, forward and backward
  head      first and last stage extras: embedding forward and gradient, language-modelling head with its loss
            ("train": loss and gradients, "loss": evaluation, the loss alone)
  lamb      one optimiser step over all parameter tensors of a block

listed() holds the sizes of the repository's benchmark configurations and a few generic ones between them, draw()
gives more of the same ranges.
"""
import math

import torch

import paper_2301_11913_amd as sw

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
ELEMENT_BYTES = {"f32": 4, "bf16": 2}


def stage(name, do, dtype, d, heads, f, batch, seq, layers=1, repeat=1, block="gelu", coded=False, scale_bits=32):
    case = {"path": "stage", "do": do, "dtype": dtype, "d": d, "heads": heads, "f": f, "batch": batch, "seq": seq,
            "layers": layers, "repeat": repeat, "block": block, "coded": coded, "scale_bits": scale_bits}
    return dict(case, name=name) if name else case


def listed():
    return [
        # the message of the smallest configuration: two launches on half a megabyte, all latency
        {"name": "codec_f32_131k", "path": "codec", "dtype": "f32", "n": 4 * 128 * 256, "scale_bits": 32},
        # the message of the largest microbatch (4 sequences of 2048 tokens, d_model 4096): memory bandwidth
        {"name": "codec_bf16_33m", "path": "codec", "dtype": "bf16", "n": 4 * 2048 * 4096, "scale_bits": 32},
        # the fp32 block, the precision that convergence and parity runs use
        stage("stage_f32_d256", "train", "f32", 256, 4, 1024, 4, 128),
        # one sequence through a small stage, forward only: what a request costs when nothing is batched
        stage("forward_bf16_d1024_one_sequence", "forward", "bf16", 1024, 16, 4096, 1, 512),
        # token count that fills no tile (a microbatch of text cut at its own length)
        stage("stage_bf16_d768_ragged", "train", "bf16", 768, 12, 3072, 5, 333),
        # two blocks of d_model 1024, microbatch of 8 sequences of 512
        stage("stage_bf16_d1024_two_blocks", "train", "bf16", 1024, 16, 4096, 8, 512, layers=2),
        # the middle of the width sweep
        stage("stage_bf16_d2048", "train", "bf16", 2048, 16, 8192, 8, 512),
        # the headline: two blocks of d_model 4096 on 4 sequences of 2048 tokens, int8 messages on all four boundaries
        stage("stage_bf16_d4096_coded", "train", "bf16", 4096, 32, 16384, 4, 2048, layers=2, coded=True),
        # the billion-parameter model's stage: one shared rotary + GeGLU block applied 16 times to one sequence
        stage("stage_bf16_d4096_shared16", "train", "bf16", 4096, 32, 16384, 1, 2048, repeat=16, block="rotary_geglu",
              coded=True),
        # linear bottleneck at a compression factor of 2 between two stages
        {"name": "boundary_bottleneck_d4096", "path": "boundary", "kind": "bottleneck", "dtype": "bf16", "d": 4096,
         "d_comp": 2048, "tokens": 8192},
        # GPT-2's vocabulary, padded to whole tiles, on one 2048-token sequence
        {"name": "head_d4096", "path": "head", "do": "train", "dtype": "bf16", "d": 4096, "vocab": 50257,
         "vocab_rows": 50432, "tokens": 2048},
        # the optimiser step of the billion-parameter model's stage, once per global batch
        {"name": "lamb_d4096", "path": "lamb", "dtype": "bf16", "d": 4096, "f": 16384, "block": "rotary_geglu"},
    ]


def log_uniform(rng, low, high):
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


def draw(rng):
    while True:
        path = rng.choices(["codec", "stage", "boundary", "head", "lamb"], [2, 7, 1, 1, 1])[0]
        dtype = "f32" if rng.random() < (0.5 if path == "codec" else 0.25) else "bf16"
        d = rng.choice([256, 512, 768, 1024, 1536, 2048, 3072, 4096])
        f = 4 * d if rng.random() < 0.7 else 64 * rng.randint(d // 64, 4 * d // 64)
        if path == "codec":
            n = log_uniform(rng, 1 << 16, 1 << 25)
            case = {"path": path, "dtype": dtype, "n": n if rng.random() < 0.5 else n // 64 * 64,
                    "scale_bits": rng.choice([32, 16])}
        elif path == "stage":
            tokens = log_uniform(rng, 64, 8192)
            seq = min(log_uniform(rng, 32, 2048), tokens)
            if rng.random() < 0.5:                      # half of the microbatches have padded, half ragged lengths
                seq = max(32, seq // 32 * 32)
            case = stage(None, rng.choices(["train", "forward", "backward"], [6, 3, 1])[0], dtype, d,
                         d // rng.choice([64, 128]), f, max(1, tokens // seq), seq, rng.choice([1, 1, 2]),
                         rng.choice([1, 1, 1, 2, 4]), rng.choice(["gelu", "gelu", "rotary_geglu"]),
                         rng.random() < 0.3, rng.choice([32, 16]))
            # fp32 is for the small configurations
            if dtype == "f32" and (d > 1024 or tokens > 2048 or seq > 1024):
                continue
        elif path == "boundary":
            case = {"path": path, "kind": rng.choice(["bottleneck", "maxout"]), "dtype": dtype, "d": d,
                    "d_comp": d // rng.choice([2, 4]), "tokens": log_uniform(rng, 128, 8192)}
        elif path == "head":
            vocab = log_uniform(rng, 2000, 50257)
            case = {"path": path, "do": rng.choice(["train", "train", "loss"]), "dtype": dtype, "d": d, "vocab": vocab,
                    "vocab_rows": -(-vocab // 256) * 256, "tokens": log_uniform(rng, 128, 2048)}
        else:
            case = {"path": path, "dtype": dtype, "d": d, "f": f, "block": rng.choice(["gelu", "rotary_geglu"])}
        if work(case)["flops"] <= (3e11 if dtype == "f32" else 2e13):
            return case


# ------------------------------------------------------------------------------------------------ inputs
class Random:
    """Tensors on the GPU, all from one seed."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)

    def normal(self, shape, dtype, std, mean=0.0):
        t = torch.randn(shape, generator=self.g, device="cuda", dtype=torch.float32)
        return t.mul_(std).add_(mean).to(dtype)

    def token_ids(self, n, vocab):
        """Log-uniform ranks: frequent ids repeat inside a microbatch, as in text."""
        u = torch.rand(n, generator=self.g, device="cuda", dtype=torch.float64)
        return torch.exp(u * math.log(vocab)).to(torch.int32).clamp_(1, vocab) - 1


def block_shapes(d, f, block):
    f1 = 2 * f if block == "rotary_geglu" else f
    return {"ln1_g": (d,), "ln1_b": (d,), "w_qkv": (3 * d, d), "b_qkv": (3 * d,), "w_o": (d, d), "b_o": (d,),
            "ln2_g": (d,), "ln2_b": (d,), "w_1": (f1, d), "b_1": (f1,), "w_2": (d, f), "b_2": (d,)}


def make_parameters(r, shapes, dtype):
    return {k: r.normal(s, dtype, 0.02, 1.0 if k in ("ln1_g", "ln2_g", "ln_g") else 0.0) for k, s in shapes.items()}


def zeros_for(params):
    return {k: torch.zeros(v.shape, dtype=torch.float32, device="cuda") for k, v in params.items()}


def message(n, scale_bits):
    return (torch.empty(n, dtype=torch.int8, device="cuda"),
            torch.empty(-(-n // 64), dtype=torch.float32 if scale_bits == 32 else torch.int16, device="cuda"))


def encode(x, msg):
    (sw.swarm_codec_encode if msg[1].dtype == torch.float32 else sw.swarm_codec_encode_s16)(x, *msg)


def decode(msg, x):
    (sw.swarm_codec_decode if msg[1].dtype == torch.float32 else sw.swarm_codec_decode_s16)(*msg, x)


def workspace(size):
    return torch.empty(size, dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    r, dt = Random(seed), DTYPES[case["dtype"]]
    s = {"case": case}
    if case["path"] == "codec":
        s["x"] = r.normal((case["n"],), dt, 1.0)
        s["message"] = message(case["n"], case["scale_bits"])
        s["decoded"] = torch.empty_like(s["x"])
    elif case["path"] == "stage":
        d, shape = case["d"], (case["batch"], case["seq"], case["d"])
        s["cfg"] = sw.StageConfig(d, case["heads"], case["f"], case["layers"], case["repeat"], case["batch"], case["seq"],
                                  case["dtype"], 1e-5, case["block"])
        s["params"] = [make_parameters(r, block_shapes(d, case["f"], case["block"]), dt) for _ in range(case["layers"])]
        x = r.normal(shape, dt, 1.0)
        s["x"] = x
        s["y"] = torch.empty_like(x)
        if case["do"] != "forward":
            dy = r.normal(shape, dt, 1.0 if case["dtype"] == "f32" else 1e-2)
            s["dy"], s["dx"] = dy, torch.empty_like(x)
            s["grads"] = [zeros_for(p) for p in s["params"]]
        if case["coded"]:
            # what the neighbouring peers sent, and room for what this peer sends
            n = x.numel()
            s["in_message"], s["out_message"] = message(n, case["scale_bits"]), message(n, case["scale_bits"])
            encode(x, s["in_message"])
            if case["do"] == "backward":
                decode(s["in_message"], x)              # the decoded input that the forward call had left
            if case["do"] != "forward":
                s["in_grad"], s["out_grad"] = message(n, case["scale_bits"]), message(n, case["scale_bits"])
                encode(dy, s["in_grad"])
        size = sw.swarm_stage_coded_workspace_bytes if case["coded"] else sw.swarm_stage_workspace_bytes
        s["workspace"] = workspace(max(size(s["cfg"], False), size(s["cfg"], case["do"] != "forward")))
    elif case["path"] == "boundary":
        T, m, c = case["tokens"], case["d"], case["d_comp"]
        s["cfg"] = sw.BoundaryConfig(m, c, case["kind"], T, case["dtype"])
        comp = {"ln_g": (m,), "ln_b": (m,)}
        if case["kind"] == "bottleneck":
            comp["w_c"] = (c, m)
        s["comp"] = make_parameters(r, comp, dt)
        s["dec"] = make_parameters(r, {"ln_g": (c,), "ln_b": (c,), "w_d": (m, c)}, dt)
        s["comp_grads"], s["dec_grads"] = zeros_for(s["comp"]), zeros_for(s["dec"])
        s["y"] = r.normal((T, m), dt, 1.0)
        s["dx"] = r.normal((T, m), dt, 1.0 if case["dtype"] == "f32" else 1e-2)
        s["z"], s["dz"] = (torch.empty((T, c), dtype=dt, device="cuda") for _ in range(2))
        s["x"], s["dy"] = torch.empty_like(s["y"]), torch.empty_like(s["y"])
        s["workspace"] = workspace(max(sw.swarm_boundary_workspace_bytes(s["cfg"], half, back)
                                       for half in (False, True) for back in (False, True)))
    elif case["path"] == "head":
        T, d, V, rows = case["tokens"], case["d"], case["vocab"], case["vocab_rows"]
        s["cfg"] = sw.HeadConfig(d, V, rows, T, case["dtype"])
        s["table"] = r.normal((rows, d), dt, 0.02)
        s["head"] = make_parameters(r, {"ln_g": (d,), "ln_b": (d,), "w_vocab": (rows, d)}, dt)
        s["table"][V:] = 0
        s["head"]["w_vocab"][V:] = 0
        s["tokens"], s["targets"] = r.token_ids(T, V), r.token_ids(T, V)
        s["x"] = r.normal((T, d), dt, 1.0)
        s["embedded"] = torch.empty_like(s["x"])
        s["loss"] = torch.zeros(1, dtype=torch.float32, device="cuda")
        s["token_loss"] = torch.zeros(T, dtype=torch.float32, device="cuda")
        if case["do"] == "train":
            s["d_embedded"] = r.normal((T, d), dt, 1e-2)
            s["dx"] = torch.empty_like(s["x"])
            s["head_grads"] = zeros_for(s["head"])
            s["table_grad"] = torch.zeros((rows, d), dtype=torch.float32, device="cuda")
        s["workspace"] = workspace(sw.swarm_head_workspace_bytes(s["cfg"], case["do"] == "train"))
    else:
        s["tensors"] = []
        for k, shape in block_shapes(case["d"], case["f"], case["block"]).items():
            w = r.normal(shape, torch.float32, 0.02, 1.0 if k in ("ln1_g", "ln2_g") else 0.0).view(-1)
            s["tensors"].append({"master": w, "param": w.to(dt), "grad": r.normal(w.shape, torch.float32, 1e-3),
                                 "m": r.normal(w.shape, torch.float32, 1e-4),
                                 "v": r.normal(w.shape, torch.float32, 1e-3).square_()})
        s["workspace"] = workspace(max(sw.swarm_lamb_workspace_bytes(t["master"].numel()) for t in s["tensors"]))
    return s


# ------------------------------------------------------------------------------------------------ one pass
def run_stage(s):
    case, ws = s["case"], s["workspace"]
    out = {}
    if case["do"] != "backward":
        if case["coded"]:
            sw.swarm_stage_forward_coded(s["cfg"], s["params"], *s["in_message"], s["x"], *s["out_message"], ws)
            # the next peer's side of the message: a code may move by one step with the rounding of a bf16
            # intermediate, so what is compared is the value that arrives
            decode(s["out_message"], s["y"])
        else:
            sw.swarm_stage_forward(s["cfg"], s["params"], s["x"], s["y"], ws)
        out["y"] = s["y"]
    if case["do"] != "forward":
        if case["coded"]:
            sw.swarm_stage_backward_coded(s["cfg"], s["params"], s["x"], *s["in_grad"], *s["out_grad"], s["grads"], ws)
            decode(s["out_grad"], s["dx"])
        else:
            sw.swarm_stage_backward(s["cfg"], s["params"], s["x"], s["dy"], s["dx"], s["grads"], ws)
        out["dx"], out["grads"] = s["dx"], s["grads"]
    return out


def run_boundary(s):
    cfg, ws = s["cfg"], s["workspace"]
    sw.swarm_compress_forward(cfg, s["comp"], s["y"], s["z"], ws)
    sw.swarm_decompress_forward(cfg, s["dec"], s["z"], s["x"], ws)
    sw.swarm_decompress_backward(cfg, s["dec"], s["z"], s["dx"], s["dz"], s["dec_grads"], ws)
    sw.swarm_compress_backward(cfg, s["comp"], s["y"], s["dz"], s["dy"], s["comp_grads"], ws)
    return {k: s[k] for k in ("z", "x", "dz", "dy", "dec_grads", "comp_grads")}


def run_head(s):
    cfg, ws, V = s["cfg"], s["workspace"], s["case"]["vocab"]
    sw.swarm_embedding_forward(s["tokens"], s["table"], V, s["embedded"])
    out = {k: s[k] for k in ("embedded", "loss", "token_loss")}
    if s["case"]["do"] == "loss":
        sw.swarm_head_loss(cfg, s["head"], s["x"], s["targets"], s["loss"], s["token_loss"], ws)
        return out
    sw.swarm_head_loss_backward(cfg, s["head"], s["x"], s["targets"], s["loss"], s["token_loss"], s["dx"],
                                s["head_grads"], ws)
    sw.swarm_embedding_backward(s["tokens"], s["d_embedded"], V, s["table_grad"])
    return dict(out, dx=s["dx"], head_grads=s["head_grads"], table_grad=s["table_grad"])


def run(state):
    path = state["case"]["path"]
    if path == "codec":
        encode(state["x"], state["message"])
        decode(state["message"], state["decoded"])
        return state["message"], state["decoded"]
    if path == "stage":
        return run_stage(state)
    if path == "boundary":
        return run_boundary(state)
    if path == "head":
        return run_head(state)
    for t in state["tensors"]:
        sw.swarm_lamb_step(t["master"], t["param"], t["grad"], t["m"], t["v"], 100, state["workspace"])
    return [{k: t[k] for k in ("master", "param", "m", "v")} for t in state["tensors"]]


# ------------------------------------------------------------------------------------------------ cost and precision
def work(case):
    """Bytes: every input read once, every output written once (gradients are added to: both).  Flops: the products
    that the interface asks for; a backward call has to recompute the forward, all but its last product."""
    es = ELEMENT_BYTES[case["dtype"]]
    path = case["path"]
    if path == "codec":
        return {"bytes": 2 * case["n"] * (es + 1 + case["scale_bits"] / 8 / 64), "flops": 0}
    if path == "stage":
        d, f, S, B = case["d"], case["f"], case["seq"], case["batch"]
        T, apps = B * S, case["layers"] * case["repeat"]
        up = 2 if case["block"] == "rotary_geglu" else 1
        params = case["layers"] * sum(math.prod(s) for s in block_shapes(d, f, case["block"]).values())
        last = 2 * T * f * d
        products = apps * 2 * T * (4 * d * d + up * d * f + d * f)
        attention = apps * 2 * B * d * S * (S + 1)               # scores and values over the causal half
        forward = products + attention
        backward = forward - last + 2 * products + 2.5 * attention
        tensor = T * d * (1 + case["scale_bits"] / 8 / 64 if case["coded"] else es)
        flops = forward * (case["do"] != "backward") + backward * (case["do"] != "forward")
        count = {"forward": 2, "backward": 3, "train": 4}[case["do"]]
        return {"bytes": params * es + count * tensor + (8 * params if case["do"] != "forward" else 0), "flops": flops}
    if path == "boundary":
        T, m, c = case["tokens"], case["d"], case["d_comp"]
        maps = 2 if case["kind"] == "bottleneck" else 1
        return {"bytes": 4 * T * (m + c) * es + maps * m * c * (es + 8), "flops": 3 * maps * 2 * T * m * c}
    if path == "head":
        T, d, rows = case["tokens"], case["d"], case["vocab_rows"]
        if case["do"] == "loss":
            return {"bytes": (3 * T * d + rows * d) * es, "flops": 2 * T * d * rows}
        return {"bytes": (5 * T * d + rows * d) * es + 8 * rows * d + 8 * min(T, case["vocab"]) * d,
                "flops": 3 * 2 * T * d * rows}
    n = sum(math.prod(s) for s in block_shapes(case["d"], case["f"], case["block"]).values())
    return {"bytes": n * (16 + 12 + es), "flops": 0}


def tolerance(case):
    """Measured: bf16 cases against the same case in fp32 (up to 6e-3 for one or two block applications, 1.2e-2 where
    the result leaves as int8 codes, 3e-2 for sixteen applications), fp32 cases against 64-bit sums (up to 1.6e-6)."""
    if case["path"] == "codec":
        return "exact"
    rel, limits = (1e-5 if case["dtype"] == "f32" else 1e-2), {}
    if case["path"] == "stage":
        if case["dtype"] == "bf16":
            rel = min(3e-2, rel * math.sqrt(case["layers"] * case["repeat"]) + (5e-3 if case["coded"] else 0.0))
        elif case["coded"]:         # a code that moves by one step (0.02 standard deviations), one in ten thousand
            rel, limits = 1e-3, {"max": 0.1}
    elif case["path"] == "boundary" and case["kind"] == "maxout":
        # a window whose two largest features are equal to rounding sends its gradient to either of them
        rel, limits = (1e-3 if case["dtype"] == "f32" else 3e-2), {"max": 0.99}
    return dict(limits, rel=rel)


# ------------------------------------------------------------------------------------------------ the same in 64 bits
def to64(tensors):
    return {k: v.double().requires_grad_() for k, v in tensors.items()}


def norm64(x, g, b):
    return torch.nn.functional.layer_norm(x, x.shape[-1:], g, b, 1e-5)


def block64(x, p, heads, kind):
    """One pre-LayerNorm block, x [batch, seq, d]."""
    B, S, d = x.shape
    qkv = norm64(x, p["ln1_g"], p["ln1_b"]) @ p["w_qkv"].T + p["b_qkv"]
    q, k, v = (t.view(B, S, heads, d // heads).transpose(1, 2) for t in qkv.split(d, -1))
    if kind == "rotary_geglu":
        half = d // heads // 2
        angle = torch.outer(torch.arange(S, device="cuda", dtype=torch.float64),
                            10000.0 ** (-torch.arange(half, device="cuda", dtype=torch.float64) / half))
        cos, sin = angle.cos(), angle.sin()
        q, k = (torch.stack((even * cos - odd * sin, even * sin + odd * cos), -1).flatten(-2)
                for even, odd in ((t[..., ::2], t[..., 1::2]) for t in (q, k)))
    later = torch.ones(S, S, dtype=torch.bool, device="cuda").triu(1)
    scores = (q @ k.transpose(-1, -2) / math.sqrt(d // heads)).masked_fill(later, -math.inf)
    o = (scores.softmax(-1) @ v).transpose(1, 2).reshape(B, S, d)
    h = x + o @ p["w_o"].T + p["b_o"]
    u = norm64(h, p["ln2_g"], p["ln2_b"]) @ p["w_1"].T + p["b_1"]
    if kind == "rotary_geglu":
        gate, up = u.chunk(2, -1)
        u = torch.nn.functional.gelu(gate) * up
    else:
        u = torch.nn.functional.gelu(u)
    return h + u @ p["w_2"].T + p["b_2"]


def through_message64(x, scale_bits):
    """What arrives of x as an int8 message: every 64 values share the scale max|x| / 127."""
    blocks = x.detach().reshape(-1, 64)
    scale = blocks.abs().amax(1, keepdim=True) / 127
    if scale_bits == 16:
        scale = scale.bfloat16().double()
    return ((blocks / torch.where(scale > 0, scale, 1.0)).round().clamp(-127, 127) * scale).view(x.shape)


def arrived64(msg, like):
    codes, scales = msg
    scales = (scales if scales.dtype == torch.float32 else scales.view(torch.bfloat16)).double()
    return (codes.double().view(-1, 64) * scales[:, None]).view(like.shape).to(like.dtype).double()


def exact_stage(s):
    case = s["case"]
    coded = case["coded"]
    x = (arrived64(s["in_message"], s["x"]) if coded else s["x"].double()).requires_grad_(case["do"] != "forward")
    params = [to64(p) for p in s["params"]]
    y = x
    with torch.set_grad_enabled(case["do"] != "forward"):
        for p in params:
            for _ in range(case["repeat"]):
                y = block64(y, p, case["heads"], case["block"])
    out = {}
    if case["do"] != "backward":
        out["y"] = through_message64(y, case["scale_bits"]) if coded else y.detach()
    if case["do"] != "forward":
        y.backward(arrived64(s["in_grad"], s["dy"]) if coded else s["dy"].double())
        out["dx"] = through_message64(x.grad, case["scale_bits"]) if coded else x.grad
        out["grads"] = [{k: v.grad for k, v in p.items()} for p in params]
    return out


def exact_boundary(s):
    case, k = s["case"], s["case"]["d"] // s["case"]["d_comp"]
    y, comp, dec = s["y"].double().requires_grad_(), to64(s["comp"]), to64(s["dec"])
    a = norm64(y, comp["ln_g"], comp["ln_b"])
    if case["kind"] == "bottleneck":
        z = a @ comp["w_c"].T
    else:
        # the window's first maximum among the values as they are stored
        stored = a.detach().to(s["y"].dtype).view(-1, case["d_comp"], k)
        best = stored == stored.amax(-1, keepdim=True)
        z = (a.view(stored.shape) * (best & (best.cumsum(-1) == 1))).sum(-1)
    sent = z.detach().requires_grad_()
    x = norm64(sent, dec["ln_g"], dec["ln_b"]) @ dec["w_d"].T
    x.backward(s["dx"].double())
    z.backward(sent.grad)
    return {"z": z.detach(), "x": x.detach(), "dz": sent.grad, "dy": y.grad,
            "dec_grads": {k: v.grad for k, v in dec.items()}, "comp_grads": {k: v.grad for k, v in comp.items()}}


def exact_head(s):
    V, tokens = s["case"]["vocab"], s["tokens"].long()
    x, head, table = s["x"].double().requires_grad_(), to64(s["head"]), s["table"].double().requires_grad_()
    embedded = table[tokens]
    logits = norm64(x, head["ln_g"], head["ln_b"]) @ head["w_vocab"][:V].T
    token_loss = torch.nn.functional.cross_entropy(logits, s["targets"].long(), reduction="none")
    out = {"embedded": embedded.detach(), "loss": token_loss.mean().detach().view(1), "token_loss": token_loss.detach()}
    if s["case"]["do"] == "loss":
        return out
    token_loss.mean().backward()
    embedded.backward(s["d_embedded"].double())
    return dict(out, dx=x.grad, head_grads={k: v.grad for k, v in head.items()}, table_grad=table.grad)


def exact_lamb(s):
    lr, b1, b2, eps, decay, step = 1e-3, 0.9, 0.95, 1e-6, 0.01, 100
    out = []
    for t in s["tensors"]:
        w, g = t["master"].double(), t["grad"].double()
        m, v = b1 * t["m"].double() + (1 - b1) * g, b2 * t["v"].double() + (1 - b2) * g * g
        u = (m / (1 - b1 ** step)) / ((v / (1 - b2 ** step)).sqrt() + eps) + decay * w
        w = w - lr * w.norm() / u.norm() * u
        out.append({"master": w, "param": w, "m": m, "v": v})
    return out


def exact(case, seed):
    if case["path"] == "codec":      # whole numbers and their products, compared bit for bit
        return None
    s = prepare(case, seed)
    del s["workspace"]
    return {"stage": exact_stage, "boundary": exact_boundary, "head": exact_head, "lamb": exact_lamb}[case["path"]](s)

"""The work that a user of this framework has it do, as cases that can be measured.

Four kinds of call, each through the public entry points:

  generate  Session.prefill of a batch of prompts, then Session.decode_into for
            each generated token
  decode    one Session.decode_into step of a batch whose caches are filled
  prefill   Session.prefill of a batch of prompts, whole or in chunks (append),
            with the last position's logits or every position's
  train     the training-side gather-scatter of every loop: train.plan, gather,
            scatter and their gradients around a block that the caller owns

The tokens of a decode step are handed in (a sampler's choice), so that two
correct implementations, whose logits differ in the last bits, decode the same
sequence.  Weights are random with the models' own initial scale, the router's
bias is fitted so that the routed depths have the long-tailed mix (mean 3.7 of
8 loops) of the decode workloads.
"""
import math

import torch

from paper_2609_15160_amd import tlf, train

# storage, vocabulary, width, heads, head width, SwiGLU width, layers, loops
MODELS = {
    "f32_d64": ("f32", 512, 64, 4, 16, 256, 1, 4),        # the tiny float32 model
    "f32_d256": ("f32", 512, 256, 4, 64, 512, 2, 4),      # a small two-layer float32 model
    "bf16_d768": ("bf16", 32000, 768, 12, 64, 2048, 2, 8),
    "bf16_d1024": ("bf16", 32000, 1024, 16, 64, 2816, 2, 8),
    "bf16_d2048": ("bf16", 32000, 2048, 16, 128, 5504, 2, 8),
}
DEPTH_MIX = (0.13, 0.17, 0.20, 0.19, 0.12, 0.09, 0.06, 0.04)  # shares of depth 1..8
EPS = 1e-5
ROOM = 1024  # decode cases: steps that a filled cache has room for before its prompts are read again


class Model:
    """The model description that Session takes."""

    def __init__(self, case):
        (self.dtype, self.vocab, self.d_model, self.n_heads, self.head_dim, self.d_ff, self.n_layers,
         self.max_loops) = MODELS[case["model"]]
        self.rms_eps = EPS
        self.adaln = bool(case.get("adaln", False))
        self.router_hidden = self.d_model if case.get("mlp_router", False) else 0
        self.max_pos = positions(case)


def positions(case):
    if case["kind"] == "decode":
        return case["prompt"] + ROOM
    return case["prompt"] + case.get("steps", 0)


def case_(kind, model, batch, prompt, **more):
    return dict(kind=kind, model=model, batch=batch, prompt=prompt, **more)


def listed():
    named = lambda name, c: dict(c, name=name)  # noqa: E731
    return [
        # a whole request on the tiny float32 model: 32 prompt tokens, 32 generated ones (launches and latency)
        named("generate_f32_d64_b1x32", case_("generate", "f32_d64", 1, 32, steps=32)),
        # one interactive user: a decode step of a single sequence
        named("decode_d768_b1x512", case_("decode", "bf16_d768", 1, 512)),
        # a decode step of a small serving batch
        named("decode_d768_b32x512", case_("decode", "bf16_d768", 32, 512)),
        # a decode step of a large batch with long caches (the benchmark's workload)
        named("decode_d768_b256x2048", case_("decode", "bf16_d768", 256, 2048)),
        # the larger model: a decode step with 4096-token caches and head width 128
        named("decode_d2048_b64x4096", case_("decode", "bf16_d2048", 64, 4096)),
        # time to first token of one request whose length fits no tile
        named("prefill_d768_b1x1000", case_("prefill", "bf16_d768", 1, 1000)),
        # one long request handed in 512-token chunks between other requests' decode steps
        named("chunked_d768_b1x2048", case_("prefill", "bf16_d768", 1, 2048, chunk=512)),
        # a serving batch's prompts at the default precision (activations in two bf16 parts)
        named("prefill_d768_b32x512", case_("prefill", "bf16_d768", 32, 512)),
        # long prompts with one bf16 part per activation (the prefill workload)
        named("prefill_d1024_b8x4096_act16", case_("prefill", "bf16_d1024", 8, 4096, act16=True)),
        # scoring ragged texts: logits of every position
        named("score_d768_b3x777", case_("prefill", "bf16_d768", 3, 777, all_logits=True)),
        # the conditioned block, the two-layer router and the cumulative depth rule: prompts and 8 tokens
        named("generate_adaln_d768_b16x200", case_("generate", "bf16_d768", 16, 200, steps=8, adaln=True,
                                                   mlp_router=True, rule="cumprob")),
        # a training step's gather-scatter, forward and backward, over all loops
        named("train_gs_d1024_b8x4096", case_("train", "bf16_d1024", 8, 4096)),
    ]


def log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("generate", "decode", "decode", "prefill", "prefill", "chunked", "train"))
    if kind == "generate":
        if rng.random() < 0.5:
            return case_("generate", rng.choice(("f32_d64", "f32_d256")), log_int(rng, 1, 16), log_int(rng, 8, 300),
                         steps=rng.randint(8, 32))
        batch = log_int(rng, 1, 32)
        return case_("generate", "bf16_d768", batch, log_int(rng, 16, 8192 // batch), steps=rng.randint(4, 12),
                     adaln=rng.random() < 0.5, mlp_router=True, rule=rng.choice(("argmax", "cumprob")))
    if kind == "decode":
        model = rng.choice(("bf16_d768", "bf16_d768", "bf16_d1024", "bf16_d2048"))
        batch = log_int(rng, 1, 64 if model == "bf16_d2048" else 256)
        most = {"bf16_d768": 524288, "bf16_d1024": 393216, "bf16_d2048": 196608}[model]
        return case_("decode", model, batch, log_int(rng, 64, min(4096, most // batch)))
    if kind == "train":
        return case_("train", rng.choice(("bf16_d768", "bf16_d1024")), log_int(rng, 1, 16), log_int(rng, 64, 2048))
    if kind == "chunked":
        chunk = log_int(rng, 64, 600)
        return case_("prefill", "bf16_d768", log_int(rng, 1, 4), chunk * rng.randint(2, 4) - rng.randint(0, chunk // 2),
                     chunk=chunk)
    batch = log_int(rng, 1, 64)
    if rng.random() < 0.25:
        return case_("prefill", "bf16_d768", min(batch, 16), log_int(rng, 16, 4096 // min(batch, 16)), all_logits=True)
    model = rng.choice(("bf16_d768", "bf16_d1024"))
    return case_("prefill", model, batch, log_int(rng, 32, min(4096, 24576 // batch)),
                 act16=model == "bf16_d1024" and rng.random() < 0.5)


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def generator(seed, stream):
    return torch.Generator(device="cuda").manual_seed(1000003 * seed + stream)


def make_weights(case, m, seed):
    """Weights on the GPU, rounded to the storage type and held as float32: linear layers [out][in]."""
    g = generator(seed, 1)
    d, F, V, R = m.d_model, m.d_ff, m.vocab, m.max_loops

    def normal(*shape, std=0.02, store=True):
        t = torch.randn(*shape, generator=g, device="cuda") * std
        return t.to(torch.bfloat16).float() if store and m.dtype == "bf16" else t

    w = {"tok_emb": normal(V, d), "pos_emb": normal(m.max_pos, d)}
    if m.router_hidden:
        w["router_w1"] = normal(m.router_hidden, d, std=1.0 / (math.sqrt(2.0 * d) * 0.02))
        w["router_b1"] = torch.zeros(m.router_hidden, device="cuda")
        w["router_w"] = normal(R, m.router_hidden, std=2.0 / math.sqrt(m.router_hidden))
    else:
        w["router_w"] = normal(R, d)
    w["layers"] = [{"w_qkv": normal(3 * d, d), "w_o": normal(d, d), "w_gate_up": normal(2 * F, d),
                    "w_down": normal(d, F)} for _ in range(m.n_layers)]
    if m.adaln:
        w["cond"] = {}
        for which in ("time", "step"):
            w["cond"].update({which + "_w1": normal(d, 256, std=1.0 / math.sqrt(128)),
                              which + "_b1": normal(d, std=0.1, store=False),
                              which + "_w2": normal(d, d, std=1.0 / math.sqrt(d)),
                              which + "_b2": normal(d, std=0.1, store=False)})
        for lw in w["layers"]:
            lw["w_mod"] = normal(4 * d, d, std=0.5 / math.sqrt(d))
            lw["b_mod"] = normal(4 * d, std=0.05, store=False)
    w["router_b"] = router_bias(w, m, g)
    return w


def router_bias(w, m, g):
    """Bias under which the argmax depths of random tokens have the target mix (float32 models: none)."""
    b = torch.zeros(m.max_loops, device="cuda")
    if m.dtype == "f32":
        return b
    n = 1 << 15
    tok = torch.randint(0, m.vocab, (n,), generator=g, device="cuda")
    pos = torch.randint(0, m.max_pos, (n,), generator=g, device="cuda")
    z = router_logits(w, w["tok_emb"][tok] + w["pos_emb"][pos])
    want = torch.tensor(DEPTH_MIX, device="cuda")
    step = 0.5 * (z - z.mean(0)).std()
    for _ in range(60):
        have = torch.bincount((z + b).argmax(1), minlength=m.max_loops) / n
        b = b + step * (want.log() - have.clamp(min=1.0 / n).log())
        b = b - b[0]
    return b


def router_logits(w, h0):
    if "router_w1" in w:
        h0 = torch.nn.functional.silu(h0 @ w["router_w1"].T + w["router_b1"])
    return h0 @ w["router_w"].T


def make_tokens(case, m, seed):
    """Prompts [B][prompt] and the tokens decoded after them [steps][B]."""
    g = generator(seed, 2)
    steps = ROOM if case["kind"] == "decode" else case.get("steps", 0)
    draw_ = lambda *s: torch.randint(0, m.vocab, s, generator=g, device="cuda", dtype=torch.int32)  # noqa: E731
    return draw_(case["batch"], case["prompt"]), draw_(steps, case["batch"])


def on_host(v):
    if isinstance(v, dict):
        return {k: on_host(x) for k, x in v.items()}
    return [on_host(x) for x in v] if isinstance(v, list) else v.cpu().numpy()


def prepare(case, seed):
    return prepare_train(case, seed) if case["kind"] == "train" else prepare_session(case, seed)


def prepare_session(case, seed):
    m = Model(case)
    weights = on_host(make_weights(case, m, seed))
    prompts, tokens = make_tokens(case, m, seed)
    sess = tlf.Session(m, weights, max_batch=case["batch"], route_rule=case.get("rule", "argmax"),
                       max_prefill_tokens=min(65536, max(case["batch"] * case["prompt"], 1)),
                       prefill_act_bf16=bool(case.get("act16", False)))
    s = {"case": case, "sess": sess, "prompts": prompts, "tokens": tokens, "at": 0}
    if case["kind"] != "prefill":
        s["tok"] = torch.empty(case["batch"], dtype=torch.int32, device="cuda")
        s["logits"] = torch.empty(case["batch"], m.vocab, device="cuda")
        s["next"], s["depths"] = torch.empty_like(s["tok"]), torch.empty_like(s["tok"])
    if case["kind"] == "decode":
        sess.prefill(prompts, want_depths=False)
    if case.get("chunk"):
        s["chunks"] = [c.contiguous() for c in prompts.split(case["chunk"], dim=1)]
    return s


def train_depths(case, seed, loops):
    """Depths in the mix's shares of the batch, in random order."""
    rows, cdf = case["batch"] * case["prompt"], 0.0
    depth = torch.full((rows,), loops, dtype=torch.int32)
    ends = [0]
    for i, share in enumerate(DEPTH_MIX[:loops - 1]):
        cdf += share
        ends.append(int(round(cdf * rows)))
        depth[ends[-2]:ends[-1]] = i + 1
    return depth.cuda()[torch.randperm(rows, generator=generator(seed, 3), device="cuda")]


def train_tensors(case, seed):
    """Depths, the states, each loop's block output, and the gradients that arrive at the last states and at
    each loop's gathered rows."""
    m = Model(case)
    depth, g = train_depths(case, seed, m.max_loops), generator(seed, 4)
    rows, d = case["batch"] * case["prompt"], m.d_model
    normal = lambda n: torch.randn(n, d, generator=g, device="cuda")  # noqa: E731
    counts = [int((depth >= i).sum()) for i in range(1, m.max_loops + 1)]
    return depth, normal(rows), [normal(n) for n in counts], normal(rows), [normal(n) for n in counts]


def prepare_train(case, seed):
    depth, h, ys, gh, gxs = train_tensors(case, seed)
    ws = train.plan_workspace(case["batch"], case["prompt"])
    return {"case": case, "depth": depth, "h": h.requires_grad_(), "ys": [y.requires_grad_() for y in ys], "gh": gh,
            "gxs": gxs, "ws": ws}


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------

def run(s):
    return {"train": run_train, "decode": run_decode, "generate": run_generate, "prefill": run_prefill}[
        s["case"]["kind"]](s)


def step(s, k):
    s["tok"].copy_(s["tokens"][k])
    s["sess"].decode_into(s["tok"], s["logits"], next_tok=s["next"], depths=s["depths"])


def run_decode(s):
    if s["at"] == ROOM:  # the caches are full: the next batch of requests
        s["sess"].prefill(s["prompts"], want_depths=False)
        s["at"] = 0
    step(s, s["at"])
    s["at"] += 1
    return {"logits": s["logits"], "depths": s["depths"]}


def run_generate(s):
    first, depths = s["sess"].prefill(s["prompts"])
    for k in range(s["case"]["steps"]):
        step(s, k)
    return {"first_logits": first, "prompt_depths": depths, "logits": s["logits"], "depths": s["depths"]}


def run_prefill(s):
    if "chunks" not in s:
        logits, depths = s["sess"].prefill(s["prompts"], all_logits=bool(s["case"].get("all_logits", False)))
        return {"logits": logits, "depths": depths}
    parts = [s["sess"].prefill(c, append=k > 0) for k, c in enumerate(s["chunks"])]
    return {"logits": parts[-1][0], "depths": [p[1] for p in parts]}


def run_train(s):
    case, h = s["case"], s["h"]
    xs = []
    for i, y in enumerate(s["ys"]):
        p = train.plan(s["depth"], case["batch"], case["prompt"], i + 1, s["ws"])
        xs.append(train.gather(h, p))
        h = train.scatter(h, y, p)
    grads = torch.autograd.grad([h] + xs, [s["h"]] + s["ys"], [s["gh"]] + s["gxs"])
    return {"x": [x.detach() for x in xs], "h": h.detach(), "grad_h": grads[0], "grad_y": list(grads[1:])}


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------

def work(case):
    """Bytes: each weight, cache entry and input read once, each output and new cache entry written once.
    flops: products of the active rows only, causal attention over the gathered tokens."""
    m = Model(case)
    s = 2 if m.dtype == "bf16" else 4
    d, F, V, J, B, T = m.d_model, m.d_ff, m.vocab, m.n_layers, case["batch"], case["prompt"]
    mix = DEPTH_MIX if m.max_loops == 8 else (1.0 / m.max_loops,) * m.max_loops
    share = [sum(mix[i:]) for i in range(m.max_loops)]  # tokens that run loop i + 1
    loops, pairs = sum(share), sum(p * p for p in share)
    if case["kind"] == "train":
        rows = B * T * d * 4
        # forward: gathered rows read and written, block outputs read, the states read and written once;
        # backward the same for the gradients
        return {"bytes": 2 * (3 * loops * rows + 2 * rows), "flops": 2 * loops * B * T * d}
    block, kv = J * (4 * d * d + 3 * d * F), 2 * J * d * s
    steps = 1 if case["kind"] == "decode" else case.get("steps", 0)
    nbytes, flops = (block + V * d) * s, 0.0
    if case["kind"] != "decode":
        rows = B * T
        out = rows if case.get("all_logits") else B * (-(-T // case["chunk"]) if case.get("chunk") else 1)
        nbytes += rows * d * s + loops * rows * kv + out * V * 4
        flops += 2 * rows * loops * block + 2 * out * V * d + 2 * J * d * B * T * T * pairs
    for k in range(steps):
        nbytes += B * (pairs * (T + k) + loops) * kv + B * V * 4
        flops += 2 * B * loops * block + 2 * B * V * d + 4 * J * d * B * (T + k) * pairs
    return {"bytes": float(nbytes), "flops": float(flops)}


def tolerance(case):
    if case["kind"] == "train":
        return {"rel": 1e-6}  # sums of a few float32 values per element, in any order
    if MODELS[case["model"]][0] == "f32":
        return {"rel": 5e-6, "differ": 0.002}
    # bf16: keys, values and attention weights are rounded to 8 bits on the way (and the activations
    # with act16): 2e-3 to 4e-3 from 64 bits, 6e-3 with act16; whole values are the routed depths,
    # decided in float32
    return {"rel": 2e-2 if case.get("act16") else 1e-2, "max": 0.1, "differ": 0.002}


# ---------------------------------------------------------------------------
# The same in 64 bits
# ---------------------------------------------------------------------------

def exact(case, seed):
    return exact_train(case, seed) if case["kind"] == "train" else exact_session(case, seed)


def exact_train(case, seed):
    depth, h, ys, gh, gxs = train_tensors(case, seed)
    at = [(depth >= i + 1).nonzero()[:, 0] for i in range(len(ys))]
    h, xs = h.double(), []
    for idx, y in zip(at, ys):
        xs.append(h[idx])
        h = h.index_add(0, idx, y.double())
    g, gys = gh.double(), []
    for idx, gx in zip(reversed(at), reversed(gxs)):
        gys.insert(0, g[idx])
        g = g.index_add(0, idx, gx.double())
    return {"x": xs, "h": h, "grad_h": g, "grad_y": gys}


def rms_norm(x):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + EPS)


def modulations(w, m):
    """[layer][loop][depth]: the four modulation vectors, side by side."""
    freq = torch.exp(-torch.arange(128, device="cuda", dtype=torch.float64) / 128 * math.log(10000.0))

    def embed(which, tau):
        c = w["cond"]
        f = torch.stack([torch.cos(tau * freq), torch.sin(tau * freq)], 1).reshape(-1)
        return c[which + "_w2"] @ torch.nn.functional.silu(c[which + "_w1"] @ f + c[which + "_b1"]) + c[which + "_b2"]

    table = {}
    for i in range(m.max_loops):
        for depth in range(i + 1, m.max_loops + 1):
            e = torch.nn.functional.silu(embed("time", i / depth) + embed("step", 1.0 / depth))
            for j, lw in enumerate(w["layers"]):
                table[j, i, depth] = lw["w_mod"] @ e + lw["b_mod"]
    return table


def depths_of(case, w, m, h0):
    z = router_logits(w, h0) + w["router_b"]
    if case.get("rule", "argmax") == "argmax":
        return z.argmax(-1) + 1
    tail = torch.softmax(z, -1).flip(-1).cumsum(-1).flip(-1)
    tail[..., 0] = 1.0
    return torch.where(tail > 0.5, torch.arange(1, m.max_loops + 1, device=z.device), 0).amax(-1)


def exact_session(case, seed):
    m = Model(case)
    up = lambda v: ({k: up(x) for k, x in v.items()} if isinstance(v, dict) else  # noqa: E731
                    [up(x) for x in v] if isinstance(v, list) else v.double())
    w = up(make_weights(case, m, seed))
    prompts, tokens = make_tokens(case, m, seed)
    steps = 1 if case["kind"] == "decode" else case.get("steps", 0)
    seqs = torch.cat([prompts, tokens[:steps].T], 1).long()
    T, n = case["prompt"], seqs.shape[1]
    if case.get("all_logits"):
        wanted = torch.arange(n, device="cuda")
    else:
        wanted = torch.tensor([T - 1, n - 1], device="cuda")
    mods = modulations(w, m) if m.adaln else None
    rows = torch.cat([exact_sequence(case, w, m, seqs[b], mods)[wanted] for b in range(case["batch"])], 0)
    logits = (rms_norm(rows) @ w["tok_emb"].T).reshape(case["batch"], len(wanted), m.vocab)
    if case["kind"] == "generate":
        return {"first_logits": logits[:, 0], "prompt_depths": None, "logits": logits[:, 1], "depths": None}
    return {"logits": logits if case.get("all_logits") else logits[:, 1], "depths": None}


def exact_sequence(case, w, m, ids, mods):
    """The last state of every position of one sequence: each loop on the tokens deep enough for it, causal
    attention among them."""
    d, F, H, D = m.d_model, m.d_ff, m.n_heads, m.head_dim
    x = w["tok_emb"][ids] + w["pos_emb"][: len(ids)]
    depth = depths_of(case, w, m, x)
    for i in range(m.max_loops):
        at = (depth > i).nonzero()[:, 0]
        n = len(at)
        if n == 0:
            break
        h = x[at]
        mask = torch.ones(n, n, dtype=torch.bool, device="cuda").tril()
        for j, lw in enumerate(w["layers"]):
            if mods is None:
                a1 = a2 = g1 = g2 = 0.0
            else:
                rows = torch.stack([mods.get((j, i, k), torch.zeros_like(mods[j, i, i + 1]))
                                    for k in range(1, m.max_loops + 1)])[depth[at] - 1]
                a1, a2, g1, g2 = rows.split(d, 1)
            q, k, v = ((rms_norm(h) * (1 + g1)) @ lw["w_qkv"].T).reshape(n, 3, H, D).permute(1, 2, 0, 3).contiguous()
            p = q @ k.transpose(1, 2).contiguous() / math.sqrt(D)
            p = torch.softmax(p.masked_fill_(~mask, -math.inf), -1)
            o = (p @ v).transpose(0, 1).reshape(n, d)
            h = h + (1 + a1) * (o @ lw["w_o"].T)
            gate, up = ((rms_norm(h) * (1 + g2)) @ lw["w_gate_up"].T).split(F, 1)
            h = h + (1 + a2) * ((torch.nn.functional.silu(gate) * up) @ lw["w_down"].T)
        x = x.index_copy(0, at, h)
    return x

"""Performance cases: planned graphs run through the framework's public API.

Every case builds a graph, measures its cost table on the GPU, plans layouts
and the arena, and times one run of the plan: eagerly (``Executor.run``) or as
a replay of the captured HIP graph (``Executor.capture``).  A program measures
and plans a graph once and then runs it for every request, so the plan of a
shape is made once per process (``_plan``); inputs, weights, buffers and the
captured graph belong to each prepared state.

Kinds of case:
  * ``stack``: whole transformer stacks of ``Graph.transformer`` (post-LN
    encoders, pre-LN causal decoders, Llama-style decoders), one sequence;
  * ``ffn``: one feed-forward block with its residual and norm (GELU with
    biases and LayerNorm in fp32, SwiGLU with RMSNorm in bf16), any batch;
  * ``attn``: one attention core (Q K^T, softmax, P V) over the heads;
  * ``vgg``: VGG-shaped convolutional networks.
"""
import math

import torch

from paper_2411_09242_amd import fluid as F

EPS = 1e-5
ROPE_BASE = 10000.0


# ------------------------------------------------------------------ cases
def listed():
    return [
        # one short request through a tiny encoder: launches and latency only
        dict(name="encoder-tiny", kind="stack", arch="post_ln", dtype="f32", layers=1, seq=32, hidden=64, heads=2,
             ffn=256, graph=False),
        # a BERT-base-shaped encoder over one 128-token text, issued eagerly
        # launch by launch and as a captured graph
        dict(name="encoder-base-eager", kind="stack", arch="post_ln", dtype="f32", layers=12, seq=128, hidden=768,
             heads=12, ffn=3072, graph=False),
        dict(name="encoder-base", kind="stack", arch="post_ln", dtype="f32", layers=12, seq=128, hidden=768, heads=12,
             ffn=3072, graph=True),
        # layers of a BERT-large-shaped encoder over a short query: the
        # weights are read for a few rows only
        dict(name="encoder-short", kind="stack", arch="post_ln", dtype="f32", layers=4, seq=16, hidden=1024, heads=16,
             ffn=4096, graph=True),
        # GPT-2-small-shaped prefill layers of one 512-token prompt
        dict(name="prefill-512", kind="stack", arch="pre_ln", dtype="f32", layers=3, seq=512, hidden=768, heads=12,
             ffn=3072, graph=True),
        # an odd sequence length (rows that are no multiple of any vector)
        dict(name="encoder-ragged", kind="stack", arch="post_ln", dtype="f32", layers=2, seq=197, hidden=384, heads=6,
             ffn=1536, graph=True),
        # the BERT-large-shaped batch of 8 x 512 tokens: its feed-forward
        # block and its attention core
        dict(name="ffn-b8", kind="ffn", dtype="f32", batch=8, seq=512, hidden=1024, ffn=4096, graph=True),
        dict(name="attn-b8", kind="attn", dtype="f32", batch=8, heads=16, seq=512, dim=64, causal=False, graph=True),
        # the Llama-style 2048-token prefill in bf16: the SwiGLU block and
        # the causal attention core
        dict(name="ffn-bf16", kind="ffn", dtype="bf16", batch=1, seq=2048, hidden=4096, ffn=11008, graph=True),
        dict(name="attn-bf16", kind="attn", dtype="bf16", batch=1, heads=32, seq=2048, dim=128, causal=True,
             graph=True),
        # a whole bf16 decoder layer at a small width and an odd prompt length
        dict(name="decoder-bf16", kind="stack", arch="llama", dtype="bf16", layers=1, seq=333, hidden=1024, heads=8,
             ffn=2816, graph=True),
        # the VGG-16-shaped network on one image
        dict(name="vgg16", kind="vgg", dtype="f32", batch=1, channels=3, image=224, stages="64x2 128x2 256x3 512x3 512x3",
             fc=4096, classes=1000, graph=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["stack", "stack", "ffn", "ffn", "attn", "vgg"])
    graph = rng.random() < 0.7
    if kind == "stack":
        arch = rng.choice(["post_ln", "pre_ln", "llama"])
        bf16 = arch == "llama"
        heads, dim = rng.randint(2, 16), rng.choice([32, 64, 64, 128] if bf16 else [32, 64, 64])
        hidden = heads * dim
        # GELU blocks are 4x as wide; SwiGLU blocks about 8/3, a multiple of 8
        ffn = 4 * hidden if not bf16 else (8 * hidden // 3 + 7) // 8 * 8
        return dict(kind=kind, arch=arch, dtype="bf16" if bf16 else "f32", layers=rng.randint(1, 2),
                    seq=_log(rng, 16, 700), hidden=hidden, heads=heads, ffn=ffn, graph=graph)
    if kind == "ffn":
        dtype = rng.choice(["f32", "bf16"])
        tokens = _log(rng, 16, 4096 if dtype == "f32" else 2048)
        hidden = 32 * _log(rng, 4, 32 if dtype == "f32" else 96)
        ffn = 4 * hidden if dtype == "f32" else (8 * hidden // 3 + 7) // 8 * 8
        return dict(kind=kind, dtype=dtype, batch=1, seq=tokens, hidden=hidden, ffn=ffn, graph=graph)
    if kind == "attn":
        return dict(kind=kind, dtype=rng.choice(["f32", "bf16"]), batch=rng.randint(1, 4), heads=rng.randint(2, 16),
                    seq=_log(rng, 16, 1024), dim=rng.choice([32, 64, 128]), causal=rng.random() < 0.5, graph=graph)
    n = rng.randint(1, 4)
    widths = [8 * rng.randint(2, 8)]
    while len(widths) < n:
        widths.append(min(256, 2 * widths[-1]))
    return dict(kind="vgg", dtype="f32", batch=rng.randint(1, 2), channels=rng.choice([1, 3]),
                image=2 ** n * rng.randint(7, max(8, 112 // 2 ** n)),
                stages=" ".join("%dx%d" % (w, rng.randint(1, 2)) for w in widths), fc=64 * rng.randint(1, 16),
                classes=rng.randint(10, 1000), graph=graph)


# ----------------------------------------------------------------- graphs
def _stages(case):
    return tuple(tuple(int(v) for v in s.split("x")) for s in case["stages"].split())


class _Desc:
    """A graph description in the framework's dict form."""

    def __init__(self, dtype, inputs):
        self.d = dict(dtype=dtype, inputs=[list(s) for s in inputs], consts=[], nodes=[], outputs=[])

    def const(self, role, *shape):
        self.d["consts"].append(dict(role=role, shape=list(shape), dtype=self.d["dtype"]))
        return ~(len(self.d["consts"]) - 1)

    def node(self, op, ins, shape, **kw):
        self.d["nodes"].append(dict(op=op, ins=ins, out_shape=list(shape), **kw))
        return len(self.d["inputs"]) + len(self.d["nodes"]) - 1


def _build(case):
    dt = case["dtype"]
    if case["kind"] == "stack":
        return F.Graph.transformer(dict(arch=case["arch"], layers=case["layers"], batch=1, seq=case["seq"],
                                        hidden=case["hidden"], heads=case["heads"], ffn=case["ffn"], dtype=dt,
                                        eps=EPS, rope_base=ROPE_BASE))
    if case["kind"] == "vgg":
        return F.Graph.transformer(dict(arch="vgg", batch=case["batch"], channels=case["channels"],
                                        image=case["image"], stages=_stages(case), fc=case["fc"],
                                        classes=case["classes"], dtype=dt, eps=EPS))
    if case["kind"] == "ffn":
        B, S, H, W = case["batch"], case["seq"], case["hidden"], case["ffn"]
        b = _Desc(dt, [(B, S, H)])
        if dt == "f32":      # post-LN block: x + GELU MLP, then LayerNorm
            e = b.node("matmul", [0, b.const("weight", H, W)], (B, S, W))
            e = b.node("add", [e, b.const("bias", W)], (B, S, W))
            e = b.node("gelu", [e], (B, S, W))
            e = b.node("matmul", [e, b.const("weight", W, H)], (B, S, H))
            e = b.node("add", [e, b.const("bias", H)], (B, S, H))
            e = b.node("add", [e, 0], (B, S, H))
            e = b.node("layernorm", [e, b.const("gamma", H), b.const("beta", H)], (B, S, H), fattr=EPS)
        else:                # SwiGLU block: x + down(SiLU(gate) * up), then RMSNorm
            wg, wu, wd = b.const("weight", H, W), b.const("weight", H, W), b.const("weight", W, H)
            g = b.node("silu", [b.node("matmul", [0, wg], (B, S, W))], (B, S, W))
            u = b.node("matmul", [0, wu], (B, S, W))
            e = b.node("matmul", [b.node("mul", [g, u], (B, S, W)), wd], (B, S, H))
            e = b.node("add", [e, 0], (B, S, H))
            e = b.node("rmsnorm", [e, b.const("gamma", H)], (B, S, H), fattr=EPS)
        b.d["outputs"] = [e]
        return F.Graph.from_desc(b.d)
    B, N, S, D = case["batch"], case["heads"], case["seq"], case["dim"]
    b = _Desc(dt, [(B, N, S, D), (B, N, D, S), (B, N, S, D)])
    s = b.node("matmul", [0, 1], (B, N, S, S))
    p = b.node("softmax", [s], (B, N, S, S), fattr=1.0 / math.sqrt(D), iattr=int(case["causal"]))
    b.d["outputs"] = [b.node("matmul", [p, 2], (B, N, S, D))]
    return F.Graph.from_desc(b.d)


_PLANS = {}


def _plan(case):
    """The graph, its layout plan and its arena plan: measured and planned
    once per shape, as a program does that then serves many requests."""
    key = tuple(sorted((k, v) for k, v in case.items() if k not in ("name", "graph")))
    if key not in _PLANS:
        g = _build(case)
        table = F.CostTable.measure(g, reps=7)
        lp = F.LayoutPlan(g, table)
        _PLANS[key] = (g, lp, F.ArenaPlan(g, lp, epilogue=True))
    return _PLANS[key]


# ----------------------------------------------------------------- inputs
def _const_roles(case):
    """(role, shape) of every constant, in graph order."""
    k = case["kind"]
    if k == "attn":
        return []
    if k == "vgg":
        out, c = [], case["channels"]
        for w, n in _stages(case):
            for _ in range(n):
                out += [("weight", (w, c, 3, 3)), ("bias", (w,))]
                c = w
        side = case["image"] >> len(_stages(case))
        sizes = [c * side * side, case["fc"], case["fc"], case["classes"]]
        for a, b in zip(sizes, sizes[1:]):
            out += [("weight", (a, b)), ("bias", (b,))]
        return out
    H, W = case["hidden"], case["ffn"]
    norm = [("gamma", (H,)), ("beta", (H,))]
    up = [("weight", (H, W)), ("bias", (W,)), ("weight", (W, H)), ("bias", (H,))]
    if k == "ffn":
        if case["dtype"] == "f32":
            return up + norm
        return [("weight", (H, W)), ("weight", (H, W)), ("weight", (W, H)), ("gamma", (H,))]
    proj = [("weight", (H, H)), ("bias", (H,))]
    if case["arch"] == "post_ln":
        return (4 * proj + norm + up + norm) * case["layers"]
    if case["arch"] == "pre_ln":
        return (norm + 4 * proj + norm + up) * case["layers"] + norm
    S, half = case["seq"], H // case["heads"] // 2
    layer = ([("gamma", (H,))] + 4 * [("weight", (H, H))] + [("gamma", (H,)), ("weight", (H, W)), ("weight", (H, W)),
                                                             ("weight", (W, H))])
    return [("cos", (S, half)), ("sin", (S, half))] + layer * case["layers"] + [("gamma", (H,))]


def _inputs(case, seed):
    """Graph inputs and constants on the GPU, from the seed alone: N(0, 1)
    activations, 0.02 N(0, 1) projections (He-scaled in the convolutional
    network), small biases, norm scales near 1, rotary tables by position."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32

    def normal(shape, std=1.0, mean=0.0):
        return (mean + std * torch.randn(shape, generator=gen, device="cuda")).to(dt)

    if case["kind"] == "attn":
        B, N, S, D = case["batch"], case["heads"], case["seq"], case["dim"]
        xs = [normal((B, N, S, D)), normal((B, N, D, S)), normal((B, N, S, D))]
    elif case["kind"] == "vgg":
        xs = [normal((case["batch"], case["channels"], case["image"], case["image"]))]
    else:
        xs = [normal((case.get("batch", 1), case["seq"], case["hidden"]))]
    consts = []
    for role, shape in _const_roles(case):
        if role == "weight":
            fan_in = shape[0] if len(shape) == 2 else shape[1] * shape[2] * shape[3]
            consts.append(normal(shape, math.sqrt(2.0 / fan_in) if case["kind"] == "vgg" else 0.02))
        elif role == "gamma":
            consts.append(normal(shape, 0.1, 1.0))
        elif role in ("cos", "sin"):
            S, half = shape
            ang = (torch.arange(S, dtype=torch.float64)[:, None] *
                   ROPE_BASE ** (-torch.arange(half, dtype=torch.float64) / half)[None, :])
            consts.append((ang.cos() if role == "cos" else ang.sin()).float().cuda())
        else:
            consts.append(normal(shape, 0.02))
    return xs, consts


class _State:
    pass


def prepare(case, seed):
    g, lp, ap = _plan(case)
    xs, consts = _inputs(case, seed)
    s = _State()
    s.ex = F.Executor(g, lp, ap, consts, xs)
    s.graph = None
    if case["graph"]:
        s.ex.run()
        torch.cuda.synchronize()
        s.graph = s.ex.capture()
    return s


def run(state):
    if state.graph is None:
        return state.ex.run()
    state.graph.replay()
    return state.ex.outputs


# ------------------------------------------------------------ work, errors
def work(case):
    """Graph inputs and constants read once, outputs written once; products
    and convolutions, of a causal attention the lower triangle alone."""
    size = 2 if case["dtype"] == "bf16" else 4
    n = sum(math.prod(s) for _, s in _const_roles(case))
    if case["kind"] == "attn":
        B, N, S, D = case["batch"], case["heads"], case["seq"], case["dim"]
        pairs = S * (S + 1) // 2 if case["causal"] else S * S
        return dict(bytes=size * 4 * B * N * S * D, flops=4 * B * N * D * pairs)
    if case["kind"] == "vgg":
        B, c, side, flops = case["batch"], case["channels"], case["image"], 0
        n += B * (c * side * side + case["classes"])
        for w, k in _stages(case):
            for _ in range(k):
                flops += 2 * B * side * side * w * c * 9
                c = w
            side //= 2
        flops += sum(2 * B * math.prod(s) for _, s in _const_roles(case) if len(s) == 2)
        return dict(bytes=size * n, flops=flops)
    rows = case.get("batch", 1) * case["seq"]
    n += 2 * rows * case["hidden"]
    flops = sum(2 * rows * math.prod(s) for r, s in _const_roles(case) if r == "weight")
    if case["kind"] == "stack":
        S, H = case["seq"], case["hidden"]
        pairs = S * S if case["arch"] == "post_ln" else S * (S + 1) // 2
        flops += case["layers"] * 4 * H * pairs
    return dict(bytes=size * n, flops=flops)


def tolerance(case):
    """About four times what is seen between a run and 64-bit arithmetic:
    4e-3 where tensors are stored in bf16, 6e-7 through the fp32 blocks and
    stacks, 4e-6 after the network whose softmax turns an absolute error of
    its logits into a relative one."""
    if case["dtype"] == "bf16":
        return {"rel": 1.6e-2}
    return {"rel": 2e-5 if case["kind"] == "vgg" else 4e-6}


# ------------------------------------------------------------------ exact
def _norm(x, gamma, beta=None):
    if beta is None:
        return x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS) * gamma
    c = x - x.mean(-1, keepdim=True)
    return c / torch.sqrt((c * c).mean(-1, keepdim=True) + EPS) * gamma + beta


def _gelu(x):
    return 0.5 * x * (1.0 + torch.erf(x / math.sqrt(2.0)))


def _silu(x):
    return x / (1.0 + torch.exp(-x))


def _attention(q, kt, v, causal):
    """softmax(q kt / sqrt(D)) v, one head at a time (q [.., S, D], kt [.., D, S])."""
    S, D = q.shape[-2:]
    out = torch.empty_like(q)
    mask = torch.ones(S, S, dtype=torch.bool, device=q.device).triu(1) if causal else None
    for i in range(q.shape[0]):
        for j in range(q.shape[1]):
            s = (q[i, j] @ kt[i, j]) / math.sqrt(D)
            if causal:
                s = s.masked_fill(mask, -math.inf)
            out[i, j] = torch.softmax(s, -1) @ v[i, j]
    return out


def _conv3x3(x, w, b):
    """Same-padded 3 x 3 convolution as nine products over shifted images."""
    B, C, H, W = x.shape
    p = torch.nn.functional.pad(x, (1, 1, 1, 1))
    y = b[None, :, None].expand(B, -1, H * W).clone()
    for u in range(3):
        for v in range(3):
            win = p[:, :, u:u + H, v:v + W].reshape(B, C, H * W)
            for i in range(B):
                y[i] += w[:, :, u, v] @ win[i]
    return y.reshape(B, -1, H, W)


def exact(case, seed):
    xs, consts = _inputs(case, seed)
    x = xs[0].double()
    it = iter(c.double() for c in consts)

    def take(n):
        return [next(it) for _ in range(n)]

    if case["kind"] == "attn":
        return [_attention(x, xs[1].double(), xs[2].double(), case["causal"])]
    if case["kind"] == "vgg":
        for _, n in _stages(case):
            for _ in range(n):
                x = _conv3x3(x, *take(2)).relu()
            B, C, H, W = x.shape
            x = x.reshape(B, C, H // 2, 2, W // 2, 2).amax((3, 5))
        x = x.reshape(x.shape[0], -1)
        for i in range(3):
            w, b = take(2)
            x = x @ w + b
            x = x.relu() if i < 2 else torch.softmax(x, -1)
        return [x]
    if case["kind"] == "ffn":
        if case["dtype"] == "f32":
            w1, b1, w2, b2, g, b = take(6)
            return [_norm(_gelu(x @ w1 + b1) @ w2 + b2 + x, g, b)]
        wg, wu, wd, g = take(4)
        return [_norm((_silu(x @ wg) * (x @ wu)) @ wd + x, g)]
    S, H, N = case["seq"], case["hidden"], case["heads"]
    D, arch = H // N, case["arch"]

    def heads(t):
        return t.reshape(1, S, N, D).transpose(1, 2)

    def attend(q, k, v):
        c = _attention(heads(q).contiguous(), heads(k).transpose(2, 3).contiguous(), heads(v).contiguous(),
                       arch != "post_ln")
        return c.transpose(1, 2).reshape(1, S, H)

    if arch == "llama":
        cos, sin = (t[None, :, None, :] for t in take(2))

        def rope(t):
            a, b = t.reshape(1, S, N, D).chunk(2, -1)
            return torch.cat([a * cos - b * sin, b * cos + a * sin], -1).reshape(1, S, H)

        for _ in range(case["layers"]):
            g, wq, wk, wv, wo = take(5)
            h = _norm(x, g)
            x = x + attend(rope(h @ wq), rope(h @ wk), h @ wv) @ wo
            g, wg, wu, wd = take(4)
            h = _norm(x, g)
            x = x + (_silu(h @ wg) * (h @ wu)) @ wd
        return [_norm(x, *take(1))]

    def attention_block(h):
        wq, bq, wk, bk, wv, bv, wo, bo = take(8)
        return attend(h @ wq + bq, h @ wk + bk, h @ wv + bv) @ wo + bo

    def mlp(h):
        w1, b1, w2, b2 = take(4)
        return _gelu(h @ w1 + b1) @ w2 + b2

    for _ in range(case["layers"]):
        if arch == "post_ln":
            x = _norm(attention_block(x) + x, *take(2))
            x = _norm(mlp(x) + x, *take(2))
        else:
            x = x + attention_block(_norm(x, *take(2)))
            x = x + mlp(_norm(x, *take(2)))
    return [x if arch == "post_ln" else _norm(x, *take(2))]

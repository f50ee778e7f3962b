"""The work a user of this library has it do, as cases that can be timed and checked.

A case is one request batch taken through one stage (or a short chain of stages): a prefill of
the prompts, then cached decode steps, through the calls of paper_2511_14450_amd.  The inputs of
the decode steps are given in advance, so the whole request is a function of the inputs and
`exact` can evaluate it as one causal pass in float64.

Keys of a case
  hidden, q_heads, kv_heads, head_dim, ffn, dtype   shape of a block ("f32" | "bf16")
  split      blocks per stage, e.g. "1" or "3,2,1" (more than one stage: a StageChain)
  prompts    prompt lengths, comma separated; NxL stands for N prompts of L tokens
  steps      decode steps after the prefill
  room       tokens a request could hold beyond prompt + steps
  paged      KV cache in pages that are handed out in a shuffled order
  decode     "reused"  one output buffer, read before the next step (a generation loop)
             "rows"    every step writes its own row of a result array
             "new"     the call allocates its result
             "noalloc" stage_decode_step_noalloc
  export     the requests' caches are copied out afterwards (a move to another node)
"""
import math

import torch

from paper_2511_14450_amd import binding
from paper_2511_14450_amd.chain import StageChain

PHI3 = {"hidden": 5120, "q_heads": 40, "kv_heads": 10, "head_dim": 128, "ffn": 17920, "dtype": "bf16"}
LLAMA3 = {"hidden": 4096, "q_heads": 32, "kv_heads": 8, "head_dim": 128, "ffn": 14336, "dtype": "bf16"}
SMALL = {"hidden": 512, "q_heads": 8, "kv_heads": 2, "head_dim": 128, "ffn": 768, "dtype": "bf16"}
TINY = {"hidden": 256, "q_heads": 4, "kv_heads": 2, "head_dim": 64, "ffn": 1024, "dtype": "f32"}
PLAIN_USE = {"split": "1", "steps": 0, "room": 0, "paged": False, "decode": "reused", "export": False}
ROPE_BASE, EPS = 10000.0, 1e-5


def listed():
    def case(name, shape, prompts, **more):
        return {"name": name, **shape, **PLAIN_USE, "prompts": prompts, **more}

    return [
        # the smallest request: one narrow float32 block, where launches are all there is
        case("tiny_f32", TINY, "64", steps=16, decode="new"),
        # float32 blocks of ordinary width, prompts of unequal length
        case("f32_request", {"hidden": 1024, "q_heads": 8, "kv_heads": 4, "head_dim": 128, "ffn": 4096, "dtype": "f32"},
             "200,131,77,512", split="2", steps=24),
        # bf16 blocks whose heads have 64 features
        case("bf16_head64", {"hidden": 1024, "q_heads": 16, "kv_heads": 4, "head_dim": 64, "ffn": 4096, "dtype": "bf16"},
             "300,511,64,190", split="2", steps=24, room=100),
        # narrow bf16 blocks driven by a loop that must not allocate
        case("small_noalloc", SMALL, "45,130,1,77,300", split="3", steps=32, decode="noalloc"),
        # time to the first token of one short request
        case("short_prefill", PHI3, "64", split="2", room=256),
        # one request of the paper's shape through consecutive stages: 64 tokens in, 128 out
        case("paper_request", PHI3, "64", split="3,2,1", steps=128),
        # one block over a small batch of equal prompts
        case("batch_prefill", PHI3, "4x512"),
        # a server's stage with capacity to spare and short chat prompts of every length
        case("chat_batch", PHI3, "23,310,64,118,7,201,395,90,33,152,260,71,180,46,129,97", split="2", steps=48, room=3600),
        # one long document, prefilled alone and continued
        case("long_document", PHI3, "6007", steps=96),
        # the narrower model at batch 8, every step's hidden states kept, caches handed to another node
        case("llama_batch", LLAMA3, "2048,1900,777,2048,1333,512,2047,1601", split="2", steps=96, decode="rows", export=True),
        # decode-heavy serving: 32 ragged contexts in a paged cache
        case("paged_batch32", PHI3, "1088,3310,2045,4096,1515,2900,1024,3777,2222,1801,3001,2608,1192,3499,4001,1333,"
             "2750,1999,3205,1456,3900,2100,2510,1700,3050,1250,3650,2350,1900,2850,4050,1600", steps=128, paged=True),
        # the largest: eight prompts of 8192 tokens and a long generation
        case("long_context", PHI3, "8x8192", steps=1024),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("f32", "general", "small", "model", "model", "model"))
    if kind in ("f32", "general"):
        d = rng.choice((64, 128) if kind == "f32" else (64, 80, 96))
        kv = rng.choice((1, 2, 4))
        shape = {"hidden": 8 * _log(rng, 32, 160), "q_heads": kv * rng.choice((1, 2, 3, 4)), "kv_heads": kv, "head_dim": d,
                 "ffn": 8 * _log(rng, 64, 512), "dtype": "f32" if kind == "f32" else "bf16"}
        batch, top, most = rng.choice((1, 2, 3, 5, 8)), 500, 1000
        steps, room, split = rng.choice((0, 4, 16, 32)), rng.choice((0, 100)), rng.choice(("1", "2"))
        paged, decode, export = False, rng.choice(("reused", "new")), rng.random() < 0.25
    elif kind == "small":
        kv = rng.choice((2, 4))
        shape = {"hidden": 256 * rng.choice((1, 2, 3, 4)), "q_heads": kv * rng.choice((1, 2, 3, 4)), "kv_heads": kv, "head_dim": 128,
                 "ffn": 256 * rng.choice((2, 3, 5, 8)), "dtype": "bf16"}
        batch, top, most = rng.choice((1, 2, 5, 13, 32)), 600, 4000
        steps, room, split = rng.choice((0, 8, 32, 64)), rng.choice((0, 1, 70, 2000)), rng.choice(("1", "2", "3"))
        paged, decode, export = rng.random() < 0.4, rng.choice(("reused", "rows", "noalloc")), rng.random() < 0.25
    else:
        shape = rng.choice((PHI3, LLAMA3))
        batch, top, most = rng.choice((1, 1, 2, 3, 4, 8, 16, 32)), 8192, 40000
        steps, room, split = rng.choice((0, 0, 16, 64, 128)), rng.choice((0, 64, 3000)), rng.choice(("1", "1", "2"))
        paged, decode, export = rng.random() < 0.3, rng.choice(("reused", "reused", "rows", "noalloc")), False
    top = min(top, most // batch)
    mean = _log(rng, 16, top)
    if rng.random() < 0.4:
        lens = [mean] * batch
    else:
        lens = [min(top, max(1, int(mean * rng.uniform(0.3, 1.7)))) for _ in range(batch)]
    return {**shape, "split": split, "prompts": ",".join(str(n) for n in lens), "steps": steps, "room": room, "paged": paged,
            "decode": decode, "export": export and batch * sum(_split({"split": split})) <= 24}


# ---------------------------------------------------------------- inputs
def _split(case):
    return [int(n) for n in case["split"].split(",")]


def _prompts(case):
    lens = []
    for part in case["prompts"].split(","):
        n, _, length = part.rpartition("x")
        lens += [int(length)] * int(n or 1)
    return lens


class _Shape:
    """A block's shape in the attributes that binding.stage_config reads."""

    def __init__(self, case):
        self.hidden, self.n_q_heads, self.n_kv_heads = case["hidden"], case["q_heads"], case["kv_heads"]
        self.head_dim, self.ffn_dim, self.dtype = case["head_dim"], case["ffn"], case["dtype"]
        self.rms_eps, self.rope_base = EPS, ROPE_BASE


def _weight_shapes(case):
    H, I, q, kv = case["hidden"], case["ffn"], case["q_heads"] * case["head_dim"], case["kv_heads"] * case["head_dim"]
    return {"attn_norm_g": (H,), "wq": (q, H), "wk": (kv, H), "wv": (kv, H), "wo": (H, q),
            "ffn_norm_g": (H,), "w_gate": (I, H), "w_up": (I, H), "w_down": (H, I)}


def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _normal(shape, dtype, seed, sigma=1.0, mean=0.0):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).mul_(sigma).add_(mean).to(dtype)


def _layer(case, seed, layer):
    """Weights of one block.  The projections' spread makes a sub-layer's update as large as N(0, 0.02^2) makes it at
    hidden size 5120, so that narrow blocks are more than the identity too."""
    sigma = 0.02 * math.sqrt(5120 / case["hidden"]) if case["hidden"] < 4096 else 0.02
    w = {}
    for t, (name, shape) in enumerate(_weight_shapes(case).items()):
        gain = name.endswith("_g")
        w[name] = _normal(shape, _dtype(case), seed * 4096 + layer * 16 + t, 0.02 if gain else sigma, 1.0 if gain else 0.0)
    return w


def _hidden(case, seed):
    """(prompt rows [T, H], decode inputs [steps, batch, H])"""
    lens, H = _prompts(case), case["hidden"]
    x = _normal((sum(lens), H), _dtype(case), seed * 4096 + 4001)
    xd = _normal((case["steps"], len(lens), H), _dtype(case), seed * 4096 + 4002)
    return x, xd


def prepare(case, seed):
    lens, split = _prompts(case), _split(case)
    shape, batch, cap = _Shape(case), len(lens), max(lens) + case["steps"] + case["room"]
    flags = binding.HYP_FLAG_PAGED_KV if case["paged"] else 0
    bounds = [sum(split[:i]) for i in range(len(split) + 1)]
    if len(split) > 1:
        model = StageChain(shape, bounds, lambda l: _layer(case, seed, l), batch, cap, sum(lens), flags)
    else:
        cfg = binding.stage_config(shape, batch, cap, sum(lens), flags)
        model = binding.stage_create(cfg, 0, split[0], [_layer(case, seed, l) for l in range(split[0])])
    if case["paged"]:
        ppr = -(-((cap + 63) // 64 * 64) // binding.HYP_KV_PAGE_KEYS)
        gen = torch.Generator()
        gen.manual_seed(seed)
        table = torch.randperm(batch * ppr, generator=gen).reshape(batch, ppr).tolist()
        for stage in model.stages if len(split) > 1 else [model]:
            stage.set_page_table(table)
    x, xd = _hidden(case, seed)
    return {"case": case, "model": model, "lens": lens, "x": x, "xd": list(xd),
            "out": torch.empty((batch, case["hidden"]), dtype=x.dtype, device="cuda")}


def run(state):
    case, model, out = state["case"], state["model"], state["out"]
    got = {"prefill": model.prefill(state["x"], state["lens"])}
    if case["steps"]:
        how = case["decode"]
        if how == "new" or isinstance(model, StageChain):  # a chain keeps its own buffers
            steps = [model.decode_step(h).clone() if how != "new" else model.decode_step(h) for h in state["xd"]]
            got["decode"] = torch.stack(steps)
        else:
            rows = torch.empty((case["steps"],) + out.shape, dtype=out.dtype, device=out.device)
            for h, row in zip(state["xd"], rows.unbind()):
                if how == "noalloc":
                    model.decode_step_noalloc(h, row)
                elif how == "rows":
                    model.decode_step(h, row)
                else:
                    row.copy_(model.decode_step(h, out))
            got["decode"] = rows
    if case["export"]:
        kv = [model.export_kv(l, r) for l in range(sum(_split(case))) for r in range(len(state["lens"]))]
        got["k"], got["v"] = torch.cat([k for k, _ in kv]), torch.cat([v for _, v in kv])
    return got


# ---------------------------------------------------------------- what a pass cannot do without
def work(case):
    lens, blocks, steps = _prompts(case), sum(_split(case)), case["steps"]
    es = 2 if case["dtype"] == "bf16" else 4
    H, q, kv = case["hidden"], case["q_heads"] * case["head_dim"], case["kv_heads"] * case["head_dim"]
    params = sum(math.prod(s) for s in _weight_shapes(case).values())
    batch, rows = len(lens), sum(lens)
    past = sum(sum(n + s + 1 for n in lens) for s in range(steps))  # keys seen by all decode queries
    seen = sum(n * (n + 1) // 2 for n in lens) + past               # keys seen by all queries
    total = rows + batch * steps
    weights = params * es * blocks * (1 + steps)                    # a step's input follows from the step before
    io = 2 * total * H * es
    cache = 2 * kv * es * blocks * (total + past)
    export = 2 * kv * es * blocks * 2 * total if case["export"] else 0
    return {"bytes": weights + io + cache + export, "flops": blocks * (2.0 * total * params + 4.0 * q * seen)}


def tolerance(case):
    """About four times the largest error against float64 seen over the listed and sixty drawn cases: float32 2.7e-6 (largest
    single difference 1.6e-5), bf16 7.5e-3 through one block (4.3e-2) and 1.0e-2 .. 1.4e-2 through two to six (7.1e-2)."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 6e-5}
    return {"rel": 0.02, "max": 0.17} if sum(_split(case)) == 1 else {"rel": 0.03, "max": 0.28}


# ---------------------------------------------------------------- the same request in float64
def _norm(x, g):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + EPS) * g


def _rope(x, pos):
    """x [n, heads, d]: element i turned with element i + d / 2 by pos * base^(-2 i / d)"""
    half = x.shape[-1] // 2
    angle = pos[:, None] * (ROPE_BASE ** (-torch.arange(half, device=x.device, dtype=torch.float64) / half))[None]
    c, s = angle.cos()[:, None], angle.sin()[:, None]
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * c - b * s, b * c + a * s], -1)


def _attend(q, k, v, group):
    """Causal attention of one request: q [n, heads, d], k / v [n, kv heads, d]; the query rows in slices that fit memory."""
    n, heads, d = q.shape
    out = torch.empty_like(q)
    at = torch.arange(n, device=q.device)
    step = max(1, min(n, (1 << 26) // n))
    for h in range(heads):
        kh, vh = k[:, h // group].contiguous(), v[:, h // group].contiguous()
        kt = kh.t().contiguous()
        for lo in range(0, n, step):
            hi = min(n, lo + step)
            s = q[lo:hi, h].contiguous() @ kt[:, :hi].contiguous() / math.sqrt(d)
            s.masked_fill_(at[None, :hi] > at[lo:hi, None], -math.inf)
            out[lo:hi, h] = torch.softmax(s, -1) @ vh[:hi]
    return out


def _mm(x, w):
    return x @ w.double().t().contiguous()


def exact(case, seed):
    lens, steps, blocks, H = _prompts(case), case["steps"], sum(_split(case)), case["hidden"]
    heads, kvh, d, batch = case["q_heads"], case["kv_heads"], case["head_dim"], len(lens)
    x, xd = _hidden(case, seed)
    # every request as one causal sequence: its prompt, then its decode inputs
    rows, first = [], 0
    for r, n in enumerate(lens):
        rows.append(torch.cat([x[first:first + n], xd[:, r]]).double())
        first += n
    size = [n + steps for n in lens]
    pos = torch.cat([torch.arange(n, device=x.device, dtype=torch.float64) for n in size])
    h = torch.cat(rows)
    caches_k, caches_v = [], []
    for l in range(blocks):
        p = _layer(case, seed, l)
        y = _norm(h, p["attn_norm_g"].double())
        q = _rope(_mm(y, p["wq"]).reshape(-1, heads, d), pos)
        k = _rope(_mm(y, p["wk"]).reshape(-1, kvh, d), pos)
        v = _mm(y, p["wv"]).reshape(-1, kvh, d)
        caches_k.append(k.reshape(-1, kvh * d))
        caches_v.append(v.reshape(-1, kvh * d))
        a = torch.cat([_attend(qr, kr, vr, heads // kvh) for qr, kr, vr in zip(q.split(size), k.split(size), v.split(size))])
        h = h + _mm(a.reshape(-1, heads * d), p["wo"])
        y = _norm(h, p["ffn_norm_g"].double())
        del q, k, v, a
        up, gate, down = p["w_up"].double().t().contiguous(), p["w_gate"].double().t().contiguous(), p["w_down"].double().t().contiguous()
        for lo in range(0, h.shape[0], 16384):
            s = y[lo:lo + 16384]
            h[lo:lo + 16384] += (torch.nn.functional.silu(s @ gate) * (s @ up)) @ down
    parts = h.split(size)
    got = {"prefill": torch.cat([p[:n] for p, n in zip(parts, lens)])}
    if steps:
        got["decode"] = torch.stack([p[n:] for p, n in zip(parts, lens)], 1)
    if case["export"]:
        got["k"], got["v"] = torch.cat(caches_k), torch.cat(caches_v)
    return got

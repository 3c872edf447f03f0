"""The work that a user of this framework has it do, as cases that can be timed.

``listed()`` names the cases, ``draw(rng)`` draws one more of the same ranges,
``prepare(case, seed)`` makes what a program holds before the call (caches,
plan or fit, alignment map, target cache), ``run(state)`` is one call through
the public entry points, ``exact(case, seed)`` the same outputs in 64 bits by
plain torch, ``work(case)`` the bytes and flops a call cannot do without and
``tolerance(case)`` how far another correct implementation may be from it.

A case is a dict of plain values:
  op          "translate" or "fit"
  sl sh sd sb source layers, KV heads, head_dim, RoPE base
  tl th td tb target layers, KV heads, head_dim, RoPE base
  mix         source layers concatenated per target layer
  tokens      source tokens of each context; batch: contexts per call
  span        largest span of the token alignment (0: same tokenizer)
  dtype       "bf16" or "f32"
  prec        operand precision of a bf16 plan (bf16x2, bf16, f16, bf16x2o)
  page        tokens per block of a paged target cache (0: contiguous)
  outliers    x20 outlier channels per source head
"""
import math
from types import SimpleNamespace

import torch

from paper_2608_30963_amd import kvx

_PREC = {"bf16x2": kvx.KVX_PREC_BF16X2, "bf16": kvx.KVX_PREC_BF16, "f16": kvx.KVX_PREC_F16,
         "bf16x2o": kvx.KVX_PREC_BF16X2_OUTLIER}

# The model pairs of the framework's workloads.
_QWEN = dict(sl=28, sh=4, sd=128, sb=1e6, tl=28, th=2, td=128, tb=1e6, mix=1, span=0, outliers=4)
_GEMMA = dict(sl=28, sh=2, sd=128, sb=1e6, tl=26, th=4, td=256, tb=1e4, mix=1, span=3, outliers=0)
_LLAMA = dict(sl=80, sh=8, sd=128, sb=5e5, tl=28, th=4, td=128, tb=1e6, mix=3, span=2, outliers=4)


def _case(name, op="translate", **kw):
    c = dict(op=op, sl=4, sh=2, sd=64, sb=1e4, tl=4, th=2, td=64, tb=1e4, mix=1, tokens=256,
             batch=1, span=0, dtype="bf16", prec="bf16x2", page=0, outliers=0)
    c.update(kw)
    return {"name": name, **c} if name else c


def listed():
    return [
        # the smallest cache anyone translates: 4 small fp32 layers, the first
        # thing a new user runs
        _case("fp32_tiny_256", dtype="f32"),
        # a translator kept in fp32 (fitted or trained weights before any cast)
        # on a 1K context of the 7B -> 1.5B pair
        _case("fp32_qwen_1k", **dict(_QWEN, outliers=0), dtype="f32", tokens=1024),
        # a bf16 pair whose head_dim (80) the matrix-core tiles do not fit
        _case("bf16_hd80_1k", sl=32, sh=8, sd=80, sb=1e4, tl=24, th=4, td=80, tb=5e5, tokens=1024),
        # a handoff of one short prompt, same tokenizer and other tokenizer
        _case("qwen_128", **_QWEN, tokens=128),
        _case("gemma_128", **_GEMMA, tokens=128),
        # the everyday handoff: one 4K context, same tokenizer
        _case("qwen_4k", **_QWEN, tokens=4096),
        # a serving step: several contexts of an odd length into a paged cache,
        # at the fp16 operand precision
        _case("qwen_paged_1531x4", **dict(_QWEN, outliers=0), tokens=1531, batch=4, page=16,
              prec="f16"),
        # one 4K context across tokenizers, and the batched long-context call
        _case("gemma_4k", **_GEMMA, tokens=4096),
        _case("gemma_8k_x8", **_GEMMA, tokens=8192, batch=8),
        # a large source model, several source layers mixed per target layer
        _case("llama_8k", **_LLAMA, tokens=8192),
        # fitting a translator: accumulate a batch of paired caches and solve
        _case("fit_qwen_4k_x4", op="fit", **_QWEN, tokens=4096, batch=4),
        _case("fit_gemma_1k_x4", op="fit", **_GEMMA, tokens=1021, batch=4),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case.  Each kind is bounded by the work of the listed cases it
    stands beside."""
    by_name = {c["name"]: work(c) for c in listed()}
    bound = {"ident": by_name["qwen_4k"], "span": by_name["gemma_8k_x8"],
             "mixed": by_name["llama_8k"], "general": by_name["fp32_qwen_1k"],
             "fit": by_name["fit_qwen_4k_x4"]}
    kind = rng.choice(["ident", "ident", "span", "span", "mixed", "general", "fit"])
    while True:
        c = dict(sl=rng.randint(4, 40), sh=rng.choice([1, 2, 4, 8]), sd=rng.choice([64, 128, 128]),
                 sb=rng.choice([1e4, 5e5, 1e6]), tl=rng.randint(4, 32),
                 th=rng.choice([1, 2, 4, 8]), td=rng.choice([64, 128, 128, 256]),
                 tb=rng.choice([1e4, 5e5, 1e6]), tokens=_log_int(rng, 16, 16384),
                 batch=rng.choice([1, 1, 1, 2, 3, 8]), outliers=rng.choice([0, 4]),
                 prec=rng.choice(["bf16x2", "bf16x2", "bf16x2", "f16", "bf16x2o"]))
        if kind == "ident":
            c["page"] = rng.choice([0, 0, 16, 64])
        elif kind == "span":
            c["span"] = rng.randint(2, 4)
            c["page"] = rng.choice([0, 0, 0, 16])
        elif kind == "mixed":
            c["mix"] = rng.randint(2, 4)
            c["span"] = rng.choice([0, 2, 3])
        elif kind == "general":
            c["prec"] = "bf16x2"
            c["dtype"] = rng.choice(["f32", "f32", "bf16"])
            if c["dtype"] == "bf16":
                c["sd"], c["td"] = rng.choice([(80, 80), (96, 96), (80, 128)])
            c["outliers"] = 0
            c["span"] = rng.choice([0, 0, 2])
        else:
            c["prec"] = "bf16x2"
            c["span"] = rng.choice([0, 0, 3])
            c["tokens"] = max(c["tokens"], 64)
        c = _case(None, op="fit" if kind == "fit" else "translate", **c)
        din = c["mix"] * c["sh"] * c["sd"]
        if c["prec"] == "f16":
            c["outliers"] = 0
        if kind != "general" and din % 128:
            continue  # the matrix-core path contracts in chunks of 128
        if kind == "fit" and c["tokens"] * c["batch"] < 4 * din * max(1, c["span"]):
            continue  # too few rows to fit that many inputs
        w = work(c)
        if w["bytes"] <= bound[kind]["bytes"] and w["flops"] <= bound[kind]["flops"]:
            return c


def _dims(c):
    return c["mix"] * c["sh"] * c["sd"], c["th"] * c["td"]


def _rows(c):
    """Expected target rows of all contexts."""
    return c["tokens"] * c["batch"] / (1 if not c["span"] else (1 + c["span"]) / 2)


def _layer_map(c):
    """One source layer per target layer, spread evenly; or windows of `mix`."""
    sl, tl, m = c["sl"], c["tl"], c["mix"]
    if m == 1:
        return [min(sl - 1, (2 * l * (sl - 1) + (tl - 1)) // (2 * (tl - 1))) for l in range(tl)]
    return [min(sl - 1, l * sl // tl + j) for l in range(tl) for j in range(m)]


def work(c):
    din, dout = _dims(c)
    rows = _rows(c)
    es = 4 if c["dtype"] == "f32" else 2
    layers = len(set(_layer_map(c)))
    src = 2 * layers * c["batch"] * c["tokens"] * c["sh"] * c["sd"] * es
    tgt = 2 * c["tl"] * rows * dout * es
    csr = rows * 4 + c["tokens"] * c["batch"] * 8 if c["span"] else 0
    if c["op"] == "fit":
        n = din + 1
        gram = 2 * c["tl"] * rows * (n * (n + 1) + 2 * n * dout)
        solve = 2 * c["tl"] * (n ** 3 / 3 + 2 * n * n * dout)
        return {"bytes": src + tgt + csr + 2 * c["tl"] * (din + 1) * dout * 4,
                "flops": gram + solve}
    return {"bytes": src + tgt + csr + 2 * c["tl"] * dout * (din * es + 4),
            "flops": 4 * c["tl"] * rows * din * dout}


def tolerance(c):
    # fit: fp32 sums over the rows and bf16 products split to 2^-16, through
    # well-conditioned normal equations (measured against 64 bits: 6e-6, 3e-5)
    if c["op"] == "fit":
        return {"rel": 5e-5, "max": 5e-4}
    # fp32 sums of up to 1024 products (measured: 4e-7, 4e-6)
    if c["dtype"] == "f32":
        return {"rel": 3e-6, "max": 3e-5}
    # bf16 outputs of nearly exact sums: values at a rounding boundary move by
    # one bf16 step, 2^-8 to 2^-7 of the value (measured against 64 bits, the
    # output rounding alone: 1.66e-3, 3.9e-3)
    if c["prec"] == "bf16x2":
        return {"rel": 2.5e-3, "max": 1.2e-2}
    # operands rounded once to fp16 (measured 1.67e-3, 4.7e-3)
    if c["prec"] == "f16":
        return {"rel": 3e-3, "max": 2e-2}
    # operands (all, or the unmarked channels') rounded once to bf16 (measured
    # 2.3e-3, 1.2e-2 where none is marked)
    return {"rel": 5e-3, "max": 4e-2}


def _spans(c, g):
    """Equal-weight spans of 1..span tokens that partition each context."""
    tt, rp, ci, wt, base = [], [torch.zeros(1, dtype=torch.int64)], [], [], 0
    for _ in range(c["batch"]):
        ln = torch.randint(1, c["span"] + 1, (c["tokens"],), generator=g)
        end = torch.cumsum(ln, 0)
        n = int((end < c["tokens"]).sum()) + 1
        end = torch.clamp(end[:n], max=c["tokens"])
        ln = torch.diff(end, prepend=torch.zeros(1, dtype=torch.int64))
        tt.append(n)
        rp.append(end + base)
        ci.append(torch.arange(c["tokens"]))
        wt.append(torch.repeat_interleave(1.0 / ln.to(torch.float32), ln))
        base += c["tokens"]
    return (tt, torch.cat(rp).to(torch.int32), torch.cat(ci).to(torch.int32), torch.cat(wt))


def _randn(g, shape, dt, scale=1.0):
    """N(0, scale^2) on the GPU in dtype dt, layer by layer."""
    out = torch.empty(shape, dtype=dt, device="cuda")
    for i in range(shape[0]):
        out[i] = torch.randn(shape[1:], generator=g, device="cuda") * scale
    return out


def _inputs(c, seed):
    """Caches, weights and alignment, from the seed alone."""
    g = torch.Generator(device="cuda").manual_seed(seed * 2 + 1)
    gc = torch.Generator().manual_seed(seed * 2 + 1)
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    din, dout = _dims(c)
    s = SimpleNamespace(dt=dt, layer_map=_layer_map(c), marks=[None, None])
    sshape = (c["sl"], c["batch"], c["sh"], c["tokens"], c["sd"])
    s.src = [_randn(g, sshape, dt), _randn(g, sshape, dt)]
    if c["outliers"]:
        for i in range(2):
            pick = torch.rand((c["sl"], c["sh"], c["sd"]), generator=gc).argsort(-1)
            mark = pick < c["outliers"]
            s.marks[i] = mark.numpy()
            s.src[i] *= torch.where(mark, 20.0, 1.0).to(dt).cuda()[:, None, :, None, :]
    if c["span"]:
        s.tt, rp, ci, wt = _spans(c, gc)
        s.rp, s.ci, s.wt = rp.cuda(), ci.cuda(), wt.cuda()
        # room for any draw of the spans: the expected rows and 4 sqrt(tokens),
        # over ten standard deviations
        s.cap = min(c["tokens"], int(2 * c["tokens"] / (1 + c["span"]) +
                                     4 * math.sqrt(c["tokens"])) + 1)
    else:
        s.tt = s.rp = s.ci = s.wt = None
        s.cap = c["tokens"]
    if c["op"] == "fit":
        # the target model's own caches of the same contexts
        tshape = (c["tl"], c["batch"], c["th"], s.cap, c["td"])
        s.native = [_randn(g, tshape, dt), _randn(g, tshape, dt)]
    else:
        s.w = [_randn(g, (c["tl"], dout, din), dt, din ** -0.5) for _ in range(2)]
        s.b = [_randn(g, (c["tl"], dout), torch.float32, 0.1) for _ in range(2)]
    if c["page"]:
        per = -(-s.cap // c["page"])
        s.blocks = c["batch"] * per
        s.table = torch.randperm(s.blocks, generator=gc).to(torch.int32).view(c["batch"], per)
    return s


def prepare(case, seed):
    c = case
    s = _inputs(c, seed)
    src = kvx.ModelShape(c["sl"], c["sh"], c["sd"], c["sb"])
    tgt = kvx.ModelShape(c["tl"], c["th"], c["td"], c["tb"])
    kd = kvx.KVX_F32 if c["dtype"] == "f32" else kvx.KVX_BF16
    if c["op"] == "fit":
        s.fit = kvx.Fitter(src, tgt, c["mix"], s.layer_map, kd)
        return s
    mk, mv = s.marks if c["prec"] == "bf16x2o" else (None, None)
    s.tr = kvx.Translator(src, tgt, c["mix"], s.layer_map, kd, s.w[0], s.w[1], s.b[0], s.b[1],
                          precision=_PREC[c["prec"]], outlier_k=mk, outlier_v=mv)
    s.w = s.b = None  # the plan holds its own copy
    if c["page"]:
        s.table = s.table.cuda()
        tshape = (c["tl"], s.blocks, c["th"], c["page"], c["td"])
    else:
        s.table = None
        tshape = (c["tl"], c["batch"], c["th"], s.cap, c["td"])
    s.tgt = [torch.zeros(tshape, dtype=s.dt, device="cuda") for _ in range(2)]
    s.page = c["page"]
    return s


def run(state):
    s = state
    if hasattr(s, "fit"):
        s.fit.reset()
        s.fit.accumulate(s.src[0], s.src[1], s.native[0], s.native[1], s.tt, s.rp, s.ci, s.wt)
        return s.fit.solve(1.0)
    s.tr(s.src[0], s.src[1], s.tgt[0], s.tgt[1], s.cap, s.tt, s.rp, s.ci, s.wt,
         block_table=s.table, block_size=s.page)
    return s.tgt[0], s.tgt[1]


def _rope(x, pos, base, sign):
    """Rotate-half RoPE of x [..., rows, D] in 64 bits at positions pos [rows]."""
    half = x.shape[-1] // 2
    th = base ** (-2.0 * torch.arange(half, dtype=torch.float64, device=x.device) / x.shape[-1])
    ang = pos.to(torch.float64)[:, None] * th
    cs, sn = torch.cos(ang), sign * torch.sin(ang)
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * cs - b * sn, b * cs + a * sn], -1)


def _pooled(c, s, kv, l, b):
    """Pooled, de-rotated rows z [T_t, din] of target layer l, context b."""
    parts = []
    pos = torch.arange(c["tokens"], device="cuda")
    for j in range(c["mix"]):
        x = s.src[kv][s.layer_map[l * c["mix"] + j], b].double()
        if kv == 0:
            x = _rope(x, pos, c["sb"], -1.0)
        parts.append(x.permute(1, 0, 2).reshape(c["tokens"], -1))
    x = torch.cat(parts, 1)
    if not c["span"]:
        return x
    r0, n = sum(s.tt[:b]), s.tt[b]
    rp = s.rp[r0:r0 + n + 1].long()
    e0, e1 = int(rp[0]), int(rp[-1])
    row = torch.repeat_interleave(torch.arange(n, device="cuda"), torch.diff(rp))
    z = torch.zeros((n, x.shape[1]), dtype=torch.float64, device="cuda")
    return z.index_add_(0, row, x[s.ci[e0:e1].long()] * s.wt[e0:e1].double()[:, None])


def exact(case, seed):
    c = case
    s = _inputs(c, seed)
    din, dout = _dims(c)
    if c["op"] == "fit":
        return _exact_fit(c, s, din, dout)
    out = []
    for kv in range(2):
        t = torch.zeros((c["tl"], c["batch"], c["th"], s.cap, c["td"]), dtype=torch.float64,
                        device="cuda")
        for l in range(c["tl"]):
            w, bias = s.w[kv][l].double(), s.b[kv][l].double()
            for b in range(c["batch"]):
                u = _pooled(c, s, kv, l, b) @ w.t().contiguous() + bias
                u = u.view(-1, c["th"], c["td"]).permute(1, 0, 2)
                if kv == 0:
                    u = _rope(u, torch.arange(u.shape[1], device="cuda"), c["tb"], 1.0)
                t[l, b, :, :u.shape[1]] = u
        if c["page"]:
            pg = torch.zeros((c["tl"], s.blocks, c["th"], c["page"], c["td"]),
                             dtype=torch.float64, device="cuda")
            for b in range(c["batch"]):
                for i in range(s.table.shape[1]):
                    part = t[:, b, :, i * c["page"]:(i + 1) * c["page"]]
                    pg[:, int(s.table[b, i]), :, :part.shape[2]] = part
            t = pg
        out.append(t)
    return tuple(out)


def _exact_fit(c, s, din, dout):
    w = [torch.empty((c["tl"], dout, din), dtype=torch.float64) for _ in range(2)]
    bias = [torch.empty((c["tl"], dout), dtype=torch.float64) for _ in range(2)]
    n = din + 1
    ridge = torch.ones(n, dtype=torch.float64)
    ridge[din] = 0.0  # the bias is not penalised
    for kv in range(2):
        for l in range(c["tl"]):
            gram = torch.zeros((n, n + dout), dtype=torch.float64, device="cuda")
            for b in range(c["batch"]):
                z = _pooled(c, s, kv, l, b)
                y = s.native[kv][l, b, :, :z.shape[0]].double()
                if kv == 0:
                    y = _rope(y, torch.arange(z.shape[0], device="cuda"), c["tb"], -1.0)
                y = y.permute(1, 0, 2).reshape(z.shape[0], dout)
                zt = torch.cat([z, torch.ones_like(z[:, :1])], 1)
                gram += zt.t().contiguous() @ torch.cat([zt, y], 1)
            gram = gram.cpu()
            x = torch.linalg.solve(gram[:, :n] + torch.diag(ridge), gram[:, n:])
            w[kv][l] = x[:din].t()
            bias[kv][l] = x[din]
    return w[0], w[1], bias[0], bias[1]

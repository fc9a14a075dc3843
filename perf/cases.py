"""What the restoration path is timed on: batches that a serving loop hands to `restore_batch`, the
eviction that produces their host blocks (`offload`), and the projections of a layer alone
(`op_gemm`).  Widths are those of the repository's model shapes; models of the large widths are cut
to a few layers (what one pipeline stage holds), so that rounding differences do not travel through
32 layers of 16-bit storage and a case fits beside two others.  Weights are N(0, 0.02), loaded KV
cells and GEMM inputs are drawn at the scale that those weights give them.

A batch is written as texts: "ctx" the context length of each request, "new" the new-turn tokens,
"k" / "cut" the split (tokens below k in layers below cut are recomputed, the rest is loaded).
"""
import math

import numpy as np
import torch

from paper_2604_25080_amd import binding as cf

#          d_model, Q heads, KV heads, head_dim, FFN, vocabulary, rope base, dtype
SHAPES = {
    "tiny": (256, 4, 4, 64, 688, 1000, 10000.0, "f32"),
    "mini-bf16": (512, 8, 2, 128, 1408, 2000, 500000.0, "bf16"),
    "mini64-bf16": (256, 4, 2, 64, 688, 1000, 10000.0, "bf16"),
    "8b": (4096, 32, 8, 128, 14336, 128256, 500000.0, "bf16"),
    "70b-tp8": (8192, 8, 1, 128, 3584, 16032, 500000.0, "bf16"),
}
EPS = 1e-5
KV_STD = 1.28          # of a K or V cell under unit-RMS rows and N(0, 0.02) weights at width 4096


def listed():
    return [
        # the whole float32 model on its own configuration: the smallest call, all latency
        dict(name="tiny f32 turn", do="restore", model="tiny", layers=2, ctx="128,64", new="16,16", k="64,32", cut="2,2"),
        # float32 over ordinary lengths, one request cut by layers, one loaded whole
        dict(name="tiny f32 batch", do="restore", model="tiny", layers=2, ctx="1024,777,300,2048", new="33,64,7,128",
             k="512,777,0,1500", cut="2,1,0,2"),
        # a whole small bf16 model over ragged lengths
        dict(name="mini bf16 ragged", do="restore", model="mini-bf16", layers=3, ctx="331,77,1502,640", new="9,33,1,64",
             k="331,32,517,0", cut="3,3,2,0"),
        # one chat turn: a short cached context is loaded, few new rows walk all weights
        dict(name="8b short turn", do="restore", model="8b", layers=4, ctx="700", new="23", k="0", cut="0"),
        # a batch of chat turns with the split where the host link and the recompute end together
        dict(name="8b chat batch", do="restore", model="8b", layers=4, ctx="4001,2600,3333,517,1024,2048,790,3700",
             new="128,128,128,128,128,128,128,128", k="512,512,512,0,0,0,0,512", cut="4,4,4,0,0,0,0,4"),
        # nothing is cached on the host: every context is prefilled, with the first turns behind it
        dict(name="8b prefill", do="restore", model="8b", layers=4, ctx="8192,3001,1500,700", new="64,201,512,100",
             k="8192,3001,1500,700", cut="4,4,4,4"),
        # one long document, cut by layers: attention over its whole length, upper layers loaded
        dict(name="8b long context", do="restore", model="8b", layers=3, ctx="40960", new="256", k="40960", cut="2"),
        # a tensor-parallel shard of a large model: one KV head, narrow projections
        dict(name="70b shard", do="restore", model="70b-tp8", layers=4, ctx="9000,4096,2777", new="128,128,128",
             k="9000,2048,2777", cut="4,4,3"),
        # one projection alone: QKV of a few rows, gate/up of an ordinary launch, down of a full one
        dict(name="gemm qkv 33 rows", do="gemm", model="8b", which="qkv", rows=33),
        dict(name="gemm gate/up 1000 rows", do="gemm", model="8b", which="gate_up", rows=1000),
        dict(name="gemm down 13389 rows", do="gemm", model="8b", which="down", rows=13389),
        # a request's KV leaves the card for its host block
        dict(name="8b offload", do="offload", model="8b", layers=4, ctx="6001"),
    ]


def _log(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    do = rng.choice(["restore"] * 8 + ["gemm"] * 3 + ["offload"])
    if do == "gemm":
        model = rng.choice(["8b", "8b", "70b-tp8"])
        return dict(do=do, model=model, which=rng.choice(["qkv", "o", "gate_up", "down", "head"]), rows=_log(rng, 1, 13389))
    if do == "offload":
        return dict(do=do, model=rng.choice(["8b", "70b-tp8", "mini-bf16", "tiny"]), layers=rng.randint(2, 4),
                    ctx=str(_log(rng, 32, 16384)))
    model = rng.choice(["tiny", "mini-bf16", "mini64-bf16", "8b", "8b", "8b", "70b-tp8"])
    small = model not in ("8b", "70b-tp8")
    layers = rng.randint(2, 3 if small else 4)
    n_req = _log(rng, 1, 8)
    total = _log(rng, 64, 4000 if small else 12000)
    part = [rng.uniform(0.3, 1.0) for _ in range(n_req)]
    ctx = [max(16, int(total * p / sum(part))) for p in part]
    new = [_log(rng, 1, 256) for _ in ctx]
    plan = rng.choice(["recompute", "load", "tokens", "layers"])
    k, cut = [], []
    for n in ctx:
        if plan == "recompute":
            k.append(n), cut.append(layers)
        elif plan == "load":
            k.append(0), cut.append(0)
        elif plan == "tokens":
            k.append(rng.randint(0, n)), cut.append(layers)
        else:
            k.append(n), cut.append(rng.randint(0, layers))
    text = lambda v: ",".join(str(x) for x in v)  # noqa: E731
    return dict(do=do, model=model, layers=layers, ctx=text(ctx), new=text(new), k=text(k), cut=text(cut))


def _ints(case, key):
    return [int(x) for x in case[key].split(",")]


def _gemm_dims(case):
    """-> N, K, epilogue of one projection (the layer's own: float32 out, or SiLU(gate) * up in bf16)."""
    d, hq, hk, hd, ffn, vocab = SHAPES[case["model"]][:6]
    return {"qkv": ((hq + 2 * hk) * hd, d, cf.EPI_STORE_F32), "o": (d, hq * hd, cf.EPI_STORE_F32),
            "gate_up": (ffn, d, cf.EPI_SILU_MUL), "down": (d, ffn, cf.EPI_STORE_F32),
            "head": (vocab, d, cf.EPI_STORE_F32)}[case["which"]]


class _Desc:
    """The fields `model_desc` reads."""

    def __init__(self, model, layers):
        (self.d_model, self.n_q_heads, self.n_kv_heads, self.head_dim, self.d_ffn, self.vocab, self.rope_base,
         self.dtype) = SHAPES[model]
        self.n_layers, self.rms_eps = layers, EPS


class _Model:
    """Random-init weights, a page pool and a context over them, as a serving process holds them."""

    def __init__(self, model, layers, seed, max_batch, max_tokens, max_positions, n_pages):
        s = self.shape = _Desc(model, layers)
        self.dev = torch.device("cuda:0")
        self.dt = torch.float32 if s.dtype == "f32" else torch.bfloat16
        self.rng = torch.Generator(self.dev)
        self.rng.manual_seed(seed)
        self.weights = _weights(s, self.rng, self.dt, self.dev)
        self.gain = torch.ones(s.d_model, device=self.dev)
        g = self.gain.data_ptr()
        wd = dict(embed=self.weights["embed"].data_ptr(), lm_head=self.weights["lm_head"].data_ptr(), final_norm=g,
                  layers=[dict(attn_norm=g, mlp_norm=g, **{n: t.data_ptr() for n, t in lw.items()})
                          for lw in self.weights["layers"]])
        dtype = cf.CF_F32 if s.dtype == "f32" else cf.CF_BF16
        self.page_elems = 2 * s.n_kv_heads * cf.PAGE_TOKENS * s.head_dim
        self.pool = torch.zeros(layers, n_pages, self.page_elems, dtype=self.dt, device=self.dev)
        self.cache = cf.Cache(self.pool.data_ptr(), self.pool.numel() * self.pool.element_size(), layers,
                              s.n_kv_heads, s.head_dim, dtype)
        desc, opts = cf.model_desc(s), cf.ctx_opts(max_batch, max_tokens, max_positions)
        need = cf.workspace_bytes(desc, opts)
        self.workspace = torch.empty(need + 256, dtype=torch.uint8, device=self.dev)
        self.streams = torch.cuda.Stream(), torch.cuda.Stream()
        torch.cuda.synchronize()
        self.ctx = cf.Ctx(desc, wd, opts, (self.workspace.data_ptr() + 255) // 256 * 256, need,
                          self.streams[0].cuda_stream, self.streams[1].cuda_stream)
        self.logits = torch.zeros(max_batch, s.vocab, device=self.dev)


def _weights(s, rng, dt, dev):
    def mat(rows, cols):
        return torch.empty(rows, cols, dtype=dt, device=dev).normal_(0.0, 0.02, generator=rng)

    qc, nq = (s.n_q_heads + 2 * s.n_kv_heads) * s.head_dim, s.n_q_heads * s.head_dim
    return dict(embed=mat(s.vocab, s.d_model), lm_head=mat(s.vocab, s.d_model),
                layers=[dict(wqkv=mat(qc, s.d_model), wo=mat(s.d_model, nq), w_gate=mat(s.d_ffn, s.d_model),
                             w_up=mat(s.d_ffn, s.d_model), w_down=mat(s.d_model, s.d_ffn))
                        for _ in range(s.n_layers)])


def _tokens(case, seed, key):
    g = np.random.default_rng([seed, 1 if key == "ctx" else 2])
    return [g.integers(0, SHAPES[case["model"]][5], size=n).astype(np.int32) for n in _ints(case, key)]


def _host_block(s, n, seed, i, dt):
    """KV of n tokens in the host layout: [layer][page][K part, V part]."""
    g = torch.Generator("cuda:0")
    g.manual_seed(seed * 1009 + 17 * i + 5)
    pages = -(-n // cf.PAGE_TOKENS)
    return torch.empty(s.n_layers, pages, 2 * s.n_kv_heads * cf.PAGE_TOKENS * s.head_dim, dtype=dt,
                       device="cuda:0").normal_(0.0, KV_STD, generator=g)


def _pinned(t):
    h = torch.empty(t.shape, dtype=t.dtype, pin_memory=True)
    h.copy_(t)
    return h


def _gemm_inputs(case, seed):
    n, k, epi = _gemm_dims(case)
    g = torch.Generator("cuda:0")
    g.manual_seed(seed)
    mat = lambda r, c, std: torch.empty(r, c, dtype=torch.bfloat16, device="cuda:0").normal_(0.0, std, generator=g)  # noqa: E731
    # rows as the norm leaves them, or an MLP activation's scale in front of the down projection
    a = mat(case["rows"], k, 1.0)
    return n, k, epi, a, mat(n, k, 0.02), mat(n, k, 0.02) if epi == cf.EPI_SILU_MUL else None


def prepare(case, seed):
    if case["do"] == "gemm":
        n, k, epi, a, w, w2 = _gemm_inputs(case, seed)
        m = _Model("mini-bf16", 1, 0, 1, 64, 64, 4)         # a projection needs a context of the dtype only
        out = torch.zeros(case["rows"], n, dtype=torch.bfloat16 if epi == cf.EPI_SILU_MUL else torch.float32, device=m.dev)
        return dict(do="gemm", m=m, a=a, w=w, w2=w2, out=out, dims=(case["rows"], n, k, epi))
    ctx = _ints(case, "ctx")
    new = _ints(case, "new") if "new" in case else [0] * len(ctx)
    pages = [-(-(n + m) // cf.PAGE_TOKENS) for n, m in zip(ctx, new)]
    rows = (sum(_ints(case, "k")) if "k" in case else 0) + sum(new)
    m = _Model(case["model"], case["layers"], seed, len(ctx), max(rows, 64), max(n + x for n, x in zip(ctx, new)), sum(pages))
    for i, (n, x) in enumerate(zip(ctx, new)):
        m.cache.alloc(1 + i, n + x)
    if case["do"] == "offload":
        m.pool[:, :pages[0]].copy_(_host_block(m.shape, ctx[0], seed, 0, m.dt))
        host = torch.zeros(m.shape.n_layers, pages[0], m.page_elems, dtype=m.dt, pin_memory=True)
        return dict(do="offload", m=m, host=host, n=ctx[0])
    k, cut = _ints(case, "k"), _ints(case, "cut")
    ct, nt = _tokens(case, seed, "ctx"), _tokens(case, seed, "new")
    blocks = [None if k[i] == n and cut[i] == case["layers"] else _pinned(_host_block(m.shape, n, seed, i, m.dt))
              for i, n in enumerate(ctx)]
    reqs = [dict(req_id=1 + i, ctx_tokens=ct[i], new_tokens=nt[i], host_kv=0 if b is None else b.data_ptr())
            for i, b in enumerate(blocks)]
    splits = [(cf.CF_TOKEN_WISE if c in (0, case["layers"]) else cf.CF_LAYER_WISE, a, c) for a, c in zip(k, cut)]
    return dict(do="restore", m=m, blocks=blocks, reqs=reqs, splits=splits)


def run(s):
    m = s["m"]
    if s["do"] == "gemm":
        rows, n, k, epi = s["dims"]
        ptr, silu = s["out"].data_ptr(), epi == cf.EPI_SILU_MUL
        m.ctx.op_gemm(s["a"].data_ptr(), s["w"].data_ptr(), s["w2"].data_ptr() if silu else 0, 0 if silu else ptr,
                      ptr if silu else 0, rows, n, k, epi)
        return s["out"]
    if s["do"] == "offload":
        m.ctx.offload(m.cache, 1, s["n"], s["host"].data_ptr())
        return s["host"]
    m.ctx.restore_batch(m.cache, s["reqs"], s["splits"], m.logits.data_ptr())
    return dict(logits=m.logits, pages=m.pool)


def _pairs(first, n):
    return n * first + n * (n + 1) / 2


def work(case):
    d, hq, hk, hd, ffn, vocab, _, dt = SHAPES[case["model"]]
    es = 4 if dt == "f32" else 2
    if case["do"] == "gemm":
        n, k, epi = _gemm_dims(case)
        silu = epi == cf.EPI_SILU_MUL
        m = case["rows"]
        return dict(bytes=m * k * 2 + n * k * 2 * (1 + silu) + m * n * (2 if silu else 4), flops=2 * m * n * k * (1 + silu))
    layers, ctx = case["layers"], _ints(case, "ctx")
    cell = 2 * hk * hd * es                                  # KV bytes of a token in a layer
    if case["do"] == "offload":
        return dict(bytes=2 * layers * ctx[0] * cell, flops=0)
    new, k, cut = _ints(case, "new"), _ints(case, "k"), _ints(case, "cut")
    qkv = d * (hq + 2 * hk) * hd
    lin = qkv + hq * hd * d + 3 * d * ffn                    # weights of a layer
    moved, flops = layers * lin * es + vocab * d * es + len(ctx) * vocab * 4, 2 * len(ctx) * vocab * d
    for n, m, kk, c in zip(ctx, new, k, cut):
        kk = kk if c else 0
        moved += (m + kk) * d * es                           # embedding rows
        moved += (n * layers - kk * c) * cell * 2 + (m * layers + kk * c) * cell
        moved += m and layers * n * cell                     # the new turn reads the restored KV
        flops += layers * (2 * m * lin + 4 * hq * hd * _pairs(n, m))
        if kk:                                               # the last recomputed layer ends with its K/V
            flops += (c - 1) * (2 * kk * lin + 4 * hq * hd * _pairs(0, kk)) + 2 * kk * qkv
    return dict(bytes=moved, flops=flops)


def tolerance(case):
    if case["do"] == "offload":
        return "exact"
    dt = SHAPES[case["model"]][-1]
    # Four times what the same inputs showed between two implementations that store in the same types:
    # the matrix-core kernels, the plain FMA kernels and torch in float32 (relative / largest).
    if case["do"] == "gemm":
        # float32 sums over up to 14336 terms in another order: 1.5e-6 / 1.4e-5; a bf16 result changes
        # where such a sum crosses a rounding edge: 7.2e-5, one step of the type at the most
        return dict(rel=3e-4, max=3.2e-2) if case["which"] == "gate_up" else dict(rel=6e-6, max=6e-5)
    if dt == "f32":
        # 7.7e-7 / 2.6e-6 from 64 bits over two layers
        return dict(rel=4e-6, max=2e-5)
    # bf16 storage between the steps of a layer: one rounding that falls the other way moves on
    # through the layers that follow (1e-2 / 5.3e-2 after four)
    return dict(rel=3e-2, max=0.22)


# ------------------------------------------------------------------ the same in 64 bits
def _norm(x):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS)


def _rope(x, pos, base):
    half = x.shape[-1] // 2
    j = torch.arange(half, dtype=torch.float64, device=x.device)
    ang = pos.double()[:, None] * torch.pow(torch.tensor(float(base), dtype=torch.float64, device=x.device), -j / half)[None]
    c, s = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * c - b * s, b * c + a * s], -1)


def _attend(q, k, v, first):
    """q [T, Hq, hd] at positions first.. over k, v [N, Hkv, hd] of positions 0..N-1."""
    t, hq, hd = q.shape
    group = hq // k.shape[1]
    out = torch.empty_like(q)
    step = max(16, int(1e8 // (group * (first + t))))
    for g in range(k.shape[1]):
        kg, vg = k[:, g].contiguous(), v[:, g].contiguous()
        for a in range(0, t, step):
            b = min(t, a + step)
            seen = first + b
            s = q[a:b, g * group:(g + 1) * group].reshape(-1, hd) @ kg[:seen].t() / math.sqrt(hd)
            s = s.view(b - a, group, seen)
            mask = torch.arange(seen, device=q.device)[None] > torch.arange(first + a, first + b, device=q.device)[:, None]
            s.masked_fill_(mask[:, None], -math.inf)
            p = torch.softmax(s, -1).view(-1, seen)
            out[a:b, g * group:(g + 1) * group] = (p @ vg[:seen]).view(b - a, group, hd)
    return out


def _cells(block, s, n):
    """Pages [P, page_elems] -> K, V [n, Hkv, hd]."""
    p = block.shape[0]
    half = s.n_kv_heads * cf.PAGE_TOKENS * s.head_dim
    k = block[:, :half].view(p, s.n_kv_heads, cf.PAGE_TOKENS, s.head_dim).permute(0, 2, 1, 3)
    v = block[:, half:].view(p, s.n_kv_heads, s.head_dim, cf.PAGE_TOKENS).permute(0, 3, 1, 2)
    return (x.reshape(-1, s.n_kv_heads, s.head_dim)[:n].double() for x in (k, v))


def _to_pages(k, v, s):
    n = k.shape[0]
    p = -(-n // cf.PAGE_TOKENS)
    full = torch.zeros(2, p * cf.PAGE_TOKENS, s.n_kv_heads, s.head_dim, dtype=k.dtype, device=k.device)
    full[0, :n], full[1, :n] = k, v
    full = full.view(2, p, cf.PAGE_TOKENS, s.n_kv_heads, s.head_dim)
    return torch.cat([full[0].permute(0, 2, 1, 3).reshape(p, -1), full[1].permute(0, 2, 3, 1).reshape(p, -1)], 1)


def exact(case, seed):
    if case["do"] == "gemm":
        _, _, epi, a, w, w2 = _gemm_inputs(case, seed)
        c = a.double() @ w.double().t()
        return c if epi != cf.EPI_SILU_MUL else c * torch.sigmoid(c) * (a.double() @ w2.double().t())
    s, ctx, dev = _Desc(case["model"], case["layers"]), _ints(case, "ctx"), torch.device("cuda:0")
    dt = torch.float32 if s.dtype == "f32" else torch.bfloat16
    if case["do"] == "offload":
        block = _host_block(s, ctx[0], seed, 0, dt)
        return torch.stack([_to_pages(*_cells(b, s, ctx[0]), s) for b in block])
    rng = torch.Generator(dev)
    rng.manual_seed(seed)
    w = _weights(s, rng, dt, dev)
    new, k, cut = _ints(case, "new"), _ints(case, "k"), _ints(case, "cut")
    k = [a if c else 0 for a, c in zip(k, cut)]
    ct, nt = _tokens(case, seed, "ctx"), _tokens(case, seed, "new")
    hosts = [_host_block(s, n, seed, i, dt) for i, n in enumerate(ctx)]
    look = lambda t: w["embed"][torch.from_numpy(t).long().to(dev)].double()  # noqa: E731
    h = [torch.cat([look(ct[i][:k[i]]), look(nt[i])]) for i in range(len(ctx))]
    pos = [torch.cat([torch.arange(a), torch.arange(n, n + m)]).to(dev) for a, n, m in zip(k, ctx, new)]
    nq, nk = s.n_q_heads * s.head_dim, s.n_kv_heads * s.head_dim
    pages = []
    for l, lw in enumerate(w["layers"]):
        lw = {n: t.double() for n, t in lw.items()}
        here = []
        for i, n in enumerate(ctx):
            x = k[i] if l < cut[i] else 0                    # context rows recomputed in this layer
            rows, at = (h[i], pos[i]) if x else (h[i][k[i]:], pos[i][k[i]:])
            qkv = _norm(rows) @ lw["wqkv"].t()
            q = _rope(qkv[:, :nq].view(-1, s.n_q_heads, s.head_dim), at, s.rope_base)
            kn = _rope(qkv[:, nq:nq + nk].view(-1, s.n_kv_heads, s.head_dim), at, s.rope_base)
            vn = qkv[:, nq + nk:].view(-1, s.n_kv_heads, s.head_dim)
            hk, hv = _cells(hosts[i][l], s, n)
            kc, vc = torch.cat([kn[:x], hk[x:], kn[x:]]), torch.cat([vn[:x], hv[x:], vn[x:]])
            here.append(_to_pages(kc, vc, s))
            go = x if l + 1 < cut[i] else 0                  # those that go on past their K/V
            o = [_attend(q[:go], kc[:go], vc[:go], 0)] if go else []
            o.append(_attend(q[x:], kc, vc, n))
            keep = rows if go else rows[x:]
            y = keep + torch.cat(o).reshape(-1, nq) @ lw["wo"].t()
            z = _norm(y)
            a = z @ lw["w_gate"].t()
            y = y + (a * torch.sigmoid(a) * (z @ lw["w_up"].t())) @ lw["w_down"].t()
            h[i] = y if go else torch.cat([h[i][:k[i]], y])
        pages.append(torch.cat(here))
    last = torch.stack([x[-1] for x in h])
    return dict(logits=_norm(last) @ w["lm_head"].double().t(), pages=torch.stack(pages))

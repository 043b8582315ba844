"""The decoding work that performance is measured on, through the package's public entry points.

A case is one call a serving program makes over and over: a decode step of a compiled graph
(`compile_graph` / `decode_step`), of a graph set (`compile_set` / `decode_step`), several greedy
tokens in one call (`decode_steps`), or a burst of requests through the paged cache
(`serve` / `submit` / `run`).  The listed cases cover batch 1 to 16, dense and mixture-of-experts
layers, head sizes 64 and 128, one to eight query heads per KV head, with and without the per-head
query/key norm, short and long caches, ragged lengths and odd sizes; `draw` gives more of the same
ranges.  Most are a few layers and an output head of a model's shape (a layer's kernels are the
same whichever layer it is); two are whole models of their class.

Weights, gains and cache rows have the distributions the repository's synthetic models use:
N(0, 0.02) matrices, 1 + N(0, 0.02) gains, N(0, 1) cached rows.
"""
import math
import random
from types import SimpleNamespace

import torch

import paper_2512_22219_amd as M

EPS = 1e-6
FUSED = dict(fusion=31, transitive_reduction=1)   # what bench.py compiles with


def _case(name, **kw):
    c = dict(call="step", layers=2, hidden=256, q_heads=4, kv_heads=2, head_dim=64, ffn=688, vocab=1024,
             theta=1e6, batch=1, max_seq=192, kv_lo=128, kv_hi=128, experts=0, top_k=0, expert_ffn=0,
             qk_norm=False, steps=1, page=0, active=0)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the repository's tiny configuration: nothing but latency, the smallest call there is
        _case("tiny batch 1", theta=1e4),
        # a whole 1B-class dense model on a single request: head size 64, a short step where every
        # hop between operators counts (an assistant on one user's stream)
        _case("1B-class batch 1", layers=16, hidden=2048, q_heads=32, kv_heads=8, head_dim=64, ffn=8192,
              vocab=128256, theta=5e5, max_seq=2112, kv_lo=777, kv_hi=777),
        # the benchmark's headline: the whole 8B-shaped model, one request, 1024 cached positions
        _case("8B batch 1", layers=36, hidden=4096, q_heads=32, kv_heads=8, head_dim=128, ffn=12288,
              vocab=151936, max_seq=1088, kv_lo=1024, kv_hi=1024),
        # layers of the 70B shape on one request: the longest weight streams per worker
        _case("70B layers batch 1", layers=6, hidden=8192, q_heads=64, kv_heads=8, head_dim=128, ffn=28672,
              vocab=32000, theta=5e5, max_seq=2112, kv_lo=2048, kv_hi=2048),
        # two requests, four greedy tokens per call, query/key norm, two query heads per KV head: a
        # 2B-class model decoding without a host round trip per token
        _case("2B-class batch 2, 4 tokens", call="steps", steps=4, layers=12, hidden=2048, q_heads=16, kv_heads=8,
              head_dim=128, ffn=6144, vocab=32000, qk_norm=True, batch=2, max_seq=1088, kv_lo=300, kv_hi=1000),
        # three open requests on the batch-4 graph of a graph set: what a lightly loaded server runs
        _case("4B-class set, 3 of 4", call="set", active=3, layers=8, hidden=4096, q_heads=32, kv_heads=8, head_dim=128,
              ffn=8192, vocab=32000, batch=4, max_seq=2112, kv_lo=200, kv_hi=2000),
        # layers of the 8B shape at the benchmark's batch 8 with its ragged cache lengths
        _case("8B layers batch 8", layers=8, hidden=4096, q_heads=32, kv_heads=8, head_dim=128, ffn=14336,
              vocab=32000, theta=5e5, batch=8, max_seq=4160, kv_lo=512, kv_hi=4096),
        # the same layers at the largest batch a graph takes
        _case("8B layers batch 16", layers=8, hidden=4096, q_heads=32, kv_heads=8, head_dim=128, ffn=14336,
              vocab=32000, theta=5e5, batch=16, max_seq=2112, kv_lo=512, kv_hi=2048),
        # mixture-of-experts layers at the benchmark's batch 16: routing, 128 experts, 8 query heads per KV head
        _case("MoE layers batch 16", layers=6, hidden=2048, q_heads=32, kv_heads=4, head_dim=128, ffn=0, vocab=32000,
              batch=16, max_seq=2112, kv_lo=2048, kv_hi=2048, experts=128, top_k=8, expert_ffn=768),
        # the same layers on one request: eight experts' weights per layer, all latency
        _case("MoE layers batch 1", layers=12, hidden=2048, q_heads=32, kv_heads=4, head_dim=128, ffn=0, vocab=32000,
              batch=1, max_seq=1088, kv_lo=1024, kv_hi=1024, experts=128, top_k=8, expert_ffn=768),
        # serving: a burst of eight requests, prompts fed through the paged cache, a few new tokens each
        _case("serving burst of 8", call="serve", steps=16, page=16, layers=8, hidden=2048, q_heads=32, kv_heads=8,
              head_dim=64, ffn=8192, vocab=32000, theta=5e5, batch=8, max_seq=512, kv_lo=0, kv_hi=0),
        # nothing a power of two: five requests, one query head per KV head, ragged everything
        _case("odd sizes batch 5", layers=7, hidden=2056, q_heads=24, kv_heads=24, head_dim=64, ffn=5000, vocab=30011,
              theta=1e4, batch=5, max_seq=1352, kv_lo=3, kv_hi=1351),
    ]


def _log(rng, lo, hi, step=1):
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step)) * step
    return max(lo, min(hi, v))


def draw(rng):
    head_dim = rng.choice([64, 128])
    grp = rng.choice([1, 2, 4, 8])
    batch = rng.choice([1, 1, 2, 3, 4, 5, 6, 7, 8, 11, 13, 16])
    moe = rng.random() < 0.25
    call = rng.choice(["step", "step", "step", "steps", "set", "serve"])
    if call == "set" and batch == 1:
        call = "step"
    c = _case(None, call=call, batch=batch, head_dim=head_dim, theta=rng.choice([1e4, 5e5, 1e6]),
              qk_norm=rng.random() < 0.5)
    c["kv_heads"] = rng.choice([4, 8]) if grp > 1 else rng.choice([8, 16])
    c["q_heads"] = c["kv_heads"] * grp
    c["hidden"] = _log(rng, 512, 4096, 16 if moe else 8)
    c["vocab"] = _log(rng, 1000, 64000)
    if moe:
        c.update(ffn=0, experts=rng.choice([16, 60, 64, 128]), top_k=rng.choice([2, 4, 8]), expert_ffn=_log(rng, 128, 1536, 8))
    else:   # (two to four rows keep their whole input in a workgroup's memory: a shorter one)
        c["ffn"] = _log(rng, 1024, 8192 if batch in (2, 3, 4) or call == "set" else 14336, 8)
    c["max_seq"] = _log(rng, 128, 4096 if batch <= 8 else 2048, 8)
    c["kv_hi"] = c["max_seq"] - 8
    c["kv_lo"] = rng.randrange(0, c["kv_hi"])
    if call == "steps":
        c["steps"] = rng.randrange(2, 5)
    if call == "set":
        c["active"] = rng.randrange(batch // 2 + 1, batch + 1)
    if call == "serve":
        c.update(steps=rng.randrange(6, 17), page=rng.choice([8, 16, 32]), kv_lo=0, kv_hi=0)
        c["max_seq"] = max(64, c["max_seq"] // 32 * 32)
    c["layers"] = 1
    budget = 2.5e9
    one = work(c)["bytes"]
    c["layers"] = 2
    per = max(1.0, work(c)["bytes"] - one)
    c["layers"] = max(1, min(_log(rng, 2, 16), int((budget - one) / per) + 1))
    return c


# ---------------------------------------------------------------------------------- inputs
def _shape(c):
    return SimpleNamespace(n_layers=c["layers"], hidden=c["hidden"], n_q_heads=c["q_heads"], n_kv_heads=c["kv_heads"],
                           head_dim=c["head_dim"], ffn=c["ffn"], vocab=c["vocab"], rms_eps=EPS, rope_theta=c["theta"],
                           batch=c["batch"], max_seq=c["max_seq"], n_experts=c["experts"], top_k=c["top_k"],
                           expert_ffn=c["expert_ffn"], qk_norm=c["qk_norm"])


def _inputs(c, seed):
    """Weights, cache, tokens and positions, from the seed alone."""
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(seed)
    rng = random.Random(seed)

    def mat(*size):
        return torch.empty(size, dtype=torch.bfloat16, device=dev).normal_(0.0, 0.02, generator=gen)

    def gain(n):
        return (1.0 + torch.empty(n, device=dev).normal_(0.0, 0.02, generator=gen)).to(torch.bfloat16)

    H, d, nq, nkv, E, Fe = c["hidden"], c["head_dim"], c["q_heads"], c["kv_heads"], c["experts"], c["expert_ffn"]
    layers = []
    for _ in range(c["layers"]):
        w = {"attn_norm": gain(H), "wqkv": mat((nq + 2 * nkv) * d, H), "wo": mat(H, nq * d), "mlp_norm": gain(H)}
        if c["qk_norm"]:
            w.update(q_norm=gain(d), k_norm=gain(d))
        if E:
            w.update(router=mat(E, H), expert_wgu=mat(E, 2 * Fe, H), expert_wd=mat(E, H, Fe))
        else:
            w.update(wgu=mat(2 * c["ffn"], H), wd=mat(H, c["ffn"]))
        layers.append(w)
    inp = {"embed": mat(c["vocab"], H), "final_norm": gain(H), "lm_head": mat(c["vocab"], H), "layers": layers}
    B = c["batch"]
    if c["call"] == "serve":
        # request b: a prompt and enough new tokens that all requests end with the call's last iteration
        n = c["steps"]
        lens = [n - rng.randrange(0, min(3, n - 1)) for _ in range(B)]
        inp["prompts"] = [[rng.randrange(c["vocab"]) for _ in range(p)] for p in lens]
    else:
        inp["tokens"] = [rng.randrange(c["vocab"]) for _ in range(B)]
        inp["positions"] = [rng.randint(c["kv_lo"], c["kv_hi"]) for _ in range(B)]
        size = (c["layers"], B, nkv, c["max_seq"], d)
        inp["k"] = torch.empty(size, dtype=torch.bfloat16, device=dev).normal_(generator=gen)
        inp["v"] = torch.empty(size, dtype=torch.bfloat16, device=dev).normal_(generator=gen)
    return inp


class _DeviceFloats:
    """A tensor's view of fp32 device memory that `owner` holds (and lives as long as the view)."""

    def __init__(self, owner, ptr, shape):
        self.owner = owner
        self.__cuda_array_interface__ = {"shape": shape, "typestr": "<f4", "data": (ptr, False), "version": 2}


def prepare(case, seed):
    c, dev = case, torch.device("cuda")
    inp = _inputs(c, seed)
    weights = {n: inp[n].data_ptr() for n in ("embed", "final_norm", "lm_head")}
    weights["layers"] = [{n: t.data_ptr() for n, t in w.items()} for w in inp["layers"]]
    s, B, V = _shape(c), c["batch"], c["vocab"]
    st = {"case": c, "inputs": inp}
    if c["call"] == "serve":
        per_request = -(-c["steps"] // c["page"])
        pages = B + B * per_request + 3
        size = (c["layers"], pages, c["kv_heads"], c["page"], c["head_dim"])
        st["pools"] = [torch.zeros(size, dtype=torch.bfloat16, device=dev) for _ in range(2)]
        g = M.compile_graph(s, weights, tuple(p.data_ptr() for p in st["pools"]), greedy_loop=1, serving=1,
                            kv_page_size=c["page"], kv_pages=pages, **FUSED)
        st["graph"] = g
        st["server"] = g.serve(max_requests=1 << 17, max_prompt=c["steps"], max_new=c["steps"])
        st["logits"] = torch.as_tensor(_DeviceFloats(st["server"], st["server"].logits_ptr(), (B, V)), device=dev)
        torch.cuda.synchronize()
        return st
    kv = (inp["k"].data_ptr(), inp["v"].data_ptr())
    st["tok0"] = torch.tensor(inp["tokens"], dtype=torch.int32, device=dev)
    st["pos0"] = torch.tensor(inp["positions"], dtype=torch.int32, device=dev)
    n, active = c["steps"], c["active"] or B
    st["logits"] = torch.zeros((B, V), dtype=torch.float32, device=dev)
    if c["call"] == "steps":
        st["graph"] = M.compile_graph(s, weights, kv, greedy_loop=1, **FUSED)
        st["tok"], st["pos"] = st["tok0"].clone(), st["pos0"].clone()
        st["picked"] = torch.zeros((n, B), dtype=torch.int32, device=dev)
        st["all"] = torch.zeros((n, B, V), dtype=torch.float32, device=dev)
        out = [st["all"], st["picked"]]
    elif c["call"] == "set":
        st["graph"] = M.compile_set(s, weights, kv, **FUSED)
        out = [st["logits"][:active]]
    else:
        st["graph"] = M.compile_graph(s, weights, kv, **FUSED)
        out = [st["logits"]]
    # the updated state: the rows the call appends to the cache
    for b, p in enumerate(inp["positions"][:active]):
        out += [inp["k"][:, b, :, p:p + n], inp["v"][:, b, :, p:p + n]]
    st["out"] = out
    torch.cuda.synchronize()
    return st


def run(st):
    c = st["case"]
    stream = torch.cuda.current_stream().cuda_stream
    if c["call"] == "serve":
        srv, n = st["server"], c["steps"]
        for p in st["inputs"]["prompts"]:
            srv.submit(p, n + 1 - len(p), stream)
        srv.run(n, stream)
        return [st["logits"]]
    if c["call"] == "steps":
        st["tok"].copy_(st["tok0"])
        st["pos"].copy_(st["pos0"])
        st["graph"].decode_steps(c["steps"], st["tok"].data_ptr(), st["pos"].data_ptr(), st["picked"].data_ptr(),
                                 st["logits"].data_ptr(), st["all"].data_ptr(), stream)
    elif c["call"] == "set":
        st["graph"].decode_step(c["active"], st["tok0"].data_ptr(), st["pos0"].data_ptr(), st["logits"].data_ptr(), stream)
    else:
        st["graph"].decode_step(st["tok0"].data_ptr(), st["pos0"].data_ptr(), st["logits"].data_ptr(), stream)
    return st["out"]


# ---------------------------------------------------------------------------------- what a pass needs
def work(case):
    c = case
    H, d, nq, nkv, V, B, E = c["hidden"], c["head_dim"], c["q_heads"], c["kv_heads"], c["vocab"], c["batch"], c["experts"]
    rows = c["active"] or B
    attn = (nq + 2 * nkv) * d * H + H * nq * d
    if E:
        expert = 3 * H * c["expert_ffn"]
        touched = E * (1.0 - (1.0 - c["top_k"] / E) ** rows)   # distinct experts under even routing
        read, used = attn + E * H + touched * expert, attn + E * H + c["top_k"] * expert
    else:
        read = used = attn + 3 * H * c["ffn"]
    if c["call"] == "serve":
        kv = sum(i + 1 for i in range(c["steps"])) / c["steps"]
    else:
        kv = (c["kv_lo"] + c["kv_hi"]) / 2 + (c["steps"] + 1) / 2
    step = 2.0 * (c["layers"] * read + V * H + rows * H) + c["layers"] * rows * 2 * nkv * d * kv * 2 + rows * V * 4.0
    flops = 2.0 * rows * (c["layers"] * used + V * H) + 4.0 * c["layers"] * rows * nq * d * kv
    return {"bytes": step * c["steps"], "flops": flops * c["steps"]}


def tolerance(case):
    # Activations are fp32 and logits come out to a few 1e-6.  What is coarser are the appended
    # cache rows: bf16, so a value on a rounding boundary may go either way (one such element moves
    # a row block by up to 2^-7 of itself), and what is read from that row later follows it.
    # A served request starts from an empty cache: everything hangs on a few such rows (4e-4 measured).
    if case["call"] == "serve":
        return {"rel": 1.7e-3, "max": 4e-2, "differ": 0.0}
    return {"rel": 1e-3, "max": 1.6e-2, "differ": 0.0}


# ---------------------------------------------------------------------------------- 64-bit results
def _mm(x, w):   # x [B][K] f64, w bf16 [N][K]
    return torch.cat([x @ part.double().t() for part in w.split(max(1, (1 << 28) // w.shape[1]))], 1)


def _rms(x, g):
    return x / torch.sqrt(x.square().mean(-1, keepdim=True) + EPS) * g.double()


def _rope(x, pos, theta):   # x [B][heads][d]
    d = x.shape[-1]
    f = theta ** (-2.0 * torch.arange(d // 2, dtype=torch.float64, device=x.device) / d)
    a = (pos.double()[:, None] * f)[:, None, :]
    lo, hi = x[..., : d // 2], x[..., d // 2:]
    return torch.cat([lo * a.cos() - hi * a.sin(), hi * a.cos() + lo * a.sin()], -1)


def _exact_step(c, inp, k, v, tok, pos):
    """Logits of one step; k, v: f64 [layers][B][nkv][rows][d], updated in place with bf16-rounded
    rows.  Also the appended rows before that rounding."""
    nq, nkv, d, B = c["q_heads"], c["kv_heads"], c["head_dim"], tok.shape[0]
    x = inp["embed"][tok.long()].double()
    new_k, new_v = [], []
    at = torch.arange(B, device=x.device)
    seen = torch.arange(k.shape[3], device=x.device)[None, :] <= pos[:, None]
    for l, w in enumerate(inp["layers"]):
        qkv = _mm(_rms(x, w["attn_norm"]), w["wqkv"]).view(B, nq + 2 * nkv, d)
        q, kk, vv = qkv[:, :nq], qkv[:, nq:nq + nkv], qkv[:, nq + nkv:]
        if c["qk_norm"]:
            q, kk = _rms(q, w["q_norm"]), _rms(kk, w["k_norm"])
        q, kk = _rope(q, pos, c["theta"]), _rope(kk, pos, c["theta"])
        new_k.append(kk)
        new_v.append(vv)
        k[l][at, :, pos] = kk.to(torch.float32).to(torch.bfloat16).double()
        v[l][at, :, pos] = vv.to(torch.float32).to(torch.bfloat16).double()
        q = q.reshape(B, nkv, nq // nkv, d)
        o = torch.empty_like(q)
        for b in range(B):
            s = torch.matmul(q[b], k[l, b].transpose(1, 2)) / math.sqrt(d)
            s = s.masked_fill(~seen[b], -math.inf)
            o[b] = torch.matmul(torch.softmax(s, -1), v[l, b])
        x = x + _mm(o.reshape(B, nq * d), w["wo"])
        h = _rms(x, w["mlp_norm"])
        if c["experts"]:
            p = torch.softmax(_mm(h, w["router"]), -1)
            top = torch.sort(p, dim=-1, descending=True, stable=True)
            y = torch.zeros_like(x)
            for b in range(B):
                e, pe = top.indices[b, : c["top_k"]], top.values[b, : c["top_k"]]
                for i, wt in zip(e.tolist(), (pe / pe.sum()).tolist()):
                    gu = _mm(h[b:b + 1], w["expert_wgu"][i])
                    g, u = gu.chunk(2, -1)
                    y[b] += wt * _mm(torch.nn.functional.silu(g) * u, w["expert_wd"][i])[0]
            x = x + y
        else:
            g, u = _mm(h, w["wgu"]).chunk(2, -1)
            x = x + _mm(torch.nn.functional.silu(g) * u, w["wd"])
    return _mm(_rms(x, inp["final_norm"]), inp["lm_head"]), torch.stack(new_k), torch.stack(new_v)


def exact(case, seed):
    c, inp, dev = case, _inputs(case, seed), torch.device("cuda")
    B = c["batch"]
    if c["call"] == "serve":
        size = (c["layers"], B, c["kv_heads"], c["steps"], c["head_dim"])
        k, v = (torch.zeros(size, dtype=torch.float64, device=dev) for _ in range(2))
        tok = torch.tensor([p[0] for p in inp["prompts"]], device=dev)
        for i in range(c["steps"]):
            pos = torch.full((B,), i, dtype=torch.int64, device=dev)
            logits, _, _ = _exact_step(c, inp, k, v, tok, pos)
            pick = logits.argmax(-1).tolist()
            tok = torch.tensor([p[i + 1] if i + 1 < len(p) else t for p, t in zip(inp["prompts"], pick)], device=dev)
        return [logits]
    active, n = c["active"] or B, c["steps"]
    rows = max(inp["positions"]) + n
    k, v = (inp[t][:, :active, :, :rows].double() for t in ("k", "v"))
    tok, pos = (torch.tensor(inp[t][:active], dtype=torch.int64, device=dev) for t in ("tokens", "positions"))
    every, ks, vs = [], [], []
    for _ in range(n):
        logits, nk, nv = _exact_step(c, inp, k, v, tok, pos)
        every.append(logits)
        ks.append(nk)
        vs.append(nv)
        tok, pos = logits.argmax(-1), pos + 1
    out = [torch.stack(every), None] if c["call"] == "steps" else [every[0]]
    nk, nv = torch.stack(ks, 3), torch.stack(vs, 3)   # [layers][B][nkv][n][d]
    for b in range(active):
        out += [nk[:, b], nv[:, b]]
    return out

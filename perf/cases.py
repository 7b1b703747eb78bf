"""The calls that a program compacting an agent's history makes, as cases that can be timed and checked: one layer's
prefill over whole, ragged, short and continued blocks, its decode steps from a single long block to many workers, the
prefix-aware layout, routed layers with 16- and 4-bit experts, and the small fp32 layer as one whole pass.

A case is a dict of plain values: `kind` (the entry point), `layer` (the shape), `blocks` of `lo` .. `hi` tokens (ragged
where they differ; the lengths follow from the case alone), `prior` rows already cached, decode `steps`, `q4` = 4-bit
experts.  Inputs are Gaussian, of the scale that normalised activations and N(0, 0.02) matrices give."""
import math
import random

import torch

from paper_2605_23296_amd import binding as B
from paper_2605_23296_amd.workloads import WORKLOADS, LayerConfig, torch_dtype

LAYERS = {
    "dense": WORKLOADS["dense_8x4096"].layer,    # d 4096, 32 query / 8 KV heads of 128, FFN 14336, bf16
    "routed": WORKLOADS["moe_16x8192"].layer,    # d 2880, 64 / 8 heads of 64, 128 experts of 2880, top-4, bf16
    "tiny": WORKLOADS["tiny_fp32"].layer,        # d 256, fp32 storage
    # a small bf16 layer of widths that no named workload has (head_dim 64, K not a power of two in the FFN)
    "small": LayerConfig(d_model=1024, n_q_heads=16, n_kv_heads=4, head_dim=64, ffn_dim=2816, rope_theta=500000.0, dtype="bf16"),
}
ROOM = 256   # cache rows beyond the prompt: a summary of a few hundred tokens


def _case(name, kind, layer, blocks, lo, hi, prior=0, steps=0, q4=False):
    c = dict(kind=kind, layer=layer, blocks=blocks, lo=lo, hi=hi, prior=prior, steps=steps, q4=q4)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: a whole pass (prefill + 16 steps) of the small fp32 layer, launches and latency
        _case("tiny_fp32_forward", "forward", "tiny", 4, 128, 128, steps=16),
        # a handful of short, odd blocks: the tail of a conversation, the last blocks of a partition
        _case("prefill_short", "prefill", "dense", 5, 61, 517),
        # a 2 k budget of chunked prefill behind 6 k cached rows
        _case("extend_2048", "extend", "dense", 1, 2048, 2048, prior=6144),
        # the headline prefill: a 32 k history in eight blocks of 4 k
        _case("prefill_8x4096", "prefill", "dense", 8, 4096, 4096),
        # the large ragged prefill: 32 blocks of 512 .. 8192 tokens
        _case("prefill_ragged32", "prefill", "dense", 32, 512, 8192),
        # the sequential baseline: one block that spans the whole history
        _case("decode_1x32768", "decode", "dense", 1, 32768, 32768, steps=8),
        # the headline decode: eight workers
        _case("decode_8x4096", "decode", "dense", 8, 4096, 4096, steps=8),
        # a 128 k history, 64 workers
        _case("decode_64x2048", "decode", "dense", 64, 2048, 2048, steps=4),
        # the paper's operating point in its own layout: a 96 k history, 24 workers, each behind its prefix
        _case("prefix_decode_24x4096", "prefix", "dense", 24, 4096, 4096, steps=4),
        # the routed layer: 16 blocks of 8 k, then their decode steps with 16-bit and with 4-bit experts
        _case("routed_prefill_16x8192", "prefill", "routed", 16, 8192, 8192),
        _case("routed_decode_16x8192", "decode", "routed", 16, 8192, 8192, steps=4),
        _case("routed_decode_16x8192_q4", "decode", "routed", 16, 8192, 8192, steps=4, q4=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["forward", "prefill", "prefill", "extend", "decode", "decode", "decode", "prefix", "routed", "routed"])
    if kind == "forward":
        layer = rng.choice(["tiny", "small"])
        hi = _log(rng, 8, 512)
        return _case(None, kind, layer, rng.randint(1, 12), max(1, hi // rng.choice([1, 4])), hi, steps=rng.randint(1, 24))
    if kind == "routed":
        if rng.random() < 0.4:
            blocks, hi = rng.randint(1, 8), _log(rng, 64, 4096)
            return _case(None, "prefill", kind, blocks, max(1, hi // rng.choice([1, 8])), hi)
        blocks, hi = _log(rng, 1, 64), _log(rng, 128, 8192)
        return _case(None, "decode", kind, blocks, max(1, hi // rng.choice([1, 8])), hi, steps=rng.randint(2, 5),
                     q4=rng.random() < 0.5)
    layer = rng.choice(["dense", "dense", "dense", "small"])
    if kind == "prefill":
        hi = _log(rng, 32, 8192)
        blocks = max(1, min(_log(rng, 1, 32), 65536 // hi))
        return _case(None, kind, layer, blocks, max(1, hi // rng.choice([1, 3, 16])), hi)
    if kind == "extend":
        blocks, hi = rng.randint(1, 6), _log(rng, 16, 4096)
        return _case(None, kind, layer, blocks, max(1, hi // rng.choice([1, 4])), hi, prior=_log(rng, 64, 16384))
    if kind == "decode":
        hi = _log(rng, 64, 32768)
        blocks = max(1, min(_log(rng, 1, 80), 131072 // hi))
        return _case(None, kind, layer, blocks, max(1, hi // rng.choice([1, 2, 16])), hi, steps=rng.randint(2, 8))
    hi = _log(rng, 128, 4096)
    return _case(None, kind, "dense", _log(rng, 2, 48) if hi < 2048 else rng.randint(2, 24), max(1, hi // rng.choice([1, 2])),
                 hi, steps=rng.randint(2, 6))


def _lens(case):
    if case["lo"] == case["hi"]:
        return [case["hi"]] * case["blocks"]
    rng = random.Random(case["blocks"] * 1000003 + case["lo"] * 1009 + case["hi"])
    return [rng.randint(case["lo"], case["hi"]) for _ in range(case["blocks"])]


def _cu(lens):
    cu = [0]
    for n in lens:
        cu.append(cu[-1] + n)
    return cu


# FP4 E2M1 values by code (sign in bit 3)
_FP4 = [0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0, -0.0, -0.5, -1.0, -1.5, -2.0, -3.0, -4.0, -6.0]


def _inputs(case, seed):
    """All tensors of a case, drawn on the GPU from the seed alone."""
    lay = LAYERS[case["layer"]]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dt = torch_dtype(lay.dtype)
    d, F, E, Dkv = lay.d_model, lay.ffn_dim, lay.n_experts, lay.Dkv

    def normal(shape, std):
        return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).mul_(std).to(dt)

    w = dict(w_qkv=normal((lay.Dq + 2 * Dkv, d), 0.02), w_o=normal((d, lay.Dq), 0.02),
             g_attn=(1.0 + normal((d,), 0.02).float()).to(dt), g_ffn=(1.0 + normal((d,), 0.02).float()).to(dt))
    if not E:
        w["w_gate_up"], w["w_down"] = normal((2 * F, d), 0.02), normal((d, F), 0.02)
    else:
        w["w_router"] = normal((E, d), 0.02)
        if case["q4"]:
            # 4-bit codes, one scale byte per 32 elements: rms near the 0.02 of the 16-bit weights
            def raw(shape, lo, hi):
                return torch.randint(lo, hi, shape, generator=gen, device="cuda", dtype=torch.uint8)
            w["w_exp_gate_up_q"], w["w_exp_gate_up_s"] = raw((E, 2 * F, d // 2), 0, 256), raw((E, 2 * F, d // 32), 119, 121)
            w["w_exp_down_q"], w["w_exp_down_s"] = raw((E, d, F // 2), 0, 256), raw((E, d, F // 32), 119, 121)
        else:
            w["w_exp_gate_up"] = torch.empty((E, 2 * F, d), dtype=dt, device="cuda")
            w["w_exp_down"] = torch.empty((E, d, F), dtype=dt, device="cuda")
            for e in range(E):
                w["w_exp_gate_up"][e], w["w_exp_down"][e] = normal((2 * F, d), 0.02), normal((d, F), 0.02)

    def rows(n):
        x = torch.randn((n, d), generator=gen, device="cuda", dtype=torch.float32)
        if E:
            # a token leans towards its top_k experts, some experts more popular than others, as a trained router has
            # it: the choice is clear, so that two correct implementations route alike
            pop = torch.randn((E,), generator=gen, device="cuda") * 0.5
            u = torch.rand((n, E), generator=gen, device="cuda").clamp_(1e-12, 1.0 - 1e-6)
            pick = (pop - torch.log(-torch.log(u))).topk(lay.top_k, dim=1).indices
            wr = w["w_router"].float()
            wr = wr / (wr * wr).sum(1, keepdim=True)
            for j in range(lay.top_k):
                x += (11.0 + 0.5 * j) * wr[pick[:, j]]
        return x.to(dt)

    lens, N, S = _lens(case), case["blocks"], case["steps"]
    out = dict(w=w, lens=lens)
    kvstd = 0.02 * math.sqrt(d)   # what a normalised row times a N(0, 0.02) matrix has
    if case["kind"] in ("prefill", "extend", "forward"):
        out["x"] = rows(sum(lens))
    if S:
        out["xd"] = rows(S * N).view(S, N, d)
    if case["kind"] in ("prefill", "forward"):
        base, caps = [0] * N, [n + ROOM for n in lens]
    elif case["kind"] == "extend":
        base = [case["prior"] + 37 * b for b in range(N)]
        caps = [p + n + ROOM for p, n in zip(base, lens)]
    elif case["kind"] == "decode":
        base, caps = lens, [n + ROOM for n in lens]
    else:   # prefix: private tails behind one shared history
        base, caps = [32 + (b % 5) for b in range(N)], [ROOM] * N
        T = sum(lens)
        out["shared"] = [normal((T + 8 - T % 8, Dkv), kvstd).view(-1) for _ in range(2)]
    total = sum((c + 7) // 8 * 8 for c in caps) * Dkv
    fill = kvstd if any(base) else 0.0
    out["base"], out["caps"] = base, caps
    out["kv"] = [normal((total,), fill) for _ in range(2)]
    return out


def _cache(lay, caps, kv, lens):
    c = B.KVCache(lay, caps, "cuda", torch_dtype(lay.dtype))
    c.k[:kv[0].numel()].copy_(kv[0][:c.k.numel()])
    c.v[:kv[1].numel()].copy_(kv[1][:c.v.numel()])
    for b, n in enumerate(lens):
        c.h_len[b] = n
    return c


def prepare(case, seed):
    lay = LAYERS[case["layer"]]
    inp = _inputs(case, seed)
    w, lens, N, S, kind = inp["w"], inp["lens"], case["blocks"], case["steps"], case["kind"]
    dt, d = torch_dtype(lay.dtype), lay.d_model
    layer = B.Layer(lay, w)
    if case["q4"]:
        # the 16-bit copy of the experts that prefill reads: the exact expansion of the same arrays
        for n in ("w_exp_gate_up", "w_exp_down"):
            q = w[n + "_q"]
            w[n] = torch.empty((q.shape[0], q.shape[1], 2 * q.shape[2]), dtype=dt, device="cuda")
            layer.compact_mxfp4_dequant(q, w[n + "_s"], w[n])
        layer = B.Layer(lay, w)
    st = dict(kind=kind, layer=layer, S=S, base=inp["base"], cu=_cu(lens), x=inp.get("x"), xd=inp.get("xd"))
    st["kv"] = _cache(lay, inp["caps"], inp["kv"], inp["base"])
    if kind == "prefix":
        T = sum(lens)
        st["shared"] = _cache(lay, [T], inp["shared"], [T])
        need = layer.prefix_workspace_bytes(N, T, ROOM)
        layer.ws = torch.empty(need, dtype=torch.uint8, device="cuda")
        st["prefix"] = _cu(lens)[1:]
    else:
        layer.ensure_workspace(sum(lens) if kind != "decode" else 0, N, max(inp["caps"]), "cuda")
    if kind in ("prefill", "extend", "forward"):
        st["y"] = torch.empty((sum(lens), d), dtype=dt, device="cuda")
    if S:
        st["yd"] = torch.empty((S, N, d), dtype=dt, device="cuda")
    if kind == "forward":
        st["y_last"] = torch.empty((N, d), dtype=dt, device="cuda")
    torch.cuda.synchronize()
    return st


def run(st):
    """One pass; a pass starts from the cached rows that prepare() left (the rows behind them are written again)."""
    layer, kv, kind = st["layer"], st["kv"], st["kind"]
    for b, n in enumerate(st["base"]):
        kv.h_len[b] = n
    if kind == "prefill":
        layer.compact_prefill(st["cu"], st["x"], kv, st["y"])
        return dict(y=st["y"], k=kv.k, v=kv.v)
    if kind == "extend":
        layer.compact_prefill_extend(st["cu"], st["x"], kv, st["y"])
        return dict(y=st["y"], k=kv.k, v=kv.v)
    if kind == "forward":
        layer.compact_layer_forward(st["cu"], st["x"], st["xd"], kv, st["y"], st["y_last"], st["yd"])
        return dict(y=st["y"], y_last=st["y_last"], yd=st["yd"], k=kv.k, v=kv.v)
    if kind == "decode":
        for s in range(st["S"]):
            layer.compact_decode_step(st["xd"][s], kv, st["yd"][s])
    else:
        for s in range(st["S"]):
            layer.compact_prefix_decode_step(st["xd"][s], st["shared"], st["prefix"], kv, st["yd"][s])
    return dict(yd=st["yd"], k=kv.k, v=kv.v)


def work(case):
    lay, lens, S, N = LAYERS[case["layer"]], _lens(case), case["steps"], case["blocks"]
    es = 2 if lay.dtype == "bf16" else 4
    d, F, kvrow = lay.d_model, lay.ffn_dim, 2 * lay.Dkv
    attn_w = (lay.Dq + 2 * lay.Dkv) * d + d * lay.Dq
    per_ffn = 3 * d * F
    per_row = attn_w + (per_ffn * lay.top_k + lay.n_experts * d if lay.n_experts else per_ffn)

    def weight_bytes(rows):
        if not lay.n_experts:
            return (attn_w + per_ffn) * es
        distinct = lay.n_experts * (1.0 - (1.0 - lay.top_k / lay.n_experts) ** rows)
        return (attn_w + lay.n_experts * d) * es + distinct * per_ffn * (4.25 / 8 if case["q4"] else es)

    nbytes = flops = 0.0
    if case["kind"] in ("prefill", "extend", "forward"):
        T = sum(lens)
        prior = [case["prior"] + 37 * b for b in range(N)] if case["kind"] == "extend" else [0] * N
        pairs = sum(n * (n + 1) / 2 + p * n for n, p in zip(lens, prior))
        nbytes += weight_bytes(T) + (2 * T * d + (sum(prior) + T) * kvrow) * es
        flops += 2.0 * per_row * T + 4.0 * lay.Dq * pairs
    if S:
        base = [32 + (b % 5) for b in range(N)] if case["kind"] == "prefix" else lens
        shared = sum(lens) if case["kind"] == "prefix" else 0
        own = sum(_cu(lens)[1:]) if shared else 0   # every worker attends its whole prefix
        for s in range(S):
            live = sum(n + s + 1 for n in base)
            nbytes += weight_bytes(N) + ((shared + live + N) * kvrow + 2 * N * d) * es
            flops += 2.0 * per_row * N + 4.0 * lay.Dq * (live + own)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # about four times the distance from exact() (fp32: 3e-7 in the norm; bf16: 2 .. 5e-3 in the norm, and the worst
    # of 10^8 elements at 2.7e-2 of the root mean square: storage roundings inside a layer)
    if LAYERS[case["layer"]].dtype == "fp32":
        return {"rel": 1.5e-6, "max": 2e-5}
    return {"rel": 1.5e-2, "max": 0.1}


def exact(case, seed):
    """The same pass in 64 bits, in plain torch."""
    lay = LAYERS[case["layer"]]
    inp = _inputs(case, seed)
    w = {n: t for n, t in inp["w"].items()}
    D = torch.float64
    d, Hq, Hkv, hd, G = lay.d_model, lay.n_q_heads, lay.n_kv_heads, lay.head_dim, lay.n_q_heads // lay.n_kv_heads
    N, S, lens, base, kind = case["blocks"], case["steps"], inp["lens"], inp["base"], case["kind"]
    wd = {n: w[n].to(D) for n in ("w_qkv", "w_o", "g_attn", "g_ffn")}
    if lay.n_experts:
        wd["w_router"] = w["w_router"].to(D)
    else:
        wd["w_gate_up"], wd["w_down"] = w["w_gate_up"].to(D), w["w_down"].to(D)
    table = torch.tensor(_FP4, dtype=D, device="cuda")

    def expert(name, e):
        if not case["q4"]:
            return w[name][e].to(D)
        q = w[name + "_q"][e].long()
        v = table[torch.stack([q & 15, q >> 4], dim=-1)].view(q.shape[0], -1, 32)
        return (v * torch.exp2(w[name + "_s"][e].to(D) - 127.0)[:, :, None]).view(q.shape[0], -1)

    def norm(x, g):
        return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + lay.rms_eps) * g

    def rope(v, pos):   # v [rows, heads, hd]
        f = lay.rope_theta ** (-torch.arange(hd // 2, device="cuda", dtype=D) * 2.0 / hd)
        a = pos.to(D)[:, None, None] * f
        lo, hi = v[..., :hd // 2], v[..., hd // 2:]
        return torch.cat([lo * a.cos() - hi * a.sin(), hi * a.cos() + lo * a.sin()], dim=-1)

    def glu(m, wgu, wdn):
        gu = m @ wgu.t()
        g, u = gu[:, :lay.ffn_dim], gu[:, lay.ffn_dim:]
        return (g * torch.sigmoid(g) * u) @ wdn.t()

    def qkv(x, pos):
        p = norm(x.to(D), wd["g_attn"]) @ wd["w_qkv"].t()
        q, k, v = p.split([lay.Dq, lay.Dkv, lay.Dkv], dim=1)
        return rope(q.reshape(-1, Hq, hd), pos), rope(k.reshape(-1, Hkv, hd), pos), v.reshape(-1, Hkv, hd)

    def attend(q, k, v, first):   # query row i sees rows 0 .. first + i
        o = torch.empty_like(q)
        for h in range(Hq):
            kh, vh = k[:, h // G].contiguous(), v[:, h // G].contiguous()
            for r in range(0, q.shape[0], 2048):
                qs = q[r:r + 2048, h]
                end = first + r + qs.shape[0]
                sc = qs @ kh[:end].t() / math.sqrt(hd)
                seen = torch.arange(end, device="cuda")[None] <= first + r + torch.arange(qs.shape[0], device="cuda")[:, None]
                sc.masked_fill_(~seen, -math.inf)
                o[r:r + 2048, h] = torch.softmax(sc, dim=1) @ vh[:end]
        return o.reshape(-1, lay.Dq)

    def back(x, o):
        return ffn(x.to(D) + o @ wd["w_o"].t())

    def ffn(y):
        m = norm(y, wd["g_ffn"])
        if not lay.n_experts:
            for r in range(0, y.shape[0], 16384):
                y[r:r + 16384] += glu(m[r:r + 16384], wd["w_gate_up"], wd["w_down"])
            return y
        top, idx = (m @ wd["w_router"].t()).topk(lay.top_k, dim=1)
        gate = torch.softmax(top, dim=1)
        for e in idx.unique().tolist():
            r, j = (idx == e).nonzero(as_tuple=True)
            for p in range(0, r.numel(), 16384):
                rr = r[p:p + 16384]
                y[rr] += gate[rr, j[p:p + 16384]][:, None] * glu(m[rr], expert("w_exp_gate_up", e), expert("w_exp_down", e))
        return y

    caps = [(c + 7) // 8 * 8 for c in inp["caps"]]
    offs = [o * lay.Dkv for o in _cu(caps)]
    kflat, vflat = (t.to(D) for t in inp["kv"])
    K = [kflat[offs[b]:offs[b + 1]].view(Hkv, caps[b], hd) for b in range(N)]
    V = [vflat[offs[b]:offs[b + 1]].view(Hkv, hd, caps[b]) for b in range(N)]
    out = {}
    lens_now = list(base)
    if kind in ("prefill", "extend", "forward"):
        cu = _cu(lens)
        y = torch.empty((cu[-1], d), dtype=D, device="cuda")
        for b in range(N):
            x, p, n = inp["x"][cu[b]:cu[b + 1]], base[b], lens[b]
            q, k, v = qkv(x, p + torch.arange(n, device="cuda"))
            K[b][:, p:p + n] = k.transpose(0, 1)
            V[b][:, :, p:p + n] = v.permute(1, 2, 0)
            o = attend(q, K[b][:, :p + n].transpose(0, 1), V[b][:, :, :p + n].permute(2, 0, 1), p)
            y[cu[b]:cu[b + 1]] = o @ wd["w_o"].t() if lay.n_experts else back(x, o)
            lens_now[b] = p + n
        if lay.n_experts:   # the experts once for all blocks
            y = ffn(y + inp["x"].to(D))
        out["y"] = y
        if kind == "forward":
            out["y_last"] = y[[c - 1 for c in cu[1:]]]
    if S:
        if kind == "prefix":
            T = sum(lens)
            cap = (T + 7) // 8 * 8
            sk = inp["shared"][0][:cap * lay.Dkv].view(Hkv, cap, hd)
            sv = inp["shared"][1][:cap * lay.Dkv].view(Hkv, hd, cap)
        first = _cu(lens)[1:] if kind == "prefix" else [0] * N
        yd = torch.empty((S, N, d), dtype=D, device="cuda")
        for s in range(S):
            x = inp["xd"][s]
            q, k, v = qkv(x, torch.tensor([first[b] + lens_now[b] for b in range(N)], device="cuda"))
            o = torch.empty_like(q)
            for b in range(N):
                n = lens_now[b]
                K[b][:, n], V[b][:, :, n] = k[b], v[b]
                kk, vv = K[b][:, :n + 1], V[b][:, :, :n + 1]
                if kind == "prefix":
                    kk = torch.cat([sk[:, :first[b]].to(D), kk], dim=1)
                    vv = torch.cat([sv[:, :, :first[b]].to(D), vv], dim=2)
                for g in range(Hkv):
                    pr = torch.softmax(q[b, g * G:(g + 1) * G] @ kk[g].t() / math.sqrt(hd), dim=1)
                    o[b, g * G:(g + 1) * G] = pr @ vv[g].t()
                lens_now[b] = n + 1
            yd[s] = back(x, o.reshape(N, lay.Dq))
        out["yd"] = yd
    out["k"], out["v"] = kflat, vflat
    return out

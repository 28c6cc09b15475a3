"""The work a user of this framework has it do, as cases that can be timed and checked one by one.

A case is one pass through a decoder weight stack of a few layers (or through a single FFN block) by the
public entry points of the Python binding: plan, stack, load, then `Stack.forward` or `chunked_forward`.
The layers have the sizes of the whole models (8B-shaped dense layers, MoE layers of 128 experts), so a
launch is as large as in a whole stack; few of them keep a case quick to prepare and its output close
enough to the mathematics to be compared.

Keys of a case:
  model    one of MODELS below
  layers   layers of the stack
  tokens   token rows of one forward (a decode step, a batch of sequences, a prompt, a chunk of a prompt)
  tier     0: the plan is made for exactly `tokens` rows and runs by `forward`; > 0: the plan's token
           count, and the rows go through it by `chunked_forward` in trips of that size
  steps    forwards of one pass, each on fresh activations (a decode loop)
  context  > 0: attention over a KV cache that holds this many positions; 0: identity on V
  vocab    > 0: an output head; the logits of the last (or only) token are asked for
  pinned   share of the weight bytes the VRAM budget holds (1: everything; below 1: the rest is streamed)
  graph    the decode mode: the step's launches replayed from a HIP graph where that applies
"""
import math

import torch

from paper_2604_26334_amd import binding as B

DEVICE = "cuda:0"
BLOCK = 32          # weights per fp16 scale

# hidden size, query heads, kv heads, FFN width, experts, selected experts, expert width
MODELS = {
    # one bare FFN block without attention and without a residual (the smallest benchmark configuration)
    "ffn": dict(hidden=1024, n_q_heads=0, n_kv_heads=0, head_dim=0, ffn_inter=2816, no_attn=True, no_residual=True),
    # the 8B-shaped dense stack of the benchmark
    "dense8b": dict(hidden=4096, n_q_heads=32, n_kv_heads=8, head_dim=128, ffn_inter=14336),
    # a dense layer of about a billion weights in 24: widths that are no multiples of 1024
    "dense1b": dict(hidden=2048, n_q_heads=16, n_kv_heads=8, head_dim=128, ffn_inter=5632),
    # the miniature of the tests
    "dense_small": dict(hidden=512, n_q_heads=4, n_kv_heads=2, head_dim=128, ffn_inter=1408),
    # the MoE stack of the benchmark
    "moe": dict(hidden=2048, n_q_heads=32, n_kv_heads=4, head_dim=128, n_experts=128, top_k=8, expert_inter=768),
}
EPS = 1e-6


def _case(name=None, model="dense8b", layers=2, tokens=1, tier=0, steps=1, context=0, vocab=0, pinned=1.0, graph=False):
    c = dict(model=model, layers=layers, tokens=tokens, tier=tier, steps=steps, context=context, vocab=vocab,
             pinned=pinned, graph=graph)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: one token through one FFN block, eight tokens one after the other (launch latency)
        _case("ffn_block_1", "ffn", 1, 1, steps=8),
        # interactive decode, one sequence: the headline of the benchmark, four layers of it
        _case("decode_1", layers=4, tokens=1, steps=4, graph=True),
        # batched decode of a few sequences, and of a full batch
        _case("batch_4", layers=2, tokens=4, steps=4, graph=True),
        _case("batch_64", layers=2, tokens=64, steps=4, graph=True),
        # a short prompt of no round length in the 512-token tier
        _case("prefill_300", layers=2, tokens=300, tier=512),
        # time to first token of a long prompt: the whole call, with the last token's logits
        _case("prefill_2048", layers=2, tokens=2048, tier=2048, vocab=128256),
        # decode at a long context: attention over the cached rows beside the weights
        _case("kv_decode_16k", layers=2, tokens=1, steps=4, context=16000, graph=True),
        # a conversation's next turn: a short prompt over the cache of the turns before, in the 64-token
        # tier (the last chunk is a ragged one), and a long one in the 512-token tier
        _case("kv_chunk_150", layers=2, tokens=150, tier=64, context=4000),
        _case("kv_prefill_1024", layers=2, tokens=1024, tier=512, context=4096),
        # MoE decode under a VRAM budget that holds half of the weights: routed experts cross PCIe
        _case("moe_stream_1", "moe", 2, 1, steps=4, pinned=0.5),
        # MoE batched decode and MoE prefill, everything in VRAM
        _case("moe_16", "moe", 2, 16, steps=2),
        _case("moe_prefill_512", "moe", 1, 512, tier=512),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["ffn", "decode", "batch", "prefill", "kv_decode", "kv_prefill", "moe", "moe_prefill"])
    dense = rng.choice(["dense8b", "dense8b", "dense1b", "dense_small"])
    layers = rng.randint(1, 3)
    if kind == "ffn":
        return _case(None, "ffn", 1, _log_uniform(rng, 1, 300), steps=rng.randint(1, 8))
    if kind == "decode":
        vocab = rng.choice([0, 0, 32000, 50272])
        return _case(None, dense, layers, 1, steps=rng.randint(1, 4), vocab=vocab, pinned=rng.choice([1.0, 1.0, 0.6]),
                     graph=rng.random() < 0.5)
    if kind == "batch":
        return _case(None, dense, layers, _log_uniform(rng, 2, 64), steps=rng.randint(1, 4), graph=rng.random() < 0.5)
    if kind == "prefill":
        n = _log_uniform(rng, 65, 2048)
        tier = rng.choice([t for t in (512, 1024, 2048) if t >= min(n, 512)])
        return _case(None, dense, rng.randint(1, 2), n, tier=tier, vocab=rng.choice([0, 32000]),
                     pinned=rng.choice([1.0, 1.0, 0.7]))
    if kind == "kv_decode":
        return _case(None, dense, rng.randint(1, 2), 1, steps=rng.randint(1, 4), context=_log_uniform(rng, 60, 16000),
                     graph=rng.random() < 0.5)
    if kind == "kv_prefill":
        tier = rng.choice([16, 64, 512, 1024])
        return _case(None, dense, rng.randint(1, 2), _log_uniform(rng, max(2, tier // 2), 2 * tier if tier < 1024 else 1024),
                     tier=tier, context=_log_uniform(rng, 60, 4096))
    if kind == "moe":
        return _case(None, "moe", rng.randint(1, 2), _log_uniform(rng, 1, 64), steps=rng.randint(1, 4),
                     pinned=rng.choice([1.0, 1.0, 0.6]))
    return _case(None, "moe", 1, _log_uniform(rng, 65, 512), tier=512)


# ---------------------------------------------------------------------------------------------------
# inputs


def _cfg(case):
    m = dict(n_experts=0, top_k=0, expert_inter=0, ffn_inter=0, no_attn=False, no_residual=False, rms_eps=EPS)
    m.update(MODELS[case["model"]])
    m["n_layers"] = case["layers"]
    if case["context"]:
        # room for what one pass appends
        m["kv_context"] = -(-(case["context"] + case["tokens"] * case["steps"] + 1) // 64) * 64
        m["kv_context"] = max(m["kv_context"], case["context"] + max(case["tier"], 1) + 64)
    if case["vocab"]:
        m["vocab"] = case["vocab"]
    return m


def _matrices(cfg):
    """(layer, kind, experts or None, N, K) of every weight matrix; a MoE layer's experts as one entry."""
    H, out = cfg["hidden"], []
    for layer in range(cfg["n_layers"]):
        if not cfg["no_attn"]:
            out.append((layer, B.PS_MAT_QKV, None, (cfg["n_q_heads"] + 2 * cfg["n_kv_heads"]) * cfg["head_dim"], H))
            out.append((layer, B.PS_MAT_O, None, H, cfg["n_q_heads"] * cfg["head_dim"]))
        E = cfg["n_experts"] or None
        inter = cfg["expert_inter"] if E else cfg["ffn_inter"]
        out += [(layer, B.PS_MAT_GATE, E, inter, H), (layer, B.PS_MAT_UP, E, inter, H), (layer, B.PS_MAT_DOWN, E, H, inter)]
    if cfg.get("vocab"):
        out.append((cfg["n_layers"], B.PS_MAT_OUT, None, cfg["vocab"], H))
    return out


def _gen(seed, stream, layer=0, kind=0):
    g = torch.Generator(device=DEVICE)
    g.manual_seed((int(seed) * 1000003 + stream * 10007 + layer * 101 + kind) % (1 << 62))
    return g


def _quantised(seed, layer, kind, experts, N, K):
    """(scales fp16 [.., N, K/32], codes u8 [.., N, K]) on the GPU: normal weights of variance 1/K, quantised
    block by block to d (q - 8), d = the block's largest magnitude / 7."""
    g = _gen(seed, 1, layer, kind)
    lead = (experts or 1) * N
    scales = torch.empty(lead, K // BLOCK, dtype=torch.float16, device=DEVICE)
    codes = torch.empty(lead, K, dtype=torch.uint8, device=DEVICE)
    step = max(1, (1 << 26) // K)
    for r in range(0, lead, step):
        n = min(step, lead - r)
        w = torch.randn(n, K // BLOCK, BLOCK, generator=g, device=DEVICE).mul_(K ** -0.5)
        d = (w.abs().amax(dim=2) / 7.0).half()
        scales[r:r + n] = d
        codes[r:r + n] = w.div_(d.float()[:, :, None]).round_().clamp_(-8, 7).add_(8.0).to(torch.uint8).view(n, K)
    shape = (experts, N) if experts else (N,)
    return scales.view(*shape, K // BLOCK), codes.view(*shape, K)


def _activations(case, cfg, seed):
    g = _gen(seed, 2)
    return torch.randn(case["steps"], case["tokens"], cfg["hidden"], generator=g, device=DEVICE).half()


def _kv_rows(case, cfg, seed, layer):
    """Cached K and V rows of one layer, fp16 [n_kv][context][head_dim]."""
    g = _gen(seed, 3, layer)
    kv = torch.randn(2, cfg["n_kv_heads"], case["context"], cfg["head_dim"], generator=g, device=DEVICE).half()
    return kv[0], kv[1]


def _router_logits(case, cfg, seed):
    """Host fp32 [steps][layers][tokens][experts]: N(0, 1) (the framework takes them from its caller)."""
    if not cfg["n_experts"]:
        return None
    g = _gen(seed, 4)
    return torch.randn(case["steps"], cfg["n_layers"], case["tokens"], cfg["n_experts"], generator=g, device=DEVICE).cpu().numpy()


def prepare(case, seed):
    """What a user's program keeps: the stack with its weights (and cache) loaded, and the inputs of one pass."""
    cfg = _cfg(case)
    M = case["tier"] or case["tokens"]
    whole = B.Plan(cfg, 1 << 62, M).summary()
    plan = B.Plan(cfg, int(whole.workspace_bytes + whole.weight_bytes * case["pinned"] + (1 << 20)), M)
    st = B.Stack(plan, DEVICE)
    if case["graph"]:
        st.set_decode_mode(1)
    for layer, kind, experts, N, K in _matrices(cfg):
        scales, codes = (t.cpu().numpy() for t in _quantised(seed, layer, kind, experts, N, K))
        if experts is None:
            st.load_matrix(layer, kind, None, scales, codes)
        else:
            for e in range(experts):
                st.load_matrix(layer, kind, e, scales[e], codes[e])
    appended = []
    if case["context"]:
        for layer in range(cfg["n_layers"]):
            k, v = (t.cpu().numpy() for t in _kv_rows(case, cfg, seed, layer))
            for h in range(cfg["n_kv_heads"]):
                st.load_kv(layer, h, k[h], v[h])
        # the rows the pass appends, in place in the caller's arena: K rows of a head, then its V rows
        arena, cap, hd, n = st.arena.view(torch.float16), cfg["kv_context"], cfg["head_dim"], case["tokens"] * case["steps"]
        for s in sorted((s for s in plan.shards() if s.kind == B.PS_SHARD_KV and s.resident == 1), key=lambda s: (s.layer, s.expert)):
            appended.append(arena.as_strided((2, n, hd), (cap * hd, hd, 1), s.offset // 2 + case["context"] * hd))
    x = _activations(case, cfg, seed)
    logits = torch.empty(case["steps"], case["vocab"], dtype=torch.float16, device=DEVICE) if case["vocab"] else None
    torch.cuda.synchronize()
    return dict(case=case, plan=plan, stack=st, x=x, y=torch.empty_like(x), logits=logits,
                route=_router_logits(case, cfg, seed), appended=appended)


def run(state):
    case, st, x, y, logits, route = (state[k] for k in ("case", "stack", "x", "y", "logits", "route"))
    here = torch.cuda.current_stream()
    st.compute.wait_stream(here)      # the caller's stream hands over the inputs ...
    for t in range(case["steps"]):
        r = None if route is None else route[t]
        if case["context"]:
            st.set_context(case["context"] + t * case["tokens"])
        if case["tier"]:
            B.chunked_forward(st, x[t], y[t], r, logits[t] if logits is not None else None)
        else:
            if logits is not None:
                st.set_logits_out(logits[t], 0, 1)
            st.forward(x[t], y[t], r)
    here.wait_stream(st.compute)      # ... and takes back the results
    out = dict(y=y)
    if logits is not None:
        out["logits"] = logits
    if state["appended"]:
        out["appended"] = state["appended"]
    return out


# ---------------------------------------------------------------------------------------------------
# what a pass cannot do without, and how far two correct implementations may be apart


def work(case):
    cfg = _cfg(case)
    H, M, E = cfg["hidden"], case["tokens"], cfg["n_experts"]
    nbytes = flops = 0.0
    for _layer, kind, experts, N, K in _matrices(cfg):
        rows = 1 if kind == B.PS_MAT_OUT else M
        if experts:
            touched = experts * (1.0 - (1.0 - cfg["top_k"] / experts) ** M)
            nbytes += 0.5625 * N * K * touched
            flops += 2.0 * N * K * M * cfg["top_k"]
        else:
            nbytes += 0.5625 * N * K
            flops += 2.0 * N * K * rows
    nbytes += 4.0 * M * H + 2.0 * case["vocab"] + 4.0 * cfg["n_layers"] * M * E
    if case["context"]:
        pos = case["context"] * M + M * (M + 1) / 2.0     # (token, visible position) pairs of a layer and kv head
        nbytes += cfg["n_layers"] * cfg["n_kv_heads"] * cfg["head_dim"] * 4.0 * (case["context"] + M)
        flops += cfg["n_layers"] * cfg["n_q_heads"] * cfg["head_dim"] * 4.0 * pos
    return dict(bytes=nbytes * case["steps"], flops=flops * case["steps"])


def tolerance(case):
    # fp16 stores between the sub-layers, fp16 weight operands, sums in fp32 and in any order: the outputs of
    # one to four layers measure 2e-4 to 7e-4 from the 64-bit ones; four times that
    return dict(rel=2.5e-3, max=2e-2)


def _rms(x):
    return x * torch.rsqrt(x.square().mean(dim=-1, keepdim=True) + EPS)


def exact(case, seed):
    """The same outputs in 64 bits, by plain torch."""
    cfg = _cfg(case)
    f64 = torch.float64
    L, H, hd, nq, nkv = cfg["n_layers"], cfg["hidden"], cfg["head_dim"], cfg["n_q_heads"], cfg["n_kv_heads"]
    n = case["steps"] * case["tokens"]

    def linear(x, layer, kind, experts, N, K):
        s, c = _quantised(seed, layer, kind, experts, N, K)
        out = torch.empty(x.shape[0], N, dtype=f64, device=DEVICE)
        step = max(1, (1 << 26) // K)
        for r in range(0, N, step):
            w = (c[r:r + step].to(f64) - 8.0).view(-1, K // BLOCK, BLOCK) * s[r:r + step].to(f64)[:, :, None]
            out[:, r:r + step] = x @ w.view(-1, K).t()
        return out

    mats = {(l, k): (l, k, e, N, K) for l, k, e, N, K in _matrices(cfg)}
    x = _activations(case, cfg, seed).to(f64).view(n, H)
    route = _router_logits(case, cfg, seed)
    appended = []
    for layer in range(L):
        h = x
        if not cfg["no_attn"]:
            qkv = linear(_rms(x), *mats[layer, B.PS_MAT_QKV])
            v_new = qkv[:, (nq + nkv) * hd:].view(n, nkv, hd)
            if case["context"]:
                kc, vc = (t.to(f64) for t in _kv_rows(case, cfg, seed, layer))
                q, k_new = qkv[:, :nq * hd].view(n, nq, hd), qkv[:, nq * hd:(nq + nkv) * hd].view(n, nkv, hd)
                a = torch.empty(n, nq, hd, dtype=f64, device=DEVICE)
                seen = torch.arange(case["context"] + n, device=DEVICE)[None, :] <= case["context"] + torch.arange(n, device=DEVICE)[:, None]
                for g in range(nkv):
                    K, V = torch.cat([kc[g], k_new[:, g]]), torch.cat([vc[g], v_new[:, g]])
                    for i in range(g * (nq // nkv), (g + 1) * (nq // nkv)):
                        sc = (q[:, i] @ K.t()) / math.sqrt(hd)
                        a[:, i] = torch.softmax(sc.masked_fill(~seen, -math.inf), dim=1) @ V
                    appended.append(torch.stack([k_new[:, g], v_new[:, g]]))
                a = a.view(n, nq * hd)
            else:
                a = v_new.repeat_interleave(nq // nkv, dim=1).reshape(n, nq * hd)
            h = x + linear(a, *mats[layer, B.PS_MAT_O])
        y = _rms(h)
        if cfg["n_experts"]:
            E, I, top = cfg["n_experts"], cfg["expert_inter"], cfg["top_k"]
            lg = torch.from_numpy(route[:, layer]).to(DEVICE).view(n, E)
            val, idx = torch.topk(lg, top, dim=1)
            wgt = torch.softmax(val.to(f64), dim=1)
            sets = [_quantised(seed, layer, k, E, N, K) for k, N, K in ((B.PS_MAT_GATE, I, H), (B.PS_MAT_UP, I, H), (B.PS_MAT_DOWN, H, I))]
            o = torch.zeros(n, H, dtype=f64, device=DEVICE)
            for e in range(E):
                tok, rank = (idx == e).nonzero(as_tuple=True)
                if tok.numel() == 0:
                    continue
                wg, wu, wd = ((c[e].to(f64) - 8.0).view(c.shape[1], -1, BLOCK).mul(s[e].to(f64)[:, :, None]).view(c.shape[1], -1) for s, c in sets)
                ye = y[tok]
                o.index_add_(0, tok, (torch.nn.functional.silu(ye @ wg.t()) * (ye @ wu.t())) @ wd.t() * wgt[tok, rank][:, None])
        else:
            o = linear(torch.nn.functional.silu(linear(y, *mats[layer, B.PS_MAT_GATE])) * linear(y, *mats[layer, B.PS_MAT_UP]), *mats[layer, B.PS_MAT_DOWN])
        x = o if cfg["no_residual"] else h + o
    out = dict(y=x.view(case["steps"], case["tokens"], H))
    if case["vocab"]:
        last = out["y"][:, case["tokens"] - 1 if case["tier"] else 0]
        out["logits"] = linear(_rms(last), *mats[L, B.PS_MAT_OUT])
    if appended and case["pinned"] >= 1.0:
        out["appended"] = appended
    return out

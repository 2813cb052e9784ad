"""The calls whose speed counts: what a program that serves or trains a long-video layer does with this library, from a
clip of a few frames to the longest context, prefill, training and decode, through the public binding.

`listed()` names twelve cases, `draw(rng)` gives more of the same ranges.  `prepare(case, seed)` makes what such a
program holds before the call, `run(state)` is the call, `work`, `tolerance` and `exact` say what it costs at least,
how far two correct implementations may differ and what 64-bit arithmetic gives.

Inputs follow the recipe of paper_2511_12201_amd/synth.py, drawn on the GPU: frames of 252 visual tokens with a cluster
mean each, then text; a positional code, a bounded key salience, 70 % lazy visual queries pulled to the sink, heads of
different sharpness with head 0 the flattest.  Index lists that a program has in hand (attention, training, decode) are
made here in plain torch from the same scores, so that they do not depend on the library's arithmetic.
"""
from __future__ import annotations

import math

import torch

from paper_2511_12201_amd import binding as ob
from paper_2511_12201_amd import synth

TAU, RECALL, PROBE_BLOCK, BLOCK = 0.08, 0.95, 256, 256
TOK_PER_FRAME = 252
KEPT, SHARE = 0.30, 0.54        # lists in hand: share of visual queries kept, of keys selected by the widest head
                                # (what tau = 0.08 and recall 0.95 come to on these inputs)


def _case(name, kind, tokens, text, *, batch=1, heads=(28, 4), head_dim=128, dtype="bf16", causal=True, **more):
    c = {"kind": kind, "tokens": tokens, "text": text, "batch": batch, "q_heads": heads[0], "kv_heads": heads[1],
         "head_dim": head_dim, "dtype": dtype, "causal": causal, **more}
    return {"name": name, **c} if name else c


def listed():
    return [
        # A question about a four-frame clip: selection and attention in one call; latency and launches count.
        _case("prefill_1k", "prefill", 1072, 64, one_call=True, budget_mode=0),
        # The long video of the benchmark, 256 frames: selection, then attention.
        _case("prefill_64k", "prefill", 65536, 1024, one_call=False, budget_mode=0),
        # Four videos of different lengths in one padded batch, a fixed share of the queries, the largest head's budget.
        _case("select_varlen_8k", "select", 8192, 128, batch=4, budget_mode=1),
        # Scores in hand: another recall target is tried on them, a budget for every head (integers come out).
        _case("lists_32k", "lists", 32768, 512, budget_mode=2),
        # One attention layer of a 64-frame video on lists in hand, ragged length.
        _case("attend_16k", "attend", 16391, 256, per_head=False),
        # The tiny float32 configuration, forward and backward: what a gradient check or a numerics study runs.
        _case("train_f32_1k", "train", 1024, 64, heads=(2, 2), head_dim=64, dtype="f32", per_head=False),
        # Training on short clips: two sequences, narrow heads, a key budget for every head, ragged length.
        _case("train_3k", "train", 3101, 77, batch=2, head_dim=64, per_head=True),
        # The training step of the benchmark: forward and backward of a 128-frame video.
        _case("train_32k", "train", 32768, 512, per_head=False),
        # The block-granular variant, forward and backward, on lists of 256-token blocks.
        _case("block_16k", "block", 16384, 256),
        # One decoded token after a short clip, the heads' lists as they are.
        _case("decode_4k", "decode", 4108, 76, store="lists"),
        # One decoded token after a 512-frame video, lists merged after prefill.
        _case("decode_131k", "decode", 131072, 2048, store="static"),
        # The same for eight sequences at once on the group lists.
        _case("decode_131k_b8", "decode", 131072, 2048, batch=8, store="group"),
    ]


def draw(rng):
    kind = rng.choice(["prefill", "prefill", "select", "lists", "attend", "attend", "train", "train", "train_f32", "block",
                       "decode", "decode"])
    log = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))  # noqa: E731
    hi = {"prefill": 65536, "select": 16384, "lists": 65536, "attend": 32768, "train": 32768, "train_f32": 2048,
          "block": 20000, "decode": 131072}[kind]
    tokens = log({"train_f32": 200, "decode": 700}.get(kind, 400), hi)
    text = max(8, int(tokens * rng.uniform(0.01, 0.08)))
    heads, head_dim = rng.choice([(28, 4), (28, 4), (8, 2), (21, 3)]), rng.choice([128, 128, 64])
    if kind == "train_f32":
        return _case(None, "train", tokens, text, heads=rng.choice([(2, 2), (4, 2)]), head_dim=64, dtype="f32", per_head=False)
    if kind == "prefill":
        return _case(None, kind, tokens, text, heads=heads, head_dim=head_dim, one_call=rng.random() < 0.5,
                     budget_mode=rng.choice([0, 1, 2]))
    if kind == "select":
        return _case(None, kind, tokens, text, heads=heads, head_dim=head_dim, batch=rng.choice([2, 3, 4]),
                     budget_mode=rng.choice([0, 1, 2]))
    if kind == "lists":
        return _case(None, kind, tokens, text, heads=heads, batch=rng.choice([1, 2]), budget_mode=rng.choice([0, 1, 2]))
    if kind in ("attend", "train"):
        batch = rng.choice([1, 2]) if tokens <= 8192 else 1
        return _case(None, kind, tokens, text, heads=heads, head_dim=head_dim, batch=batch, per_head=rng.random() < 0.5,
                     causal=rng.random() < 0.85 or tokens > 16384)
    if kind == "block":
        return _case(None, kind, max(1024, tokens // BLOCK * BLOCK + rng.choice([0, 0, 91])), text, heads=heads, head_dim=head_dim)
    return _case(None, kind, tokens, text, heads=heads, head_dim=head_dim, batch=rng.choice([1, 1, 2, 4, 8]),
                 store=rng.choice(["lists", "static", "group", "compact", "paged"]))


# ------------------------------------------------------------------------------------------------ inputs

def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _dtype(c):
    return torch.bfloat16 if c["dtype"] == "bf16" else torch.float32


def _layer(c, seed):
    """Q [B,Hq,N,D], K, V [B,Hkv,N,D] in the case's type (the recipe of synth.make_layer, drawn on the GPU)."""
    g = _generator(seed)
    B, H, Hkv, N, D = c["batch"], c["q_heads"], c["kv_heads"], c["tokens"], c["head_dim"]
    G, nv = H // Hkv, c["tokens"] - c["text"]
    rand = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
    frame = torch.arange(nv, device="cuda") // TOK_PER_FRAME
    mean = math.sqrt(synth.CLUSTER_VAR) * rand(B, Hkv, -(-nv // TOK_PER_FRAME), D)
    K, V = rand(B, Hkv, N, D), rand(B, Hkv, N, D)
    K[:, :, :nv] += mean[:, :, frame]
    beta = math.sqrt(synth.LOCAL_GAIN * math.sqrt(D))
    omega, theta = rand(D) / synth.WINDOW, 2 * math.pi * torch.rand(D, generator=g, device="cuda")
    phi = math.sqrt(2 / D) * torch.cos(torch.arange(N, device="cuda", dtype=torch.float32)[:, None] * omega + theta)
    K += beta * phi
    norm = K[:, :, 0].norm(dim=-1, keepdim=True)
    u_sink = K[:, :, 0] / norm
    lam = synth.SINK_LOGIT * math.sqrt(D) / norm
    gamma = math.sqrt(synth.SALIENCE_GAIN * math.sqrt(D))
    w = rand(B, Hkv, D)
    w = w - (w * u_sink).sum(-1, keepdim=True) * u_sink
    w = w / w.norm(dim=-1, keepdim=True)
    salience = 2 * torch.rand(B, Hkv, N, 1, generator=g, device="cuda") - 1
    salience[:, :, 0] = 0
    K += gamma * salience * w[:, :, None]
    Q = torch.empty(B, H, N, D, dtype=_dtype(c), device="cuda")
    sharp = synth.head_sharpness(H).tolist()
    for i in range(H):
        q = rand(B, N, D) + gamma * w[:, i // G, None]
        q[:, :nv] += mean[:, i // G, frame]
        lazy = torch.rand(B, N, 1, generator=g, device="cuda") < synth.LAZY_FRACTION
        lazy[:, nv:] = False
        pulled = 0.25 * q + (lam * u_sink)[:, i // G, None] + beta * phi
        Q[:, i] = sharp[i] * torch.where(lazy, pulled, q)
    return Q, K.to(_dtype(c)), V.to(_dtype(c))


def _probe_keys(K, nv):
    return torch.stack([K[..., 0, :].double(), K[..., :nv, :].double().mean(-2)], dim=-2)


def _query_scores(Q, probe, scale):
    """Probability of the active class [B,H,N] in 64 bits."""
    B, H, N, _ = Q.shape
    G = H // probe.shape[1]
    out = torch.empty(B, H, N, dtype=torch.float64, device=Q.device)
    for b in range(B):
        for i in range(H):
            z = (Q[b, i].double() @ probe[b, i // G].T) * scale
            out[b, i] = torch.sigmoid(z[:, 1] - z[:, 0])
    return out


def _key_scores(Q, K, causal, scale, pool_keys=0):
    """Accumulated key scores of the pooled queries [B,H,N] in 64 bits; pool_keys: keys pooled in blocks too."""
    B, H, N, D = Q.shape
    G, step = H // K.shape[1], pool_keys or PROBE_BLOCK
    ends = torch.arange(step, N + step, step, device=Q.device).clamp(max=N)
    width = torch.diff(ends, prepend=ends.new_zeros(1)).double()

    def pooled(x):
        s = torch.nn.functional.pad(x.double(), (0, 0, 0, len(ends) * step - N)).view(len(ends), step, D).sum(1)
        return s / width[:, None]

    cols = ends - 1 if pool_keys else torch.arange(N, device=Q.device)
    out = torch.empty(B, H, len(cols), dtype=torch.float64, device=Q.device)
    for b in range(B):
        for i in range(H):
            k = pooled(K[b, i // G]) if pool_keys else K[b, i // G].double()
            s = pooled(Q[b, i]) @ k.T * scale
            if pool_keys:
                s += width.log()
            if causal:
                s = s.masked_fill(cols[None] >= ends[:, None], -math.inf)
            out[b, i] = width @ torch.softmax(s, -1)
    return out * (len(ends) / N) if pool_keys else out


def _kurtosis(a):
    d = a - a.mean(-1, keepdim=True)
    return (d ** 4).mean(-1) / (d * d).mean(-1) ** 2 - 3


def _budgets(a, recall, mode, total):
    """(budget [B] or [B,H], kurtosis, recall of every head) for scores a [B,H,N] of `total` mass a head."""
    need = float(torch.tensor(recall, dtype=torch.float32)) * total
    mass = a.sort(-1, descending=True).values.cumsum(-1)
    own = (mass < need).sum(-1).clamp(max=a.shape[-1] - 1) + 1
    kurt = _kurtosis(a)
    budget = own if mode == 2 else own.amax(-1) if mode == 1 else own.gather(1, kurt.argmin(-1, keepdim=True))[:, 0]
    per_head = budget if mode == 2 else budget[:, None].expand_as(own)
    return budget.int(), kurt, mass.gather(-1, per_head[..., None].long() - 1)[..., 0] / total


def _ascending(member):
    """Index lists [.., N] int32 (ascending, zeros behind) and their lengths of a membership array [.., N]."""
    n = member.shape[-1]
    order = torch.where(member, torch.arange(n, device=member.device), n).sort(-1).values
    return torch.where(order < n, order, 0).int(), member.sum(-1).int()


def _top(a, count):
    """Membership of the count[..] largest entries of a [.., N]."""
    order = torch.sort(a, dim=-1, descending=True, stable=True).indices
    taken = torch.arange(a.shape[-1], device=a.device) < count[..., None]
    return torch.zeros_like(a, dtype=torch.bool).scatter_(-1, order, taken)


def _lists(c, Q, K, scale):
    """Lists that a program has in hand: (q_idx, q_cnt, kv_idx, budget)."""
    B, H, N, nv = c["batch"], c["q_heads"], c["tokens"], c["tokens"] - c["text"]
    s = _query_scores(Q, _probe_keys(K, nv), scale)
    keep = torch.ones(B, H, N, dtype=torch.bool, device="cuda")
    keep[:, 1:, :nv] = _top(s[:, 1:, :nv], torch.full((B, H - 1), math.ceil(KEPT * nv), device="cuda"))
    b = torch.tensor([math.ceil(s * N) for s in _shares(c)], device="cuda").expand(B, H)
    kv_idx, _ = _ascending(_top(_key_scores(Q, K, c["causal"], scale), b))
    return (*_ascending(keep), kv_idx, (b if c.get("per_head") else b[:, 0]).int().contiguous())


def _shares(c):
    """Share of the keys that each head selects: one budget, or one that falls from head to head."""
    H = c["q_heads"]
    return [SHARE * 0.25 ** (i / (H - 1)) if c.get("per_head") else SHARE for i in range(H)]


def _lengths(c):
    """Tokens and visual tokens of the sequences of a padded batch: from the whole length down to a third of it."""
    n = [c["tokens"] - (2 * c["tokens"] // 3) * b // max(1, c["batch"] - 1) for b in range(c["batch"])]
    return n, [x - min(c["text"], x // 4) for x in n]


def _decode_inputs(c, seed):
    g = _generator(seed)
    B, H, Hkv, N, D = c["batch"], c["q_heads"], c["kv_heads"], c["tokens"], c["head_dim"]
    G, nv, dt = H // Hkv, c["tokens"] - c["text"], _dtype(c)
    rand = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
    K = torch.empty(B, Hkv, N + 64, D, dtype=dt, device="cuda")
    V = torch.empty_like(K)
    for b in range(B):
        K[b], V[b] = rand(Hkv, N + 64, D), rand(Hkv, N + 64, D)
    probe = torch.stack([torch.stack([K[b, :, 0].float(), K[b, :, :nv].float().mean(1)], 1) for b in range(B)])
    q = rand(B, H, D)
    lazy = torch.rand(B, H, 1, generator=g, device="cuda") < synth.LAZY_FRACTION
    sink = probe[:, :, 0].repeat_interleave(G, 1)
    pulled = 0.25 * q + synth.SINK_LOGIT * math.sqrt(D) * sink / (sink * sink).sum(-1, keepdim=True)
    q = torch.where(lazy, pulled, q) * torch.from_numpy(synth.head_sharpness(H)).cuda()[:, None]
    salience = torch.rand(B, Hkv, nv, generator=g, device="cuda").repeat_interleave(G, 1)
    member = torch.empty(B, H, nv, dtype=torch.bool, device="cuda")
    for b in range(B):     # the heads of a group pick nearly the same keys
        member[b] = _top(salience[b] + 0.08 * rand(H, nv), torch.full((H,), math.ceil(SHARE * nv), device="cuda"))
    ctx = torch.full((B,), N + 17, dtype=torch.int32, device="cuda")
    return dict(q=q.to(dt), K=K, V=V, probe=probe, member=member, ctx=ctx)


# ------------------------------------------------------------------------------------------------ the calls

def prepare(case, seed):
    c = case
    B, H, Hkv, N, D = c["batch"], c["q_heads"], c["kv_heads"], c["tokens"], c["head_dim"]
    nv, i32, f32 = N - c["text"], torch.int32, torch.float32
    new = lambda *s, dtype=f32: torch.zeros(*s, dtype=dtype, device="cuda")  # noqa: E731
    st = {"case": dict(c)}
    if c["kind"] == "decode":
        x = _decode_inputs(c, seed)
        st.update(x, ddesc=ob.make_decode_desc(x["q"], x["K"], 0, nv, TAU, static_lists=c["store"] == "static"),
                  O=torch.empty_like(x["q"]), active=new(B, H, dtype=torch.uint8))
        member = st.pop("member")
        if c["store"] in ("lists", "static"):
            st["vis_idx"], st["vis_cnt"] = (t.contiguous() for t in _ascending(member))
            if c["store"] == "static":
                st["ws"] = ob.Workspace()
                ob.omni_slim_decode_prepare(st["ddesc"], st["vis_idx"], st["vis_cnt"], nv, ws=st["ws"])
            return st
        bits = (member.view(B, Hkv, H // Hkv, nv).long() << torch.arange(H // Hkv, device="cuda")[:, None]).sum(2)
        st["grp_idx"], st["grp_cnt"] = _ascending(bits > 0)
        st["grp_mask"] = bits.gather(-1, st["grp_idx"].long()).int()
        if c["store"] == "compact":
            st["Kc"], st["Vc"] = ob.omni_compact_cache(st["ddesc"], st["K"], st["V"], st["grp_idx"], st["grp_cnt"])
        elif c["store"] == "paged":
            rows = 256
            per = -(-nv // rows)
            table = torch.randperm(B * Hkv * per, generator=_generator(seed + 1), device="cuda").view(B, Hkv, per).int()
            pages = new(2, B * Hkv * per, rows, D, dtype=_dtype(c))
            st["pool"] = ob.make_page_pool(pages[0], pages[1], table)
            ob.omni_compact_cache_paged(st["ddesc"], st["K"], st["V"], st["grp_idx"], st["grp_cnt"], st["pool"])
        return st

    Q, K, V = _layer(c, seed)
    desc = ob.make_layer_desc(Q, K, 0, nv, 0, c["causal"])
    scale = desc.softmax_scale
    st.update(Q=Q, K=K, V=V, desc=desc)
    if c["kind"] in ("attend", "train", "block"):
        st["q_idx"], st["q_cnt"], st["kv_idx"], st["budget"] = _lists(c, Q, K, scale)
    if c["kind"] in ("prefill", "attend", "train", "block"):
        st["O"], st["lse"] = torch.empty_like(Q), new(B, H, N)
    if c["kind"] in ("train", "block"):
        st["dO"] = torch.empty_like(Q)
        g = _generator(seed + 1)
        for i in range(H):
            st["dO"][:, i] = torch.randn(B, N, D, generator=g, device="cuda") / math.sqrt(D)
        st["dQ"], st["dK"], st["dV"] = torch.empty_like(Q), torch.empty_like(K), torch.empty_like(V)
    if c["kind"] == "prefill":
        b = ob.BudgetResult(new(B, H, N), new(B, H, dtype=torch.float64), new(B, dtype=i32),
                            new(*((B, H) if c["budget_mode"] == 2 else (B,)), dtype=i32), new(B, H))
        st["out"] = ob.SelectionResult(new(B, Hkv, 2, D), new(B, H, N), new(B, H, N, dtype=i32), new(B, H, dtype=i32), b,
                                       new(B, H, N, dtype=i32))
    if c["kind"] == "lists":
        st["scores"] = _query_scores(Q, _probe_keys(K, nv), scale).float()
        st["key_scores"] = _key_scores(Q, K, c["causal"], scale).float()
        st["q_idx"], st["q_cnt"], st["kv_idx"] = new(B, H, N, dtype=i32), new(B, H, dtype=i32), new(B, H, N, dtype=i32)
        del st["Q"], st["K"], st["V"]
    if c["kind"] == "block":
        st["bdesc"] = ob.block_level_desc(desc, BLOCK)
        st["blk_idx"] = new(B, H, -(-N // BLOCK), dtype=i32)
    return st


def run(s):
    c = s["case"]
    return {"prefill": _run_prefill, "select": _run_select, "lists": _run_lists, "attend": _run_attend, "train": _run_train,
            "block": _run_block, "decode": _run_decode}[c["kind"]](c, s)


def _run_prefill(c, s):
    d, Q, K, V, mode = s["desc"], s["Q"], s["K"], s["V"], c["budget_mode"]
    if c["one_call"]:
        out, O, lse = ob.omni_sparse_prefill(d, Q, K, V, 0, TAU, RECALL, PROBE_BLOCK, mode, out=s["out"], O=s["O"], lse=s["lse"])
    else:
        out = ob.omni_prefill_select(d, Q, K, 0, TAU, RECALL, PROBE_BLOCK, mode, out=s["out"])
        attend = ob.omni_sparse_attn_fwd_per_head if mode == 2 else ob.omni_sparse_attn_fwd
        O, lse = attend(d, Q, K, V, out.q_idx, out.q_cnt, out.kv_idx, out.budget.budget, c["tokens"], s["O"], s["lse"])
    b = out.budget
    return {"O": O, "lse": lse, "probe_keys": out.probe_keys, "scores": out.scores, "key_scores": b.key_scores,
            "kurtosis": b.kurtosis, "recall": b.recall}


def _run_select(c, s):
    n, nv = _lengths(c)
    out = ob.omni_prefill_select_varlen(s["desc"], s["Q"], s["K"], n, [0] * len(n), nv, 1, KEPT, RECALL, PROBE_BLOCK,
                                        c["budget_mode"])
    b = out.budget     # rows beyond a sequence's length are unspecified
    return {"probe_keys": out.probe_keys, "scores": [out.scores[i, :, :x] for i, x in enumerate(n)], "q_cnt": out.q_cnt,
            "key_scores": [b.key_scores[i, :, :x] for i, x in enumerate(n)], "kurtosis": b.kurtosis, "recall": b.recall}


def _run_lists(c, s):
    d, N, mode = s["desc"], c["tokens"], c["budget_mode"]
    q_idx, q_cnt = ob.omni_select_queries(d, s["scores"], 0, TAU, s["q_idx"], s["q_cnt"])
    b = ob.omni_budget_from_scores(d, s["key_scores"], RECALL, mode)
    select = ob.omni_select_kv_per_head if mode == 2 else ob.omni_select_kv
    kv_idx = select(d, s["key_scores"], b.budget, N, s["kv_idx"])
    return {"q_idx": q_idx, "q_cnt": q_cnt, "kv_idx": kv_idx, "budget": b.budget, "flattest": b.flattest,
            "kurtosis": b.kurtosis, "recall": b.recall}


def _run_attend(c, s):
    attend = ob.omni_sparse_attn_fwd_per_head if c["per_head"] else ob.omni_sparse_attn_fwd
    O, lse = attend(s["desc"], s["Q"], s["K"], s["V"], s["q_idx"], s["q_cnt"], s["kv_idx"], s["budget"], c["tokens"],
                    s["O"], s["lse"])
    return {"O": O, "lse": lse}


def _run_train(c, s):
    out = _run_attend(c, s)
    back = ob.omni_sparse_attn_bwd_per_head if c["per_head"] else ob.omni_sparse_attn_bwd
    dQ, dK, dV = back(s["desc"], s["Q"], s["K"], s["V"], s["O"], s["dO"], s["lse"], s["q_idx"], s["q_cnt"], s["kv_idx"],
                      s["budget"], c["tokens"], s["dQ"], s["dK"], s["dV"])
    return {**out, "dQ": dQ, "dK": dK, "dV": dV}


def _run_block(c, s):
    d, Q, K, V = s["desc"], s["Q"], s["K"], s["V"]
    a = ob.omni_block_scores(d, Q, K, BLOCK)
    b = ob.omni_budget_from_scores(s["bdesc"], a, RECALL)
    blocks = ob.omni_select_kv(s["bdesc"], a, b.budget, s["blk_idx"].shape[-1], s["blk_idx"])
    O, lse = ob.omni_block_attn_fwd(d, Q, K, V, s["q_idx"], s["q_cnt"], blocks, b.budget, BLOCK, s["O"], s["lse"])
    dQ, dK, dV = ob.omni_block_attn_bwd(d, Q, K, V, O, s["dO"], lse, s["q_idx"], s["q_cnt"], blocks, b.budget, BLOCK,
                                        s["dQ"], s["dK"], s["dV"])
    return {"block_scores": a, "recall": b.recall, "O": O, "lse": lse, "dQ": dQ, "dK": dK, "dV": dV}


def _run_decode(c, s):
    d, q, K, V, ctx, probe = s["ddesc"], s["q"], s["K"], s["V"], s["ctx"], s["probe"]
    if c["store"] in ("lists", "static"):
        O, active = ob.omni_slim_decode(d, q, K, V, ctx, probe, s["vis_idx"], s["vis_cnt"], s["vis_idx"].shape[-1], s["O"],
                                        s["active"], ws=s.get("ws"))
        return {"O": O, "active": active}
    grp = s["grp_idx"], s["grp_mask"], s["grp_cnt"]
    if c["store"] == "group":
        O, active = ob.omni_slim_decode_grouped(d, q, K, V, ctx, probe, *grp, s["O"], s["active"])
    elif c["store"] == "compact":
        O, active = ob.omni_slim_decode_compact(d, q, K, V, ctx, probe, s["Kc"], s["Vc"], *grp, s["O"], s["active"])
    else:
        O, active = ob.omni_slim_decode_paged(d, q, K, V, ctx, probe, s["pool"], *grp, s["O"], s["active"])
    return {"O": O, "active": active}


# ------------------------------------------------------------------------------------------------ what it costs at least

def work(case):
    """Bytes in and out, and the contractions on the (query, key) pairs of the lists, of one pass."""
    c = case
    B, H, Hkv, N, D = c["batch"], c["q_heads"], c["kv_heads"], c["tokens"], c["head_dim"]
    nv, e = N - c["text"], 2 if c["dtype"] == "bf16" else 4
    q_bytes, kv_bytes, row = B * H * N * D * e, 2 * B * Hkv * N * D * e, B * H * N * 4
    if c["kind"] == "decode":
        # rows of the union of the active heads' lists (a group of seven has an active head nine times in ten)
        rows = c["text"] + 17 + (1 - synth.LAZY_FRACTION ** (H // Hkv)) * (SHARE + 0.06) * nv
        lists = {"lists": 0.35 * H * SHARE * nv * 4}.get(c["store"], Hkv * (SHARE + 0.06) * nv * 8)
        return {"bytes": B * (Hkv * rows * 2 * D * e + lists + 2 * H * D * e), "flops": B * H * rows * 4.0 * D * 0.5}
    if c["kind"] == "lists":
        return {"bytes": 4 * row, "flops": 0.0}
    keep = 1 + (H - 1) * (KEPT * nv / N + c["text"] / N)                  # kept rows of all heads, in units of N
    pooled = 2.0 * B * H * -(-N // PROBE_BLOCK) * N * D / (2 if c["causal"] else 1)
    select = {"bytes": q_bytes + kv_bytes / 2 + 4 * row, "flops": pooled + 4.0 * B * H * N * D}
    if c["kind"] == "select":
        part = sum(_lengths(c)[0]) / (B * N)
        return {k: v * part for k, v in select.items()}
    share = sum(_shares(c)) / H if c["kind"] != "block" else 0.85
    pairs = B * keep * N * share * N / (2 if c["causal"] else 1)
    fwd = {"bytes": q_bytes * (1 + keep / H) + kv_bytes + row, "flops": 4.0 * D * pairs}
    if c["kind"] == "attend":
        return fwd
    if c["kind"] == "prefill":
        return {"bytes": fwd["bytes"] + select["bytes"], "flops": fwd["flops"] + select["flops"]}
    return {"bytes": fwd["bytes"] + q_bytes * (1 + 3 * keep / H) + 2 * kv_bytes + row, "flops": fwd["flops"] * 3.5}


def tolerance(case):
    """About four times the distance from 64-bit results measured on these inputs."""
    c = case
    if c["kind"] == "lists":
        return {"rel": 1e-7}                       # kurtosis and recall (2e-8 off); the lists, counts and budgets are exact
    if c["kind"] == "select" or c["dtype"] == "f32":
        return {"rel": 1e-5}                       # key scores 3e-6 off, float32 gradients 2e-6
    if c["kind"] == "prefill":
        return {"rel": 7e-3, "max": 0.9}           # a key at the cut may change sides: the rows that look at it move
    if c["kind"] in ("attend", "decode"):
        return {"rel": 7e-3}                       # O in bf16 is 1.7e-3 off
    return {"rel": 2.2e-2}                         # dQ is 5.5e-3 off


# ------------------------------------------------------------------------------------------------ 64-bit results

def _exact_attention(c, s, kv_lists, per_head_budget, gradients):
    """O, lse (and dQ, dK, dV) on the lists of the state, in 64 bits, one head at a time."""
    Q, K, V, scale = s["Q"], s["K"], s["V"], s["desc"].softmax_scale
    B, H, N, D = Q.shape
    G = H // K.shape[1]
    zeros = lambda x: torch.zeros(x.shape, dtype=torch.float64, device="cuda")  # noqa: E731
    O, lse = zeros(Q), torch.full((B, H, N), -math.inf, dtype=torch.float64, device="cuda")
    dQ, dK, dV = (zeros(Q), zeros(K), zeros(V)) if gradients else (None, None, None)
    for b in range(B):
        for i in range(H):
            rows, cols = s["q_idx"][b, i, :s["q_cnt"][b, i]].long(), kv_lists[b, i, :per_head_budget[b, i]].long()
            k, v = K[b, i // G, cols].double(), V[b, i // G, cols].double()
            for r in rows.split(2048):
                q = Q[b, i, r].double()
                z = q @ k.T * scale
                if c["causal"]:
                    z.masked_fill_(cols[None] > r[:, None], -math.inf)
                m = torch.logsumexp(z, -1)
                p = torch.exp(z.sub_(torch.where(m > -math.inf, m, 0.0)[:, None]))
                O[b, i, r], lse[b, i, r] = p @ v, m
                if gradients:
                    g = s["dO"][b, i, r].double()
                    dV[b, i // G].index_add_(0, cols, p.T @ g)
                    ds = p.mul_(g @ v.T - (g * O[b, i, r]).sum(-1, keepdim=True)) * scale
                    dQ[b, i, r] = ds @ k
                    dK[b, i // G].index_add_(0, cols, ds.T @ q)
    out = {"O": O, "lse": lse}
    return {**out, "dQ": dQ, "dK": dK, "dV": dV} if gradients else out


def exact(case, seed):
    c = case
    s = prepare(c, seed)
    B, H, N, D = c["batch"], c["q_heads"], c["tokens"], c["head_dim"]
    nv = N - c["text"]
    if c["kind"] == "decode":
        return _exact_decode(c, seed)
    scale = s["desc"].softmax_scale
    if c["kind"] == "lists":
        _, kurt, recall = _budgets(s["key_scores"].double(), RECALL, c["budget_mode"], N)
        return {**dict.fromkeys(["q_idx", "q_cnt", "kv_idx", "budget", "flattest"]), "kurtosis": kurt, "recall": recall}
    if c["kind"] == "prefill":
        probe, a = _probe_keys(s["K"], nv), _key_scores(s["Q"], s["K"], c["causal"], scale)
        _, kurt, recall = _budgets(a, RECALL, c["budget_mode"], N)
        return {"O": None, "lse": None, "probe_keys": probe, "scores": _query_scores(s["Q"], probe, scale), "key_scores": a,
                "kurtosis": kurt, "recall": recall}
    if c["kind"] == "select":
        n, n_vis = _lengths(c)
        probe = torch.cat([_probe_keys(s["K"][b:b + 1, :, :x], v) for b, (x, v) in enumerate(zip(n, n_vis))])
        scores = [_query_scores(s["Q"][b:b + 1, :, :x], probe[b:b + 1], scale)[0] for b, x in enumerate(n)]
        a = [_key_scores(s["Q"][b:b + 1, :, :x], s["K"][b:b + 1, :, :x], c["causal"], scale) for b, x in enumerate(n)]
        got = [_budgets(x, RECALL, c["budget_mode"], x.shape[-1]) for x in a]
        return {"probe_keys": probe, "scores": scores, "q_cnt": None, "key_scores": [x[0] for x in a],
                "kurtosis": torch.cat([x[1] for x in got]), "recall": torch.cat([x[2] for x in got])}
    if c["kind"] == "block":
        a = _key_scores(s["Q"], s["K"], c["causal"], scale, pool_keys=BLOCK)
        budget, _, recall = _budgets(a, RECALL, 0, a.shape[-1])
        member = _top(a, budget[:, None].expand(B, H).long()).repeat_interleave(BLOCK, -1)[..., :N]
        kv, count = _ascending(member)
        return {"block_scores": a, "recall": recall, **_exact_attention(c, s, kv, count, True)}
    budget = s["budget"] if c["per_head"] else s["budget"][:, None].expand(B, H)
    return _exact_attention(c, s, s["kv_idx"], budget, c["kind"] == "train")


def _exact_decode(c, seed):
    x = _decode_inputs(c, seed)
    B, H, D, nv = c["batch"], c["q_heads"], c["head_dim"], c["tokens"] - c["text"]
    G, scale = H // c["kv_heads"], D ** -0.5
    O = torch.empty(B, H, D, dtype=torch.float64, device="cuda")
    for b in range(B):
        for i in range(H):
            q, n = x["q"][b, i].double(), int(x["ctx"][b])
            z = x["probe"][b, i // G].double() @ q * scale
            seen = torch.ones(n, dtype=torch.bool, device="cuda")
            seen[:nv] = x["member"][b, i] if i == 0 or float(torch.sigmoid(z[1] - z[0])) > TAU else False
            p = torch.softmax((x["K"][b, i // G, :n][seen].double() @ q) * scale, -1)
            O[b, i] = p @ x["V"][b, i // G, :n][seen].double()
    return {"O": O, "active": None}

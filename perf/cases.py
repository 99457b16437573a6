"""Performance cases of the pruning stage: what a serving program has this library do, over its range.

A serving program keeps one context, the parameter block, the output buffers and the workspace of a
shape, and calls the library once per batch with the batch's queries, keys, hidden states and caches:

  stage       the whole stage as one call (asap_stage), contiguous K/V caches
  paged       the single calls with a block-table cache (asap_score, asap_select, asap_positions,
              asap_compact_kv_paged on a second stream, asap_merge)
  attention   the attention forward of a layer in front of the pruning layer under the salience mask

Shapes are the workloads of paper_2603_14549_amd/synth.py and tests/ plus odd sizes between them.  Inputs
follow the same recipe as synth.py (cluster mixture, projections, RoPE), drawn on the GPU.
"""
from __future__ import annotations

import math

import torch

from paper_2603_14549_amd import binding as A
from paper_2603_14549_amd import harness

# hidden size, query heads, key/value heads, head dim
_7B = dict(D=4096, H=32, Hkv=32, d=128)
_GQA = dict(D=3584, H=28, Hkv=4, d=128)
_13B = dict(D=5120, H=40, Hkv=40, d=128)
_SMALL = dict(D=1024, H=16, Hkv=16, d=128)
_SMALL_GQA = dict(D=768, H=8, Hkv=2, d=128)
_SMALL_64 = dict(D=512, H=8, Hkv=8, d=64)
_MODELS = [_7B, _GQA, _13B, _SMALL, _SMALL_GQA, _SMALL_64]

_BF16 = dict(qk="bf16", h="bf16", kv="bf16")
_F32 = dict(qk="f32", h="f32", kv="f32")
_F32_KV16 = dict(qk="f32", h="f32", kv="bf16")

_TDTYPE = {"bf16": torch.bfloat16, "f32": torch.float32}


def _case(name, kind, model, types, B, P, V, Tmax, k, layers, clusters, **kw):
    c = dict(name=name, kind=kind, **model, **types, B=B, P=P, V=V, Tmax=Tmax, k=k, layers=layers, clusters=clusters,
             text_lo=Tmax, outliers=False, rows="all", route="absorb", mask=True, page=0)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: one 576-token image through a small model, where launches count
        _case("small_576", "stage", _SMALL, _BF16, 1, 35, 576, 32, 144, 2, 48),
        # one 576-token image in full precision, interactive use
        _case("single_576_f32", "stage", _7B, _F32, 1, 35, 576, 32, 144, 2, 48),
        # one high-resolution image (2304 tokens), interactive use
        _case("single_2304", "stage", _7B, _BF16, 1, 35, 2304, 64, 320, 2, 192, outliers=True),
        # a full-precision evaluation batch with ragged prompts
        _case("ragged_576_b16_f32", "stage", _7B, _F32_KV16, 16, 35, 576, 128, 144, 2, 48, text_lo=16),
        # large dynamic-resolution images, grouped-query model, small batch
        _case("gqa_4096_b4", "stage", _GQA, _BF16, 4, 0, 4096, 48, 512, 2, 256),
        # first of two pruning stages of a larger model
        _case("first_of_two_2304_b8", "stage", _13B, _BF16, 8, 0, 2304, 64, 576, 2, 192, outliers=True),
        # the second, with the K/V caches of 16 layers to compact
        _case("second_of_two_576_b8", "stage", _13B, _BF16, 8, 0, 576, 64, 160, 16, 192, outliers=True),
        # throughput serving, the headline workload
        _case("serving_2304_b16", "stage", _7B, _BF16, 16, 35, 2304, 64, 320, 2, 192, outliers=True),
        # ranking by the last text token, sizes that divide nothing, ragged prompts
        _case("last_token_2083_b5", "stage", _GQA, _BF16, 5, 7, 2083, 57, 301, 2, 160, text_lo=9, rows="last"),
        # the consolidation inside the kept set instead of absorption
        _case("paper_route_2304_b16", "stage", _7B, _BF16, 16, 35, 2304, 64, 320, 2, 192, outliers=True,
              route="paper"),
        # paged caches (serving engine with block tables), odd sizes, ragged prompts
        _case("paged_1225_b6", "paged", _GQA, _BF16, 6, 35, 1225, 77, 203, 4, 96, text_lo=12, page=16),
        # one layer's attention forward under the salience mask at the headline shape
        _case("attention_2304_b16", "attention", _7B, _BF16, 16, 35, 2304, 64, 320, 0, 192, outliers=True),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    most = {"stage": work(listed()[7]), "attention": work(listed()[11])}
    most["paged"] = most["stage"]
    while True:
        kind = rng.choices(["stage", "paged", "attention"], [0.7, 0.15, 0.15])[0]
        model = rng.choices(_MODELS, [4, 2, 2, 1, 1, 1])[0]
        types = rng.choices([_BF16, _F32, _F32_KV16], [6, 1, 2])[0]
        V = _log_int(rng, 128, 4096)
        if rng.random() < 0.5:
            V = max(128, V // 64 * 64)                      # whole grids are as common as odd sizes
        Tmax = _log_int(rng, 4, 128)
        c = _case("", kind, model, types, _log_int(rng, 1, 16), rng.choice([0, 5, 35, rng.randint(0, 64)]), V, Tmax,
                  max(8, int(V * rng.uniform(0.08, 0.4))), rng.choice([1, 2, 2, 4, 16]), max(4, V // rng.choice([8, 12, 16])))
        c["outliers"] = rng.random() < 0.5
        c["text_lo"] = rng.choice([Tmax, max(1, Tmax // 8)])
        if kind == "stage":
            c["rows"] = rng.choices(["all", "last"], [5, 1])[0]
            c["route"] = rng.choices(["absorb", "paper"], [5, 1])[0]
            c["mask"] = rng.random() < 0.9
        elif kind == "paged":
            c["page"] = rng.choice([16, 32, 64])
        else:
            c["layers"] = 0
            c["mask"] = rng.random() < 0.8
        del c["name"]
        w = work(c)
        if w["bytes"] <= most[kind]["bytes"] and w["flops"] <= most[kind]["flops"]:
            return c


# ---------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------
_CTX = None


def _context():
    global _CTX
    if _CTX is None:
        _CTX = A.Context(torch.cuda.current_device())
    return _CTX


def _params(c):
    return A.make_params(c["B"], c["H"], c["Hkv"], c["d"], c["D"], c["P"], c["V"], c["Tmax"], c["k"], c["qk"], c["h"],
                         c["kv"], sim_threshold=0.8 if c["route"] == "paper" else float("-inf"),
                         mask_mode=A.ASAP_MASK_KEYBIAS if c["mask"] else A.ASAP_MASK_OFF,
                         route=A.ASAP_ROUTE_PAPER if c["route"] == "paper" else A.ASAP_ROUTE_ABSORB,
                         score_rows=A.ASAP_ROWS_LAST if c["rows"] == "last" else A.ASAP_ROWS_ALL)


def _rope(x, theta=10000.0):
    n, d = x.shape[-2:]
    freq = theta ** (-2.0 * torch.arange(d // 2, device=x.device, dtype=torch.float64) / d)
    ang = torch.arange(n, device=x.device, dtype=torch.float64)[:, None] * freq
    cos, sin = ang.cos().float(), ang.sin().float()
    a, b = x[..., :d // 2], x[..., d // 2:]
    return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)


def _hidden_and_qk(c, g):
    """Hidden states [B,N,D] (prefix and text N(0,1), visual tokens a cluster mixture, every 64th scaled by 8
    when there are outliers) and their projected, rotated queries and keys."""
    B, P, V, T, D, H, Hkv, d = (c[x] for x in ("B", "P", "V", "Tmax", "D", "H", "Hkv", "d"))
    N = P + V + T
    rn = lambda *s: torch.randn(*s, generator=g, device="cuda")
    wt = torch.bfloat16 if c["qk"] == "bf16" else torch.float32
    wq, wk = (rn(D, H * d) / math.sqrt(D)).to(wt), (rn(D, Hkv * d) / math.sqrt(D)).to(wt)
    hidden = torch.empty(B, N, D, dtype=_TDTYPE[c["h"]], device="cuda")
    q = torch.empty(B, H, N, d, dtype=_TDTYPE[c["qk"]], device="cuda")
    k = torch.empty(B, Hkv, N, d, dtype=_TDTYPE[c["qk"]], device="cuda")
    for b in range(B):
        x = rn(N, D)
        which = torch.randint(c["clusters"], (V,), generator=g, device="cuda")
        x[P:P + V] = rn(c["clusters"], D)[which] + 0.3 * x[P:P + V]
        if c["outliers"]:
            x[P:P + V:64] *= 8.0
        hidden[b] = x
        xw = x.to(wt)
        q[b] = _rope((xw @ wq).float().view(N, H, d).transpose(0, 1))
        k[b] = _rope((xw @ wk).float().view(N, Hkv, d).transpose(0, 1))
    return hidden, q, k


def _salience(c, q, k):
    """Eq. 2-3 for the attention case, whose caller has the layer's salience in hand."""
    P, V, G = c["P"], c["V"], c["H"] // c["Hkv"]
    out = torch.empty(c["B"], V, dtype=torch.float32, device="cuda")
    for b in range(c["B"]):
        qs = q[b, :, P:P + V].float().sum(1).view(c["Hkv"], G, 1, c["d"]).sum(1)
        s = (k[b, :, P:P + V].float() * qs).sum(-1).sum(0)
        out[b] = (s - s.min()) / (s.max() - s.min() + 1e-6)
    return out


def prepare(case, seed):
    c, g = case, torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    p = _params(c)
    hidden, q, k = _hidden_and_qk(c, g)
    st = {"case": c, "ctx": _context(), "p": p, "q": q, "k": k}
    N = c["P"] + c["V"] + c["Tmax"]
    if c["kind"] == "attention":
        st["v"] = torch.randn(c["B"], c["Hkv"], N, c["d"], generator=g, device="cuda").to(_TDTYPE[c["qk"]])
        st["s_hat"] = _salience(c, q, k) if c["mask"] else None
        st["out"] = torch.empty(c["B"], c["H"], N, c["d"], dtype=_TDTYPE[c["qk"]], device="cuda")
        st["workspace"] = torch.empty(max(A.asap_attention_workspace_bytes(p), 256), dtype=torch.uint8, device="cuda")
        return st
    st["hidden"] = hidden
    st["text_len"] = torch.randint(c["text_lo"], c["Tmax"] + 1, (c["B"],), generator=g, device="cuda").to(torch.int32)
    cache = lambda: [torch.randn(c["B"], c["Hkv"], N, c["d"], generator=g, device="cuda").to(_TDTYPE[c["kv"]])
                     for _ in range(c["layers"])]
    kc, vc = cache(), cache()
    if c["kind"] == "paged":
        st["paged"] = harness.PagedKV(p, kc, vc, c["page"], seed=int(seed))
        st["side"] = torch.cuda.Stream()
        st["buf"] = harness.StageBuffers(p, 0)
    else:
        st["k_cache"], st["v_cache"] = kc, vc
        st["buf"] = harness.StageBuffers(p, c["layers"])
        st["io"] = harness.stage_io(p, q, k, hidden, st["text_len"], kc, vc, st["buf"])
    return st


# ---------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------
def run(st):
    c, ctx, p = st["case"], st["ctx"], st["p"]
    if c["kind"] == "attention":
        ctx.asap_attention(p, st["q"], st["k"], st["v"], st["s_hat"], st["out"], st["workspace"])
        return st["out"]
    buf = st["buf"]
    if c["kind"] == "paged":
        harness.run_stage(ctx, p, st["q"], st["k"], st["hidden"], st["text_len"], [], [], buf, side_stream=st["side"],
                          paged=st["paged"])
    else:
        ctx.asap_stage(p, st["io"])
    n = c["V"] - c["k"]
    assign, best = buf.assign, buf.best_sim
    if c["route"] == "paper":                    # these two are then laid out [B,k] at the start of their buffers
        n = c["k"]
        assign, best = assign.view(-1)[:c["B"] * n].view(-1, n), best.view(-1)[:c["B"] * n].view(-1, n)
    out = {"s_raw": buf.s_raw, "s_hat": buf.s_hat, "score": buf.score, "kept_idx": buf.kept_idx,
           "pruned_idx": buf.pruned_idx, "out_hidden": buf.out_hidden, "pos_out": buf.pos_out, "new_len": buf.new_len,
           "assign": assign, "best_sim": best, "wsum": buf.wsum, "final_idx": buf.final_idx}
    if c["kind"] == "paged":
        out["k_cache"], out["v_cache"] = st["paged"].k_pool, st["paged"].v_pool
    else:
        out["k_cache"], out["v_cache"] = buf.k_dst, buf.v_dst
    return out


def work(case):
    c = case
    B, H, Hkv, d, D, P, V, k = (c[x] for x in ("B", "H", "Hkv", "d", "D", "P", "V", "k"))
    eq, eh, ek = (2 if c[x] == "bf16" else 4 for x in ("qk", "h", "kv"))
    if c["kind"] == "attention":
        N = P + V + c["Tmax"]
        pairs = N * (N + 1) // 2 + (V * (V - 1) // 2 if c["mask"] else 0)
        return {"bytes": B * N * d * eq * (2 * H + 2 * Hkv) + (4 * B * V if c["mask"] else 0),
                "flops": 4.0 * d * B * H * pairs}
    T = (c["text_lo"] + c["Tmax"]) / 2.0                     # mean text length
    rows = 1 if c["rows"] == "last" else T
    out_rows = B * (P + k + T)
    paper = c["route"] == "paper"
    # hidden rows that matter: every visual row when pruned tokens are absorbed, the kept ones otherwise
    # (the refills are among the pruned rows and at most k in number: not counted)
    vis = B * (k if paper else V) * D * eh
    src = k if paper else V - k
    byts = (B * V * d * (H + Hkv) + B * H * rows * d) * eq + 12 * B * V       # queries, keys -> s, s_hat, score
    byts += 4 * B * V                                                         # kept and pruned lists
    byts += vis + B * (P + T) * D * eh + out_rows * D * eh + 8 * B * src + 8 * B * k + 4 * out_rows
    byts += 4 * c["layers"] * Hkv * out_rows * d * ek                         # K/V rows read and written
    flops = B * H * V * d + 2.0 * B * Hkv * V * d + 2.0 * B * H * rows * V * d + 2.0 * B * src * k * D
    return {"bytes": byts, "flops": flops}


def tolerance(case):
    """Scores and masses are good to about 1e-6 and copies exact, but the cosine search decides: where two kept
    tokens are equally similar to a pruned one to within the 32-bit sums (about 1 token in 1000 of a dense
    cluster), another order of addition takes the other one, and two merged rows then hold or miss that token.
    This is what rel, max and differ leave room for in the stage, in both precisions."""
    if case["kind"] == "attention":
        return {"rel": 1e-2 if case["qk"] == "bf16" else 2e-5}
    return {"rel": 1e-2, "max": 0.9, "differ": 2e-3}

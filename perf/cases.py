"""What the performance of this framework is measured on.

Every case is work that a serving program has the library do through its public entry points:
decode steps over a compressed cache (`step`, `per_head`), construction of that cache (`build`,
`vlm_build`), the router that feeds it (`router`) and the move of recent tokens into it
(`flush`).  Inputs are synthetic, made on the GPU from the seed alone, with the shapes, budgets
and value structure of the framework's own workloads: normal keys, values, queries and router
logits, keys with four channels per head scaled by 8, kept-group counts spread around their mean.
"""
import math

import torch

import paper_2604_21335_amd as stc

DEV = "cuda:0"
PAGE = 16


# --------------------------------------------------------------------------------------------
# The cases
# --------------------------------------------------------------------------------------------
def listed():
    return [
        # One layer, one short sequence, 8 heads of 64: the smallest decode step there is, where
        # launches and latency are everything.
        dict(name="step_tiny", kind="step", B=1, Hq=8, Hkv=8, D=64, N=1024, G=4, k=16, keep=0.5,
             text=0, tail=0, layers=1),
        # LLaMA-2-7B-shaped layer, batch 8, 4096 tokens, budget 1024: multi-head attention.
        dict(name="step_llama2_7b_4k", kind="step", B=8, Hq=32, Hkv=32, D=128, N=4096, G=8, k=64,
             keep=0.5625, text=0, tail=0, layers=1),
        # Qwen2.5-7B-shaped layer, batch 16, 32768 tokens, budget 2048: the framework's headline,
        # a full serving batch over long contexts with grouped queries.
        dict(name="step_qwen25_7b_32k", kind="step", B=16, Hq=28, Hkv=4, D=128, N=32768, G=8,
             k=128, keep=0.5, text=0, tail=0, layers=1),
        # One token of one user with a 131072-token context: 28 layer caches one after the other.
        dict(name="step_qwen25_7b_128k", kind="step", B=1, Hq=28, Hkv=4, D=128, N=131072, G=16,
             k=256, keep=0.25, text=0, tail=0, layers=28),
        # LLaVA-1.5-7B-shaped prefix, batch 64: 144 retained visual and 64 text tokens, every
        # page attended.
        dict(name="step_llava15_7b_prefix", kind="step", B=64, Hq=32, Hkv=32, D=128, N=208, G=8,
             k=13, keep=0.0, text=64, tail=0, layers=1),
        # A small batch in mid-generation, grouped queries 4:1, a token count that fills neither
        # its last page nor its last tile: the new token is appended to the uncompressed tail,
        # then the step attends the selected pages and the tail.
        dict(name="step_tail_ragged", kind="step", B=5, Hq=32, Hkv=8, D=128, N=12013, G=8, k=90,
             keep=0.5, text=0, tail=100, layers=1),
        # Every query head selects and attends its own pages (the other reading of the page
        # selection under grouped queries) on the headline's cache.
        dict(name="per_head_qwen25_7b_32k", kind="per_head", B=16, Hq=28, Hkv=4, D=128, N=32768,
             G=8, k=128, keep=0.5, union=False),
        # Cache construction after the prefill of the headline batch: page bounds, routing by
        # per-token counts, packed values.
        dict(name="build_qwen25_7b_32k", kind="build", B=16, Hkv=4, D=128, N=32768, G=8,
             mode="topk", shared=False, keep=0.5),
        # Cache construction in the paper's LLM setting: one set of router logits per token and
        # layer for all 32 heads, a global budget of token-group pairs.
        dict(name="build_llama2_7b_4k_global", kind="build", B=8, Hkv=32, D=128, N=4096, G=8,
             mode="global", shared=True, keep=0.5),
        # The same for a batch of images: compaction to the retained tokens, then routing with
        # a fixed count per visual token and full values for text.
        dict(name="build_llava15_7b_prefix", kind="vlm_build", B=64, Hkv=32, D=128, visual=576,
             text=64, retained=144, G=8, groups=3),
        # The router's projection of the hidden states of the headline batch's prefill.
        dict(name="router_qwen25_7b_32k", kind="router", B=16, N=32768, d_model=3584, G=8),
        # 64 recent tokens of every sequence move from the tail into the compressed cache.
        dict(name="flush_qwen25_7b_32k", kind="flush", B=16, Hkv=4, D=128, N=32768, G=8, n=64,
             keep=0.5),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _heads(rng):
    """(D, Hkv, query heads per KV head, G)"""
    D = rng.choice([64, 128, 128, 128])
    Hkv = rng.choice([1, 2, 4, 4, 8, 8, 16, 32])
    R = rng.choice([1, 1, 2, 4, 4, 5, 7, 8, 16]) if Hkv <= 8 else 1
    return D, Hkv, R, rng.choice([4, 8, 8, 16 if D == 128 else 4])


def _batch(rng, Hkv, D, N, most_bytes):
    """A batch whose keys take at most most_bytes (and whose streams a launch can number)."""
    return _log(rng, 1, max(1, min(64, most_bytes // (Hkv * N * D * 2))))


KEYS = 16 * 4 * 32768 * 128 * 2   # bytes of the keys of the headline's cache


def draw(rng):
    kind = rng.choice(["step"] * 5 + ["per_head", "build", "build", "vlm_build", "router", "flush"])
    D, Hkv, R, G = _heads(rng)
    keep = rng.choice([0.25, 0.375, 0.5, 0.5625, 0.75])
    if kind == "step":
        N = _log(rng, 200, 131072)
        B = _batch(rng, Hkv, D, N, KEYS // 2)
        NP = (N + PAGE - 1) // PAGE
        k = NP if rng.random() < 0.15 else max(1, min(NP, 512, int(NP * rng.uniform(0.03, 0.3))))
        if B * Hkv * k > 32 * 1024:            # selected keys of at most 128 MiB
            B = max(1, 32 * 1024 // (Hkv * k))
        tail = rng.choice([0, 0, 0, rng.randint(1, 128)])
        return dict(kind=kind, B=B, Hq=Hkv * R, Hkv=Hkv, D=D, N=N, G=G, k=k, keep=keep, text=0,
                    tail=tail, layers=1)
    if kind == "per_head":
        N = _log(rng, 1000, 65536)
        Hkv = min(Hkv, 8)
        B = _batch(rng, Hkv, D, N, KEYS // 4)
        NP = (N + PAGE - 1) // PAGE
        k = max(1, min(NP, 256, int(NP * rng.uniform(0.03, 0.2))))
        if B * Hkv * R * k > 32 * 1024:
            B = max(1, 32 * 1024 // (Hkv * R * k))
        return dict(kind=kind, B=B, Hq=Hkv * R, Hkv=Hkv, D=D, N=N, G=G, k=k, keep=keep,
                    union=rng.random() < 0.5)
    if kind == "build":
        N = _log(rng, 200, 131072)
        B = _batch(rng, Hkv, D, N, KEYS)
        return dict(kind=kind, B=B, Hkv=Hkv, D=D, N=N, G=G,
                    mode=rng.choice(["topk", "topk", "global", "mask"]),
                    shared=rng.random() < 0.5, keep=keep)
    if kind == "vlm_build":
        visual, text = rng.randint(140, 900), rng.randint(8, 128)
        retained = max(8, int(visual * rng.choice([0.125, 0.25, 0.5])))
        B = _batch(rng, Hkv, D, visual + text, KEYS // 2)
        return dict(kind=kind, B=B, Hkv=Hkv, D=D, visual=visual, text=text, retained=retained,
                    G=G, groups=max(1, G // 4))
    if kind == "router":
        d_model = rng.choice([2048, 3584, 4096, 5120])
        N = _log(rng, 100, 65536)
        B = _log(rng, 1, max(1, min(64, 16 * 32768 * 3584 // (N * d_model))))
        return dict(kind=kind, B=B, N=N, d_model=d_model, G=rng.choice([4, 8, 8, 16]))
    N = _log(rng, 500, 65536)
    B = _batch(rng, Hkv, D, N, KEYS // 2)
    return dict(kind=kind, B=B, Hkv=Hkv, D=D, N=N, G=G, n=rng.randint(1, 128), keep=keep)


# --------------------------------------------------------------------------------------------
# Inputs
# --------------------------------------------------------------------------------------------
class _Draw:
    """Tensors from one seeded generator on the GPU, in the order asked for."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(int(seed))

    def normal(self, *shape, dtype=torch.bfloat16):
        return torch.randn(*shape, generator=self.g, device=DEV, dtype=dtype)

    def keys(self, B, Hkv, N, D):
        scale = torch.ones(Hkv, D, device=DEV, dtype=torch.bfloat16)
        scale.scatter_(1, torch.rand(Hkv, D, generator=self.g, device=DEV).argsort(1)[:, :4], 8.0)
        return self.normal(B, Hkv, N, D).mul_(scale[None, :, None, :])

    def counts(self, B, H, N, G, keep):
        """Kept groups per token: uniform on 1 .. 2*keep*G - 1, at most G."""
        return torch.randint(1, _most(G, keep) + 1, (B, H, N), generator=self.g,
                             device=DEV).clamp_(max=G).to(torch.uint8)


def _most(G, keep):
    return max(1, int(round(2 * keep * G)) - 1)


def _mean_kept(G, keep):
    m = _most(G, keep)
    return sum(min(c, G) for c in range(1, m + 1)) / m


def _vlm_counts(B, H, visual, text, groups, G):
    row = torch.full((visual + text,), G, dtype=torch.uint8, device=DEV)
    row[:visual] = groups
    return row.expand(B, H, visual + text).contiguous()


def _cache_inputs(c, seed):
    """Keys, values, logits, counts of a decode case's cache, then its query and tail."""
    d = _Draw(seed)
    B, Hkv, D, N, G = c["B"], c["Hkv"], c["D"], c["N"], c["G"]
    i = dict(K=d.keys(B, Hkv, N, D), V=d.normal(B, Hkv, N, D),
             logits=d.normal(B, Hkv, N, G, dtype=torch.float32))
    i["kcount"] = (_vlm_counts(B, Hkv, N - c["text"], c["text"], 3, G) if c.get("text")
                   else d.counts(B, Hkv, N, G, c["keep"]))
    i["q"] = d.normal(B, c["Hq"], D)
    if c.get("tail"):
        i["K_tail"], i["V_tail"] = d.keys(B, Hkv, c["tail"], D), d.normal(B, Hkv, c["tail"], D)
    return i


def _build_inputs(c, seed):
    d = _Draw(seed)
    B, Hkv, D, N, G = c["B"], c["Hkv"], c["D"], c["N"], c["G"]
    H = 1 if c["shared"] else Hkv
    i = dict(K=d.keys(B, Hkv, N, D), V=d.normal(B, Hkv, N, D), route={})
    r = i["route"]
    if c["mode"] == "mask":
        r["mask_in"] = torch.randint(1, 1 << G, (B, H, N), generator=d.g,
                                     device=DEV).to(torch.int16)
    else:
        r["logits"] = d.normal(B, H, N, G, dtype=torch.float32)
        if c["mode"] == "topk":
            r["kcount"] = d.counts(B, H, N, G, c["keep"])
        else:
            r["global_k"] = max(1, int(c["keep"] * G))
    return i


def _vlm_inputs(c, seed):
    d = _Draw(seed)
    B, Hkv, D, G = c["B"], c["Hkv"], c["D"], c["G"]
    n = c["visual"] + c["text"]
    vis = torch.rand(B, c["visual"], generator=d.g, device=DEV).argsort(1)[:, :c["retained"]]
    txt = torch.arange(c["visual"], n, device=DEV).expand(B, -1)
    return dict(K=d.normal(B, Hkv, n, D), V=d.normal(B, Hkv, n, D),
                token_idx=torch.cat([vis.sort(1).values, txt], 1).to(torch.int32).contiguous(),
                logits=d.normal(B, 1, c["retained"] + c["text"], G, dtype=torch.float32),
                kcount=_vlm_counts(B, 1, c["retained"], c["text"], c["groups"], G))


def _router_inputs(c, seed):
    d = _Draw(seed)
    return dict(h=d.normal(c["B"], c["N"], c["d_model"]),
                W=d.normal(c["G"], c["d_model"]).mul_(c["d_model"] ** -0.5),
                bias=d.normal(c["G"], dtype=torch.float32))


def _flush_inputs(c, seed):
    d = _Draw(seed)
    B, Hkv, D, N, G, n = c["B"], c["Hkv"], c["D"], c["N"], c["G"], c["n"]
    return dict(K=d.keys(B, Hkv, N + n, D), V=d.normal(B, Hkv, N + n, D),
                logits=d.normal(B, Hkv, N + n, G, dtype=torch.float32),
                kcount=d.counts(B, Hkv, N + n, G, c["keep"]))


# --------------------------------------------------------------------------------------------
# What a program has before the call, and the call
# --------------------------------------------------------------------------------------------
def _layer_seed(seed, layer):
    return seed * 64 + layer


def prepare(case, seed):
    c = case
    kind = c["kind"]
    if kind == "step":
        layers = []
        for n in range(c["layers"]):
            i = _cache_inputs(c, _layer_seed(seed, n))
            cap = c["tail"] + 28 if c["tail"] else 0
            cache = stc.RoutedCache(c["B"], c["Hq"], c["Hkv"], c["D"], c["N"], c["G"], c["k"],
                                    device=DEV, tail_cap=cap, n_cap=c["N"] + 512 if cap else 0)
            cache.build(i["K"], i["V"], logits=i["logits"], kcount=i["kcount"])
            s = dict(cache=cache, q=i["q"])
            if cap:                        # all tail tokens but the newest are there already
                t = c["tail"] - 1
                cache.K_tail[:, :, :t].copy_(i["K_tail"][:, :, :t])
                cache.V_tail[:, :, :t].copy_(i["V_tail"][:, :, :t])
                s["k_new"] = i["K_tail"][:, :, t].contiguous()
                s["v_new"] = i["V_tail"][:, :, t].contiguous()
            layers.append(s)
        return dict(case=c, layers=layers)
    if kind == "per_head":
        i = _cache_inputs(c, seed)
        cache = stc.RoutedCache(c["B"], c["Hq"], c["Hkv"], c["D"], c["N"], c["G"], c["k"],
                                device=DEV)
        cache.build(i["K"], i["V"], logits=i["logits"], kcount=i["kcount"])
        NP, R = cache.NP, c["Hq"] // c["Hkv"]
        k = min(c["k"], NP)
        u = min(NP, R * k)

        def ws(which, n):
            return torch.empty(max(stc.stc_workspace_bytes(cache.shape, which, n), 16),
                               dtype=torch.uint8, device=DEV)
        return dict(case=c, cache=cache, q=i["q"], k=k,
                    page_idx=torch.empty(c["B"], c["Hq"], k, dtype=torch.int32, device=DEV),
                    page_score=torch.empty(c["B"], c["Hq"], NP, dtype=torch.float32, device=DEV),
                    union_idx=torch.empty(c["B"], c["Hkv"], u, dtype=torch.int32, device=DEV),
                    union_heads=torch.empty(c["B"], c["Hkv"], u, dtype=torch.int16, device=DEV),
                    ws_sel=ws(stc.STC_WS_SELECT_PER_HEAD, k),
                    ws_att=ws(stc.STC_WS_ATTENTION, u) if c["union"]
                    else ws(stc.STC_WS_ATTENTION_PER_HEAD, k))
    if kind == "build":
        i = _build_inputs(c, seed)
        cache = stc.RoutedCache(c["B"], c["Hkv"], c["Hkv"], c["D"], c["N"], c["G"], 1, device=DEV)
        cache.vpacked.zero_()              # slots behind the kept groups are never written
        return dict(case=c, cache=cache, **i)
    if kind == "vlm_build":
        i = _vlm_inputs(c, seed)
        n = c["retained"] + c["text"]
        cache = stc.RoutedCache(c["B"], c["Hkv"], c["Hkv"], c["D"], n, c["G"], (n + 15) // 16,
                                device=DEV)
        cache.vpacked.zero_()
        K = torch.empty(c["B"], c["Hkv"], n, c["D"], dtype=torch.bfloat16, device=DEV)
        return dict(case=c, cache=cache, K_kept=K, V_kept=torch.empty_like(K), **i)
    if kind == "router":
        i = _router_inputs(c, seed)
        return dict(case=c, logits=torch.empty(c["B"], 1, c["N"], c["G"], device=DEV), **i)
    i = _flush_inputs(c, seed)             # flush
    N, n = c["N"], c["n"]
    cache = stc.RoutedCache(c["B"], c["Hkv"], c["Hkv"], c["D"], N, c["G"], 1, device=DEV,
                            tail_cap=n, n_cap=N + n)
    for t in (cache.K, cache.vpacked, cache.bounds):
        t.zero_()
    cache.build(i["K"][:, :, :N], i["V"][:, :, :N].contiguous(),
                logits=i["logits"][:, :, :N].contiguous(),
                kcount=i["kcount"][:, :, :N].contiguous())
    cache.K_tail.copy_(i["K"][:, :, N:])
    cache.V_tail.copy_(i["V"][:, :, N:])
    return dict(case=c, cache=cache, logits=i["logits"][:, :, N:].contiguous(),
                kcount=i["kcount"][:, :, N:].contiguous())


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "step":
        out = []
        for l in s["layers"]:
            cache = l["cache"]
            if c["tail"]:
                cache.n_tail = c["tail"] - 1
                cache.append(l["k_new"], l["v_new"])
            out.append((cache.step(l["q"]), cache.page_idx))
        return out
    if kind == "per_head":
        cache, q = s["cache"], s["q"]
        stc.stc_select_pages_per_head(cache.shape, q, cache.bounds, s["k"], s["page_idx"],
                                      s["page_score"], s["ws_sel"])
        if c["union"]:
            stc.stc_union_pages(cache.shape, s["page_idx"], s["k"], s["union_idx"],
                                s["union_heads"])
            stc.stc_decode_attention_union(cache.shape, q, cache.K, cache.vpacked, cache.mask,
                                           cache.tok_off, s["union_idx"], s["union_heads"],
                                           cache.out, s["ws_att"])
            return cache.out, s["page_idx"], s["union_idx"], s["union_heads"]
        stc.stc_decode_attention_per_head(cache.shape, q, cache.K, cache.vpacked, cache.mask,
                                          cache.tok_off, s["page_idx"], s["k"], cache.out,
                                          s["ws_att"])
        return cache.out, s["page_idx"]
    if kind == "router":
        stc.stc_router_logits(s["h"], s["W"], s["bias"], s["logits"], 1)
        return s["logits"]
    cache = s["cache"]
    if kind == "build":
        cache.build(s["K"], s["V"], shared=c["shared"], **s["route"])
        return cache.bounds, cache.mask, cache.tok_off, cache.vpacked
    if kind == "vlm_build":
        n_src, n = c["visual"] + c["text"], c["retained"] + c["text"]
        stc.stc_compact_tokens(s["K"], s["token_idx"], s["K_kept"], c["B"], c["Hkv"], n_src, n,
                               c["D"], cache.dev_status)
        stc.stc_compact_tokens(s["V"], s["token_idx"], s["V_kept"], c["B"], c["Hkv"], n_src, n,
                               c["D"], cache.dev_status)
        cache.build(s["K_kept"], s["V_kept"], logits=s["logits"], kcount=s["kcount"], shared=True)
        return s["K_kept"], cache.bounds, cache.mask, cache.tok_off, cache.vpacked
    # flush: the whole tail, so that a pass leaves its own inputs as they were
    stc.stc_flush_tail(cache.shape, cache.K_tail, cache.V_tail, c["n"], c["n"], c["n"],
                       stc.STC_ROUTE_TOPK, s["logits"], s["kcount"], 0, None, cache.K,
                       cache.bounds, cache.mask, cache.tok_off, cache.vpacked, cache.dev_status)
    return cache.K, cache.bounds, cache.mask, cache.tok_off, cache.vpacked


# --------------------------------------------------------------------------------------------
# What a pass cannot do without
# --------------------------------------------------------------------------------------------
def work(case):
    c = case
    kind = c["kind"]
    if kind == "router":
        tokens = c["B"] * c["N"]
        return {"bytes": tokens * (c["d_model"] * 2 + c["G"] * 4) + c["G"] * c["d_model"] * 2,
                "flops": 2 * tokens * c["d_model"] * c["G"]}
    B, Hkv, D, G = c["B"], c["Hkv"], c["D"], c["G"]
    row, gd2 = D * 2, D // G * 2
    if kind in ("step", "per_head"):
        N, Hq = c["N"], c["Hq"]
        S, R, NP = B * Hkv, Hq // Hkv, (N + PAGE - 1) // PAGE
        k = min(c["k"], NP)
        per_head = kind == "per_head"
        # pages that a KV head's query heads read together, if each chose its own at random
        pages = NP * (1 - (1 - k / NP) ** R) if per_head else k
        tok = pages * N / NP
        kept = ((3 * (N - c["text"]) + G * c["text"]) / N if c.get("text")
                else _mean_kept(G, c["keep"]))
        score = NP * 4 * D if (k < NP) else 0
        nbytes = S * (score + tok * (row + kept * gd2 + 2) + pages * 12)
        nbytes += B * Hq * D * 6 + (B * Hq if per_head else S) * k * 4
        attended = k * N / NP + c.get("tail", 0)
        flops = B * Hq * (attended * D * 4 + (3 * D * NP if k < NP else 0))
        if c.get("tail"):
            nbytes += S * (c["tail"] + 2) * row * 2
        n = c.get("layers", 1)
        return {"bytes": n * nbytes, "flops": n * flops}
    if kind == "vlm_build":
        n = c["retained"] + c["text"]
        kept = c["retained"] * c["groups"] + c["text"] * G
        return {"bytes": B * (Hkv * (3 * n * row + (n + 15) // 16 * 4 * D + kept * gd2 + 6 * n)
                              + n * (5 + 4 * G)), "flops": B * Hkv * n * D}
    if kind == "build":
        N = c["N"]
        H = 1 if c["shared"] else Hkv
        kept = {"topk": _mean_kept(G, c["keep"]), "global": max(1, int(c["keep"] * G)),
                "mask": G / 2}[c["mode"]]
        routing = 2 if c["mode"] == "mask" else 4 * G + (c["mode"] == "topk")
        return {"bytes": B * (Hkv * ((N + 15) // 16 * 4 * D + N * (row + 2 * kept * gd2 + 6))
                              + H * N * routing), "flops": B * Hkv * N * D}
    n, kept = c["n"], _mean_kept(G, c["keep"])      # flush
    pages = (c["N"] + n - 1) // PAGE - c["N"] // PAGE + 1
    return {"bytes": B * Hkv * (n * (2 * row + 2 * kept * gd2 + 4 * G + 7)
                                + (c["N"] % PAGE) * row + pages * 4 * D),
            "flops": B * Hkv * n * D}


def tolerance(case):
    # Masks, offsets, packed values, page lists: integers and bytes, always the same.
    if case["kind"] in ("build", "vlm_build", "flush"):
        return "exact"
    # Router logits: float sums of up to 5120 exact products; 9e-8 against 64 bits.
    if case["kind"] == "router":
        return {"rel": 4e-7, "max": 4e-6, "differ": 0.0}
    # Attention: float accumulation, softmax weights carried as two bf16 parts (2^-17 each);
    # 5e-7 .. 1e-6 against 64 bits.
    return {"rel": 4e-6, "max": 4e-5, "differ": 0.0}


# --------------------------------------------------------------------------------------------
# The same in 64 bits, with torch alone
# --------------------------------------------------------------------------------------------
def _kept_bits(logits, kcount):
    """[..., N, G] booleans: the kcount largest logits of every token (ties: lower group)."""
    order = logits.argsort(dim=-1, descending=True, stable=True)
    rank = torch.empty_like(order)
    rank.scatter_(-1, order, torch.arange(order.shape[-1], device=DEV).expand_as(order))
    return rank < kcount.long().unsqueeze(-1)


def _page_bounds(K):
    """Per page and channel minimum and maximum over the page's tokens: two [..., NP, D]."""
    N = K.shape[-2]
    pad = -N % PAGE
    NP = (N + pad) // PAGE

    def pages(fill):
        t = torch.nn.functional.pad(K, (0, 0, 0, pad), value=fill) if pad else K
        return t.reshape(*K.shape[:-2], NP, PAGE, K.shape[-1])
    return pages(math.inf).amin(-2), pages(-math.inf).amax(-2)


def _tiled_bounds(K, cap_pages):
    """The bounds in the library's layout: tiles of 8 pages, see the header."""
    B, Hkv, _, D = K.shape
    mn, mx = _page_bounds(K)
    nt = (cap_pages + 7) // 8
    rows = torch.zeros(B, Hkv, nt * 8, 2, D, dtype=torch.float64, device=DEV)
    rows[:, :, :mn.shape[2], 0] = mn.double()
    rows[:, :, :mn.shape[2], 1] = mx.double()
    t = rows.view(B, Hkv, nt, 2, 4, 2, 8, D // 32, 4)     # t, g, col, min|max, e, j, w
    return t.permute(0, 1, 2, 7, 3, 6, 4, 8, 5).reshape(-1)


def _select(q, mn, mx, k):
    """The k pages of largest upper bound (ties: lowest), ascending.  q [R, D], mn/mx [NP, D].
    The selection is defined on float sums of a balanced tree, so those are what it uses."""
    x = torch.maximum(q[:, None, :].float() * mn.float(), q[:, None, :].float() * mx.float())
    while x.shape[-1] > 1:
        x = x[..., 0::2] + x[..., 1::2]
    score = x[..., 0].amax(0)
    return score.argsort(dim=0, descending=True, stable=True)[:k].sort().values


def _attend(q, K, V, bits, pages, K_tail=None, V_tail=None):
    """q [R, D] over the tokens of `pages` and the tail, dropped value groups as zeros."""
    N, D = K.shape
    t = (pages[:, None] * PAGE + torch.arange(PAGE, device=DEV)).reshape(-1)
    t = t[t < N]
    k, v = K[t].double(), V[t].double()
    G = bits.shape[-1]
    v = (v.view(-1, G, D // G) * bits[t].unsqueeze(-1)).view(-1, D)
    if K_tail is not None:
        k, v = torch.cat([k, K_tail.double()]), torch.cat([v, V_tail.double()])
    p = torch.softmax(q.double() @ k.t().contiguous() / math.sqrt(D), -1)
    return p @ v


def _exact_attention(c, i):
    """(out [B, Hq, D], page lists per KV head, per query head, unions with head sets)."""
    B, Hq, Hkv, D, N = c["B"], c["Hq"], c["Hkv"], c["D"], c["N"]
    R, NP = Hq // Hkv, (N + PAGE - 1) // PAGE
    k = min(c["k"], NP)
    per_head = c["kind"] == "per_head"
    out = torch.empty(B, Hq, D, dtype=torch.float64, device=DEV)
    lists = torch.empty(B, Hq if per_head else Hkv, k, dtype=torch.int32, device=DEV)
    u = min(NP, R * k)
    uidx = torch.full((B, Hkv, u), -1, dtype=torch.int32, device=DEV)
    uheads = torch.zeros(B, Hkv, u, dtype=torch.int16, device=DEV)
    for b in range(B):
        for h in range(Hkv):
            K, V = i["K"][b, h], i["V"][b, h]
            bits = _kept_bits(i["logits"][b, h], i["kcount"][b, h])
            q = i["q"][b, h * R:(h + 1) * R]
            tail = (i["K_tail"][b, h], i["V_tail"][b, h]) if c.get("tail") else ()
            mn, mx = _page_bounds(K)
            if not per_head:
                pages = _select(q, mn, mx, k)
                lists[b, h] = pages.int()
                out[b, h * R:(h + 1) * R] = _attend(q, K, V, bits, pages, *tail)
                continue
            sets = torch.zeros(NP, dtype=torch.int32, device=DEV)
            for r in range(R):
                pages = _select(q[r:r + 1], mn, mx, k)
                lists[b, h * R + r] = pages.int()
                out[b, h * R + r] = _attend(q[r:r + 1], K, V, bits, pages)[0]
                sets[pages] += 1 << r
            p = sets.nonzero()[:, 0]
            uidx[b, h, :len(p)] = p.int()
            uheads[b, h, :len(p)] = sets[p].to(torch.int16)
    return out, lists, uidx, uheads


def _exact_store(bits, V, cap_tokens):
    """mask, tok_off, vpacked of a store for cap_tokens tokens, unused places 0."""
    B, Hkv, N, G = bits.shape
    gd = V.shape[-1] // G
    mask = (bits.long() << torch.arange(G, device=DEV)).sum(-1).to(torch.int16)
    slot = bits.reshape(B, Hkv, N * G).long().cumsum(-1)
    off = torch.zeros(B, Hkv, N + 1, dtype=torch.int32, device=DEV)
    off[:, :, 1:] = slot.view(B, Hkv, N, G)[..., -1].int()
    packed = torch.zeros(B, Hkv, cap_tokens * G, gd, dtype=torch.float64, device=DEV)
    flat = V.reshape(B, Hkv, N * G, gd)
    for b in range(B):
        for h in range(Hkv):
            packed[b, h, :int(off[b, h, -1])] = flat[b, h][bits[b, h].reshape(-1)].double()
    return mask, off, packed


def exact(case, seed):
    c = case
    kind = c["kind"]
    if kind == "step":
        if c["B"] * c["Hkv"] * c["layers"] > 4096:  # one small product each: over 20 seconds
            return None
        return [_exact_attention(c, _cache_inputs(c, _layer_seed(seed, n)))[:2]
                for n in range(c["layers"])]
    if kind == "per_head":
        if c["B"] * c["Hq"] > 4096:
            return None
        out, lists, uidx, uheads = _exact_attention(c, _cache_inputs(c, seed))
        return (out, lists, uidx, uheads) if c["union"] else (out, lists)
    if kind == "router":
        i = _router_inputs(c, seed)
        W = i["W"].double().t().contiguous()
        out = [(h.double() @ W + i["bias"].double()) for h in i["h"].view(-1, c["d_model"])
               .split(16384)]
        return torch.cat(out).view(c["B"], 1, c["N"], c["G"])
    if kind == "build":
        i = _build_inputs(c, seed)
        B, Hkv, N, G = c["B"], c["Hkv"], c["N"], c["G"]
        r = i["route"]
        if c["mode"] == "mask":
            bits = ((r["mask_in"].long().unsqueeze(-1) >> torch.arange(G, device=DEV)) & 1).bool()
        elif c["mode"] == "topk":
            bits = _kept_bits(r["logits"], r["kcount"])
        else:
            H = r["logits"].shape[1]
            order = r["logits"].view(B, H, N * G).argsort(dim=-1, descending=True, stable=True)
            bits = torch.zeros(B, H, N * G, dtype=torch.bool, device=DEV)
            bits.scatter_(-1, order[..., :N * r["global_k"]], True)
            bits = bits.view(B, H, N, G)
        bits = bits.expand(B, Hkv, N, G)
        return (_tiled_bounds(i["K"], (N + 15) // 16),) + _exact_store(bits, i["V"], N)
    if kind == "vlm_build":
        i = _vlm_inputs(c, seed)
        B, Hkv, D, G = c["B"], c["Hkv"], c["D"], c["G"]
        n = c["retained"] + c["text"]
        at = i["token_idx"].long()[:, None, :, None].expand(B, Hkv, n, D)
        K, V = i["K"].gather(2, at), i["V"].gather(2, at)
        bits = _kept_bits(i["logits"], i["kcount"]).expand(B, Hkv, n, G)
        return (K.double(), _tiled_bounds(K, (n + 15) // 16)) + _exact_store(bits, V, n)
    i = _flush_inputs(c, seed)                      # flush
    bits = _kept_bits(i["logits"], i["kcount"])
    return ((i["K"].double(), _tiled_bounds(i["K"], (c["N"] + c["n"] + 15) // 16))
            + _exact_store(bits, i["V"], c["N"] + c["n"]))

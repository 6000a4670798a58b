"""What a user of this package has it do, as cases that can be timed and compared.

Five kinds of call, each through the package's public entry points as a training loop or a server
calls them:

  train     mark + compact the separators of a batch, forward, backward (one layer's hot path);
            plain rows, rows packed from documents, or a neighbour window per query head
  prefill   mark + compact, forward, and optionally the hand-over of the prompt's K/V to the caches
  decode    one token per sequence over caches that are in use
  generate  a stretch of streaming generation: compress the caches, then append + decode token by token
  check     forward + backward in fp32, the path that a bf16 run is checked against

`keep` says whether the program keeps its output buffers and workspaces from step to step (a training
loop or a server that preallocates) or takes what the calls allocate for it (a notebook, autograd).
Sizes are those of workloads/generators.py and of the tests, and their neighbourhood.
"""
import ctypes
import math

import torch

import paper_2412_12094_amd as sp

# nine ids of a 32000-entry vocabulary stand for the nine separator strings
SEP_IDS = [17, 402, 1999, 5003, 8191, 12000, 20480, 27777, 31999]
VOCAB = 32000
ROPE_BASE = 500000.0

TRAIN = dict(kind="train", form="plain", docs=1, full_every=0)
DECODE = dict(kind="decode")


def listed():
    return [
        # the Llama-3-8B attention shape at 8K context: the headline training step
        dict(TRAIN, name="train_8k", B=1, Hq=32, Hkv=8, L=8192, d=128, a=4, n=256, p=0.08, keep=True),
        # the Pythia-160m training shape: many short sequences, one query head per KV head
        dict(TRAIN, name="train_2k", B=8, Hq=12, Hkv=12, L=2048, d=64, a=4, n=64, p=0.10, keep=True),
        # a small step from a notebook or a unit of fine-tuning: launches and allocations count
        dict(TRAIN, name="train_small", B=1, Hq=8, Hkv=2, L=600, d=128, a=4, n=96, p=0.10, keep=False),
        # a batch of odd sizes: ragged length, window not a multiple of anything, 7 heads per KV head
        dict(TRAIN, name="train_ragged", B=3, Hq=28, Hkv=4, L=3077, d=128, a=3, n=200, p=0.08, keep=False),
        # the headline row packed from eight documents
        dict(TRAIN, name="train_packed", form="packed", docs=8, B=1, Hq=32, Hkv=8, L=8192, d=128, a=4, n=256, p=0.08,
             keep=True),
        # head-wise variant: the heads of every fourth KV head see everything, the others a short window
        dict(TRAIN, name="train_headwise", form="headwise", full_every=4, B=1, Hq=32, Hkv=8, L=4096, d=128, a=4, n=128,
             p=0.08, keep=True),
        # long-context prefill, the largest call
        dict(name="prefill_64k", kind="prefill", B=1, Hq=32, Hkv=8, L=65536, d=128, a=4, n=1024, p=0.08, s=0, w=0, c=0,
             keep=True),
        # prompts of a serving batch, forward and hand-over to the streaming caches
        dict(name="prefill_serve", kind="prefill", B=4, Hq=32, Hkv=8, L=1531, d=128, a=4, n=256, p=0.08, s=64, w=256, c=800,
             keep=False),
        # a full serving batch over large caches: bound by reading the caches
        dict(DECODE, name="decode_batch", S=32, Hq=32, Hkv=8, d=128, a=4, s=2048, w=256, c=3332, fill=1.0, rope=False,
             keep=True),
        # one conversation over the smallest cache of the streaming experiments, positions within the cache
        dict(DECODE, name="decode_one", S=1, Hq=32, Hkv=8, d=128, a=4, s=64, w=256, c=800, fill=0.77, rope=True, keep=False),
        # one period of streaming generation with that cache: a compression, then the tokens until the next
        dict(name="generate", kind="generate", S=4, Hq=32, Hkv=8, d=128, a=4, s=64, w=256, c=800, p=0.08, rope=True),
        # the fp32 path at the size it is used for: checking
        dict(name="check_fp32", kind="check", B=1, Hq=2, Hkv=1, L=512, d=64, a=4, n=64, p=0.125),
    ]


def _logint(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


HEADS = [(8, 8), (12, 12), (32, 8), (16, 4), (28, 4), (8, 2), (16, 8), (32, 32), (6, 3), (8, 1)]


def _attn_sizes(rng, l_max, budget):
    """Head counts, length and window whose visible pairs x heads x d stay within `budget`."""
    while True:
        Hq, Hkv = rng.choice(HEADS)
        L = _logint(rng, 130, l_max)
        c = dict(B=rng.choice([1, 1, 1, 2, 3, 4, 8]), Hq=Hq, Hkv=Hkv, L=L, d=rng.choice([64, 128]), a=rng.choice([0, 1, 3, 4, 4, 8]),
                 n=min(L, _logint(rng, 16, 1024)), p=round(rng.uniform(0.04, 0.16), 3))
        if c["B"] * Hq * c["d"] * _pairs(L, c["a"], c["n"], c["p"]) <= budget and c["B"] * Hq * L <= 1 << 21:
            return c


def _cache_sizes(rng):
    d = rng.choice([64, 128])
    Hq, Hkv = rng.choice([(32, 8), (32, 8), (8, 8), (12, 12), (28, 4), (16, 2), (32, 32)])
    a, s, w = rng.choice([0, 3, 4, 4]), _logint(rng, 16, 2048), _logint(rng, 32, 512)
    return dict(Hq=Hq, Hkv=Hkv, d=d, a=a, s=s, w=w, c=a + s + w + _logint(rng, 32, 1024))


def draw(rng):
    kind = rng.choice(["train", "train", "train", "prefill", "decode", "decode", "generate", "check"])
    if kind == "train":
        form = rng.choice(["plain", "plain", "packed", "headwise"])
        c = dict(TRAIN, form=form, **_attn_sizes(rng, 16384, 2.0e10))
        if form == "packed":
            c["docs"] = rng.randint(2, max(2, min(16, c["L"] // 64)))
        if form == "headwise":
            c["L"] = min(c["L"], 4096)
            c["n"] = min(c["n"], c["L"])
            c["full_every"] = min(c["Hkv"], rng.choice([1, 2, 4, 8]))
        return dict(c, keep=rng.random() < 0.5)
    if kind == "prefill":
        c = dict(kind=kind, **_attn_sizes(rng, 65536, 3.0e11))
        c.update(s=0, w=0, c=0)
        if rng.random() < 0.6:
            s, w = _logint(rng, 16, 512), min(_logint(rng, 32, 512), max(1, c["L"] // 3))
            c.update(s=s, w=w, c=c["a"] + s + w + _logint(rng, 32, 512))
        return dict(c, keep=rng.random() < 0.5)
    if kind == "decode":
        while True:
            c = dict(kind=kind, S=_logint(rng, 1, 64), **_cache_sizes(rng))
            if c["S"] * c["Hkv"] * c["c"] * c["d"] <= 32 * 8 * 3332 * 128:
                return dict(c, fill=round(rng.uniform(0.3, 1.0), 2), rope=rng.random() < 0.5, keep=rng.random() < 0.5)
    if kind == "generate":
        while True:
            c = dict(kind=kind, S=_logint(rng, 1, 16), **_cache_sizes(rng))
            if c["c"] - c["a"] - c["s"] - c["w"] <= 512 and c["S"] * c["Hkv"] * c["c"] * c["d"] <= 1 << 24:
                return dict(c, p=round(rng.uniform(0.04, 0.16), 3), rope=rng.random() < 0.6)
    return dict(kind="check", B=rng.choice([1, 2]), Hq=4, Hkv=rng.choice([1, 2, 4]), L=_logint(rng, 64, 1024), d=rng.choice([64, 128]),
                a=rng.choice([0, 3, 4]), n=_logint(rng, 8, 128), p=round(rng.uniform(0.04, 0.2), 3))


# ------------------------------------------------------------------------------------------------
def _tokens(c, g):
    """int32 [B, L] token ids in which a position holds a separator with probability p."""
    dev = "cuda"
    shape = (c["B"], c["L"])
    ids = torch.randint(0, VOCAB - len(SEP_IDS), shape, device=dev, generator=g)
    for s in SEP_IDS:  # ascending: skip over the separators
        ids += ids >= s
    which = torch.tensor(SEP_IDS, device=dev)[torch.randint(0, len(SEP_IDS), shape, device=dev, generator=g)]
    return torch.where(torch.rand(shape, device=dev, generator=g) < c["p"], which, ids).to(torch.int32)


def _normal(g, shape, scale=1.0, dtype=torch.bfloat16):
    x = torch.randn(shape, device="cuda", generator=g, dtype=dtype)
    return x.mul_(scale) if scale != 1.0 else x


def _head_windows(c):
    """n of every query head: the heads of every `full_every`-th KV head see the whole sequence."""
    G = c["Hq"] // c["Hkv"]
    return [c["L"] if (h // G) % c["full_every"] == c["full_every"] - 1 else c["n"] for h in range(c["Hq"])]


def _prepare_attn(c, g):
    B, Hq, Hkv, L, d = c["B"], c["Hq"], c["Hkv"], c["L"], c["d"]
    dtype = torch.float32 if c["kind"] == "check" else torch.bfloat16
    st = dict(c, scale=1.0 / math.sqrt(d), tok=_tokens(c, g), Q=_normal(g, (B, Hq, L, d), 0.5, dtype),
              K=_normal(g, (B, Hkv, L, d), 0.5, dtype), V=_normal(g, (B, Hkv, L, d), 0.5, dtype))
    if c["kind"] != "prefill":
        st["dO"] = _normal(g, (B, Hq, L, d), 1.0, dtype)
    if c.get("form") == "packed":
        cuts = []
        for _ in range(B):
            inner = torch.randperm(L - 1, device="cuda", generator=g)[: c["docs"] - 1] + 1
            ends = torch.tensor([0, L], device="cuda", dtype=inner.dtype)
            cuts.append(torch.cat([ends, inner]).sort().values.to(torch.int32))
        st["cu"] = cuts
    if c.get("form") == "headwise":
        st["nh"] = _head_windows(c)
    st.update(idx_out=None, bounds=None, ows=None, cws=None, gout=None, bws=None)
    if c.get("keep"):
        i32 = dict(dtype=torch.int32, device="cuda")
        st["idx_out"] = (torch.empty((B, L), dtype=torch.uint8, device="cuda"), torch.full((B, L), -1, **i32),
                         torch.empty((B,), **i32), torch.empty((B, L + 1), **i32))
        st["bounds"] = (torch.empty((B, L), **i32), torch.empty((B, L), **i32))
        st["ows"] = (torch.empty_like(st["Q"]), torch.empty((B, Hq, L), dtype=torch.float32, device="cuda"))
        st["cws"] = torch.empty(max(256, sp.load().sepattn_compact_workspace_bytes(B, L)), dtype=torch.uint8, device="cuda")
        if c["kind"] == "train":
            st["gout"] = tuple(torch.empty_like(st[k]) for k in ("Q", "K", "V"))
            n = max(st["nh"]) if "nh" in st else c["n"]
            nb = sp.sepattn_backward_workspace_bytes(st["Q"], st["K"], 0 if c["form"] == "packed" else c["a"], n, st["scale"], L)
            st["bws"] = torch.empty(nb, dtype=torch.uint8, device="cuda")
    if c["kind"] == "prefill" and c["c"]:
        room = c["c"] - c["a"] - c["s"]
        # what the append / compression policy holds in its window after L tokens
        st["nw"] = max(0, min(room, L - c["a"], c["w"] + L % (room - c["w"] + 1)))
        st["cache_out"] = None
        if c["keep"]:
            cache = torch.zeros((B, Hkv, c["c"], d), dtype=dtype, device="cuda")
            st["cache_out"] = (cache, torch.zeros_like(cache), torch.zeros((B, room), dtype=torch.uint8, device="cuda"),
                               torch.zeros((B, 6), dtype=torch.int32, device="cuda"))
    return st


def _prepare_cache(c, g):
    S, Hq, Hkv, d, a, s, w, cc = (c[k] for k in ("S", "Hq", "Hkv", "d", "a", "s", "w", "c"))
    room = cc - a - s
    st = dict(c, scale=1.0 / math.sqrt(d), Kc=_normal(g, (S, Hkv, cc, d)), Vc=_normal(g, (S, Hkv, cc, d)))
    st["table"] = sp.sepkv_rope_table(cc, d, ROPE_BASE, "cuda") if c["rope"] else None
    pick = lambda lo, hi: torch.randint(lo, hi + 1, (S,), device="cuda", generator=g)
    sizes = torch.zeros((S, 6), dtype=torch.int64, device="cuda")
    sizes[:, 0], sizes[:, 1], sizes[:, 3] = a, s, w
    sizes[:, 4], sizes[:, 5] = pick(0, s - 1), pick(0, room - 1)
    if c["kind"] == "decode":
        # sequences in different phases between two compressions, `fill` of the capacity in use on average
        past = c["fill"] * (room - w)
        sizes[:, 2] = pick(int(0.8 * past), min(room - w, int(1.2 * past))) if c["fill"] < 1.0 else room - w
        st["q"] = _normal(g, (S, Hq, d))
        st["out"] = (torch.empty_like(st["q"]), torch.empty((S, Hq), dtype=torch.float32, device="cuda")) if c["keep"] else None
        st["ws"] = _decode_ws(c) if c["keep"] else None
    else:
        T = room - w
        sizes[:, 2] = T
        st["flags"] = (torch.rand((S, room), device="cuda", generator=g) < c["p"]).to(torch.uint8)
        k, v = _normal(g, (T, S, Hkv, d)), _normal(g, (T, S, Hkv, d))
        q, sep = _normal(g, (T, S, Hq, d)), (torch.rand((T, S), device="cuda", generator=g) < c["p"]).to(torch.uint8)
        st["outs"], st["lses"] = torch.empty_like(q), torch.empty((T, S, Hq), dtype=torch.float32, device="cuda")
        st["steps"] = [(k[t], v[t], sep[t], q[t], (st["outs"][t], st["lses"][t])) for t in range(T)]
        st["ws"] = _decode_ws(c)
    st["sizes"] = sizes.to(torch.int32)
    return st


def _decode_ws(c):
    p = sp.SepkvParams(c["S"], c["Hq"], c["Hkv"], c["d"], c["a"], c["s"], c["w"], c["c"], 1.0 / math.sqrt(c["d"]), sp.SEPATTN_BF16)
    return torch.empty(max(256, sp.load().sepattn_decode_workspace_bytes(ctypes.byref(p))), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return _prepare_cache(case, g) if case["kind"] in ("decode", "generate") else _prepare_attn(case, g)


# ------------------------------------------------------------------------------------------------
def _index(st):
    return sp.sepattn_mark_compact(st["tok"], SEP_IDS, out=st["idx_out"], ws=st["cws"])


def _index_packed(st):
    """Separators, and the first tokens of every document, into the list; per-position document bounds."""
    keep = st["keep"]
    is_sep = sp.sepattn_mark_separators(st["tok"], SEP_IDS, out=st["idx_out"][0] if keep else None)
    ds, de = st["bounds"] if keep else (torch.empty_like(st["tok"]), torch.empty_like(st["tok"]))
    for b in range(st["B"]):
        sp.sepattn_doc_bounds(st["cu"][b], st["L"], st["a"], is_sep[b], out=(ds[b], de[b]))
    idx, cnt, pre = sp.sepattn_compact_indices(is_sep, out=st["idx_out"][1:] if keep else None, ws=st["cws"])
    return is_sep, idx, cnt, pre, ds, de


def _run_train(st):
    Q, K, V, dO, a, n, scale = (st[k] for k in ("Q", "K", "V", "dO", "a", "n", "scale"))
    form = st.get("form", "plain")
    if form == "packed":
        is_sep, idx, cnt, pre, ds, de = _index_packed(st)
        O, LSE = sp.sepattn_forward_packed(Q, K, V, ds, de, idx, cnt, pre, n, scale, out=st["ows"])
        grads = sp.sepattn_backward_packed(Q, K, V, O, LSE, dO, ds, de, idx, cnt, pre, n, scale, out=st["gout"], ws=st["bws"])
        return dict(is_sep=is_sep, idx=idx, cnt=cnt, pre=pre, ds=ds, de=de, O=O, LSE=LSE, dQ=grads[0], dK=grads[1], dV=grads[2])
    is_sep, idx, cnt, pre = _index(st)
    if form == "headwise":
        O, LSE = sp.sepattn_forward_headwise(Q, K, V, idx, cnt, pre, a, st["nh"], scale, out=st["ows"])
        grads = sp.sepattn_backward_headwise(Q, K, V, O, LSE, dO, idx, cnt, pre, a, st["nh"], scale, out=st["gout"], ws=st["bws"])
    else:
        O, LSE = sp.sepattn_forward(Q, K, V, idx, cnt, pre, a, n, scale, out=st["ows"])
        grads = sp.sepattn_backward(Q, K, V, O, LSE, dO, idx, cnt, pre, a, n, scale, out=st["gout"], ws=st["bws"])
    return dict(is_sep=is_sep, idx=idx, cnt=cnt, pre=pre, O=O, LSE=LSE, dQ=grads[0], dK=grads[1], dV=grads[2])


def _run_prefill(st):
    is_sep, idx, cnt, pre = _index(st)
    O, LSE = sp.sepattn_forward(st["Q"], st["K"], st["V"], idx, cnt, pre, st["a"], st["n"], st["scale"], out=st["ows"])
    r = dict(is_sep=is_sep, idx=idx, cnt=cnt, pre=pre, O=O, LSE=LSE)
    if st["c"]:
        r["cache"] = sp.sepkv_fill_from_prefill(st["K"], st["V"], is_sep, idx, pre, st["Hq"], st["a"], st["s"], st["w"], st["c"],
                                                st["nw"], out=st["cache_out"])
    return r


def _decode(st, q, out):
    if st["rope"]:
        return sp.sepattn_decode_rope(q, st["Kc"], st["Vc"], st["sizes"], st["table"], st["a"], st["s"], st["w"], st["scale"],
                                      out=out, ws=st["ws"])
    return sp.sepattn_decode(q, st["Kc"], st["Vc"], st["sizes"], st["a"], st["s"], st["w"], st["scale"], out=out, ws=st["ws"])


def _run_generate(st):
    # the window is full: compress, then generate until it is full again (every pass ends as it began)
    Kc, Vc, flags, sizes, Hq, a, s, w = (st[k] for k in ("Kc", "Vc", "flags", "sizes", "Hq", "a", "s", "w"))
    sp.sepkv_evict_window(Kc, Vc, flags, sizes, Hq, a, s, w)
    for k, v, sep, q, out in st["steps"]:
        sp.sepkv_append(k, v, sep, Kc, Vc, flags, sizes, Hq, a, s, w)
        _decode(st, q, out)
    return dict(out=st["outs"], lse=st["lses"], Kc=Kc, Vc=Vc, flags=flags, sizes=sizes)


def run(state):
    kind = state["kind"]
    if kind == "prefill":
        return _run_prefill(state)
    if kind == "decode":
        return _decode(state, state["q"], state["out"])
    if kind == "generate":
        return _run_generate(state)
    return _run_train(state)


# ------------------------------------------------------------------------------------------------
def _pairs(L, a, n, p):
    """Expected number of visible (query, key) pairs of one sequence and head: per query the window, the
    initial tokens before it, and p of the other tokens before it."""
    def tri(m):  # 0 + 1 + ... + (m - 1)
        return m * (m - 1) // 2

    n = min(n, L)
    out = L - n  # rows whose window does not reach the start, ws = 1 .. L - n
    band = tri(n + 1) + n * out
    m = min(a, out)
    init = tri(m + 1) + m * (out - m)
    return band + init + p * (tri(out + 1) - init)


def work(case):
    c = case
    d = c["d"]
    if c["kind"] in ("decode", "generate"):
        S, Hq, Hkv = c["S"], c["Hq"], c["Hkv"]
        room = c["c"] - c["a"] - c["s"]
        T = room - c["w"]
        held = c["a"] + c["s"] + c["w"]
        if c["kind"] == "decode":
            rows, tokens = held + c["fill"] * T, 1
            extra = 0
        else:
            # the caches are read once per token (each holds one entry more than before); every token's K/V is
            # read and written once more by the append, and p of the dropped entries move
            rows, tokens = held + 0.5 * (T + 1), T
            extra = 8 * T * S * Hkv * d + 8 * c["p"] * T * S * Hkv * d
        b = tokens * (4 * S * Hkv * rows * d + 4 * S * Hq * d + 4 * S * Hq + (4 * rows * d if c["rope"] else 0)) + extra
        return {"bytes": b, "flops": tokens * 4.0 * S * Hq * rows * d}
    B, Hq, Hkv, L, a, n, p = (c[k] for k in ("B", "Hq", "Hkv", "L", "a", "n", "p"))
    es = 4 if c["kind"] == "check" else 2
    qb, kb = es * B * Hq * L * d, es * B * Hkv * L * d
    index = B * L * (4 + 1 + 4 + 4 * p)
    if c.get("form") == "packed":
        D = c["docs"]  # documents of one length have the fewest pairs
        pairs = Hq * D * _pairs(L // D, a, n, p)
        index += 8 * B * L
    elif c.get("form") == "headwise":
        pairs = sum(_pairs(L, a, nh, p) for nh in _head_windows(c))
    else:
        pairs = Hq * _pairs(L, a, n, p)
    if c["kind"] == "prefill":
        by = index + 2 * qb + 2 * kb + 4 * B * Hq * L
        if c["c"]:
            kept = min(L, a) + min(c["s"], p * max(0, L - a - c["w"])) + min(c["w"], L)
            by += 2 * es * B * Hkv * kept * d
        return {"bytes": by, "flops": 4.0 * d * B * pairs}
    # Q, K, V, dO in; O, LSE, dQ, dK, dV out
    return {"bytes": index + 4 * qb + 4 * kb + 4 * B * Hq * L, "flops": 14.0 * d * B * pairs}


def tolerance(case):
    # fp32 sums of up to a few thousand terms
    if case["kind"] == "check":
        return {"rel": 1e-5, "max": 1e-3}
    # bf16 results, bf16 operands of the second matrix product, fp32 accumulation; an element of a gradient of an
    # early token adds far more such terms than most, so its error reaches a larger part of the tensor's mean size
    return {"rel": 1e-2, "max": 0.3}

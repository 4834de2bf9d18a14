"""The work that a user of the streaming-constrained attention library has it do, as cases that can be timed.

Every case goes through the public entry points of the Python binding, as a model's attention layer would call them:
a prefill or training step of one layer over a packed batch (segment tables, rotation, attention, gradients), decoding
steps over the paged source and reasoning caches, and the arrival of a source chunk.  The structures (segment lengths,
cache lengths) follow from the case alone, the values from the seed.  Values are N(0, 1) like the benchmark's: what
normalised queries and keys look like.
"""
import numpy as np
import torch

import paper_2510_17238_amd as st

THETA = 1.0e6
PAGE = 16
TOKEN_KINDS = ("prefill", "train")


# ------------------------------------------------------------------ the cases
def _layer(name, kind, dtype, batch, tokens, src, rsn, heads, dim, layout, fused, lens):
    """One attention layer over `batch` sequences of tokens[0] .. tokens[1] tokens, segments of src / rsn tokens."""
    return {"name": name, "kind": kind, "dtype": dtype, "batch": batch, "tokens_lo": tokens[0], "tokens_hi": tokens[1],
            "src_lo": src[0], "src_hi": src[1], "rsn_lo": rsn[0], "rsn_hi": rsn[1], "q_heads": heads[0], "kv_heads": heads[1],
            "head_dim": dim, "layout": layout, "fused_rope": fused, "lens": lens}


def _cached(name, kind, layers, batch, src, rsn, new, heads, dim, fp8, side, lens):
    """`layers` layers with paged caches of src[0] .. src[1] source and rsn[0] .. rsn[1] reasoning tokens; `new` tokens
    a pass; side: source tokens appended per layer on a second stream beside the decoding (0: none)."""
    return {"name": name, "kind": kind, "layers": layers, "batch": batch, "src_lo": src[0], "src_hi": src[1],
            "rsn_lo": rsn[0], "rsn_hi": rsn[1], "new": new, "q_heads": heads[0], "kv_heads": heads[1], "head_dim": dim,
            "fp8": fp8, "side": side, "lens": lens}


def listed():
    return [
        # the smallest problem: one short exchange in fp32, as somebody tries the operator out or checks a model with it
        _layer("prefill_tiny_f32", "prefill", "f32", 1, (128, 128), (16, 16), (16, 16), (2, 1), 64, "interleaved", False, 0),
        # fp32 training step of a layer: gradients of a small batch in full precision (numerics studies, debugging)
        _layer("train_f32", "train", "f32", 2, (700, 1100), (24, 64), (32, 128), (16, 8), 128, "interleaved", False, 1),
        # prefill of a small model's layer: four sequences of about 4K tokens
        _layer("prefill_4x4k", "prefill", "bf16", 4, (3800, 4200), (24, 64), (32, 128), (16, 8), 128, "interleaved", False, 2),
        # the largest: eight long documents, 16K tokens each
        _layer("prefill_8x16k", "prefill", "bf16", 8, (16384, 16384), (64, 192), (64, 256), (32, 8), 128, "interleaved", False, 3),
        # a serving batch of many short ragged prompts, the rotation fused into the attention call
        _layer("prefill_96_short", "prefill", "bf16", 96, (60, 900), (5, 40), (8, 80), (32, 8), 128, "interleaved", True, 4),
        # fine-tuning step (forward, gradients) of the small model's layer
        _layer("train_4x4k", "train", "bf16", 4, (3800, 4200), (24, 64), (32, 128), (16, 8), 128, "interleaved", False, 5),
        # fine-tuning with heads of 64, in the grouped layout, sequences of unlike length
        _layer("train_ragged_d64", "train", "bf16", 10, (333, 3111), (5, 90), (8, 200), (16, 2), 64, "grouped", False, 6),
        # one listener: a token decoded through 36 layers over short caches, everything bound by latency
        _cached("token_batch1", "decode", 36, 1, (96, 96), (300, 300), 1, (32, 8), 128, False, 0, 7),
        # serving: 32 streams, 2K source and 1K to 6K reasoning tokens, 64 source tokens arriving per layer meanwhile
        _cached("decode_32", "decode", 3, 32, (2048, 2048), (1024, 6144), 1, (16, 8), 128, False, 64, 8),
        # the same streams over 8-bit caches
        _cached("decode_32_fp8", "decode_fp8", 3, 32, (2048, 2048), (1024, 6144), 1, (16, 8), 128, True, 0, 9),
        # 64 long streams, eight reasoning tokens stored and attended in one call (a verified draft)
        _cached("decode_64_of_8", "decode_many", 1, 64, (1024, 8192), (2048, 16384), 8, (32, 8), 128, False, 0, 10),
        # 64 streams take in a chunk of 32 source tokens and attend it over source caches of up to 8K tokens
        _cached("chunk_64", "chunk", 1, 64, (1024, 8192), (16, 16), 32, (32, 8), 128, False, 0, 11),
    ]


def _log(rng, lo, hi):
    """An integer of [lo, hi], spread over the logarithm."""
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    kind = rng.choice(("prefill", "prefill", "train", "train", "f32", "decode1", "decode", "decode", "decode_fp8", "decode_many", "chunk"))
    lens = rng.randrange(1 << 20)
    if kind in ("prefill", "train", "f32"):
        heads = rng.choice(((16, 8), (32, 8), (16, 2), (8, 4), (4, 2)))
        dim = rng.choice((64, 128, 128))
        batch = _log(rng, 1, {"prefill": 96, "train": 24, "f32": 4}[kind])
        total = _log(rng, *{"prefill": (512, 131072), "train": (512, 24576), "f32": (64, 2048)}[kind])
        top = min(max(total // batch, 17), {"prefill": 16384, "train": 8192, "f32": 1200}[kind])
        tokens = (max(16, int(top * rng.choice((0.1, 0.5, 0.95)))), top)
        src, rsn = rng.choice((((5, 40), (8, 80)), ((24, 64), (32, 128)), ((64, 192), (64, 256))))
        direction = rng.choice(TOKEN_KINDS) if kind == "f32" else kind
        case = _layer("", direction, "f32" if kind == "f32" else "bf16", batch, tokens, src, rsn, heads, dim,
                      rng.choice(("interleaved", "grouped")), kind == "prefill" and rng.random() < 0.4, lens)
    elif kind == "decode1":
        case = _cached("", "decode", rng.choice((28, 36)), rng.choice((1, 1, 2, 4)), (17, _log(rng, 40, 400)), (1, _log(rng, 16, 600)), 1,
                       rng.choice(((16, 8), (32, 8))), rng.choice((64, 128)), False, 0, lens)
    else:
        heads = rng.choice(((16, 8), (32, 8)))
        dim = rng.choice((64, 128, 128))
        batch = _log(rng, 2, 64)
        src, rsn = _log(rng, 256, 8192), _log(rng, 256, 16384)
        new = {"chunk": rng.choice((7, 32, 64)), "decode_many": rng.choice((2, 4, 8))}.get(kind, 1)
        side = rng.choice((0, 0, 32, 64)) if kind == "decode" else 0
        layers = 2 if kind == "decode" else 1
        lo = rng.choice((0.12, 0.5, 1.0))
        case = _cached("", kind, layers, batch, (max(1, int(src * lo)), src), (max(new, int(rsn * lo)), rsn) if kind != "chunk" else (16, 16),
                       new, heads, dim, kind == "decode_fp8", side, lens)
    del case["name"]
    return case


# ------------------------------------------------------------------ structures: from the case alone
def _sequence(rng, total, case):
    """(source lengths, reasoning lengths) of one sequence of `total` tokens; the last segment is cut short."""
    src, rsn, n = [], [], 0
    while n < total:
        s = min(int(rng.integers(case["src_lo"], case["src_hi"] + 1)), total - n)
        r = min(int(rng.integers(case["rsn_lo"], case["rsn_hi"] + 1)), total - n - s)
        src.append(s)
        rsn.append(r)
        n += s + r
    return np.array(src), np.array(rsn)


def _structure(case):
    """Per sequence the segment lengths, and with them (source tokens, reasoning tokens, visible pairs)."""
    rng = np.random.default_rng([case["lens"], 1])
    seqs = [_sequence(rng, int(rng.integers(case["tokens_lo"], case["tokens_hi"] + 1)), case) for _ in range(case["batch"])]
    pairs = 0
    for s, r in seqs:
        n_s, n_r = int(s.sum()), int(r.sum())
        pairs += n_s * (n_s + 1) // 2 + n_r * (n_r + 1) // 2 + int((r * np.cumsum(s)).sum())
    return seqs, pairs


def _ids(seqs, layout):
    """Stream, segment and position ids of the packed batch and its offsets."""
    streams, segments, positions, cu = [], [], [], [0]
    for s, r in seqs:
        runs = [(kind, t + 1, int(n)) for t in range(len(s)) for kind, n in ((st.ST_SOURCE, s[t]), (st.ST_REASONING, r[t]))]
        if layout == "grouped":
            runs.sort(key=lambda run: run[0])
        stream = np.concatenate([np.full(n, kind, np.int32) for kind, _, n in runs])
        position = np.zeros(len(stream), np.int32)
        for kind in (st.ST_SOURCE, st.ST_REASONING):
            position[stream == kind] = np.arange(int((stream == kind).sum()))
        streams.append(stream)
        segments.append(np.concatenate([np.full(n, t, np.int32) for _, t, n in runs]))
        positions.append(position)
        cu.append(cu[-1] + len(stream))
    return [torch.from_numpy(np.concatenate(x)).cuda() for x in (streams, segments, positions)], np.array(cu, np.int32)


def _lengths(case):
    """Cache lengths before the pass's tokens arrive (source) and with them (reasoning), per sequence."""
    rng = np.random.default_rng([case["lens"], 2])
    src = rng.integers(case["src_lo"], case["src_hi"] + 1, case["batch"]).astype(np.int32)
    rsn = rng.integers(case["rsn_lo"], case["rsn_hi"] + 1, case["batch"]).astype(np.int32)
    return src, rsn


# ------------------------------------------------------------------ inputs
def _normal(gen, *shape, dtype=torch.bfloat16):
    return torch.randn(shape, generator=gen, device="cuda", dtype=dtype)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return (_prepare_layer if case["kind"] in TOKEN_KINDS else _prepare_cached)(case, gen)


def _prepare_layer(case, gen):
    seqs, _ = _structure(case)
    (streams, segments, positions), cu = _ids(seqs, case["layout"])
    n, hq, hkv, d = int(cu[-1]), case["q_heads"], case["kv_heads"], case["head_dim"]
    dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    s = {"case": case, "ids": (segments, streams, positions), "cu": cu, "turn": 0, "plans": [None, None],
         "q": _normal(gen, n, hq, d, dtype=dtype), "k": _normal(gen, n, hkv, d, dtype=dtype), "v": _normal(gen, n, hkv, d, dtype=dtype),
         "d_out": _normal(gen, n, hq, d, dtype=dtype) if case["kind"] == "train" else None,
         # two in turn: the tables of one batch stay while the next batch's are built
         "plan_ws": [torch.empty(st.st_plan_workspace_bytes(case["batch"], n), dtype=torch.uint8, device="cuda") for _ in range(2)]}
    return s


def _caches(gen, case, lens, room):
    """A paged cache for each layer, with pages for `room` more tokens than `lens` and its page ids shuffled; the pools
    of all layers are one tensor.  Returns (caches, (k pools, v pools))."""
    pages = (int(lens.max()) + room + PAGE - 1) // PAGE
    batch, layers = case["batch"], case["layers"]
    caches = []
    for _ in range(layers):
        table = torch.randperm(batch * pages, generator=gen, device="cuda").to(torch.int32).view(batch, pages)
        caches.append(st.KVCache(batch * pages, batch, pages, case["kv_heads"], case["head_dim"], table, fp8=case["fp8"]))
    if case["fp8"]:
        return caches, None
    pools = [_normal(gen, layers, *pool.shape) for pool in (caches[0].k_pool, caches[0].v_pool)]
    for i, cache in enumerate(caches):
        cache.k_pool, cache.v_pool = pools[0][i], pools[1][i]
    return caches, pools


def _prepare_cached(case, gen):
    src, rsn = _lengths(case)
    batch, hq, hkv, d, new, side = (case[k] for k in ("batch", "q_heads", "kv_heads", "head_dim", "new", "side"))
    chunk = case["kind"] == "chunk"
    s = {"case": case, "src": torch.from_numpy(src).cuda(), "rsn": torch.from_numpy(rsn).cuda(),
         "max_src": int(src.max()), "max_rsn": int(rsn.max()), "layers": [], "stream": torch.cuda.Stream() if side else None,
         "len0": torch.from_numpy(np.stack([src, rsn - (0 if chunk or case["fp8"] else new)])).cuda()}
    s["src_after"] = s["src"] + new
    # the lengths of all layers' caches in one tensor, so that a pass can set them back with one copy
    s["len"] = torch.empty((case["layers"], 2, batch), dtype=torch.int32, device="cuda")
    s["out"] = torch.empty((case["layers"], batch, new, hq, d), dtype=torch.bfloat16, device="cuda")
    source, source_pools = _caches(gen, case, src, side + (new if chunk else 0))
    reasoning, reasoning_pools = _caches(gen, case, rsn, 0)
    s["stored"] = {"source": source_pools if chunk or side else None, "reasoning": None if chunk else reasoning_pools}
    for i in range(case["layers"]):
        caches = st.DualCache(source[i], reasoning[i])
        caches.source.appended_len, caches.reasoning.appended_len = s["len"][i, 0], s["len"][i, 1]
        if case["fp8"]:
            s["len"][i] = 0
            for which, n in ((st.ST_SOURCE, s["src"]), (st.ST_REASONING, s["rsn"])):
                top = int(n.max())
                st.st_kv_append(caches, which, _normal(gen, batch, top, hkv, d), _normal(gen, batch, top, hkv, d), n)
        s["layers"].append({"caches": caches, "out": s["out"][i], "q": _normal(gen, batch, new, hq, d), "k": _normal(gen, batch, new, hkv, d),
                            "v": _normal(gen, batch, new, hkv, d),
                            "side_k": _normal(gen, batch, side, hkv, d) if side else None,
                            "side_v": _normal(gen, batch, side, hkv, d) if side else None})
    s["len"].copy_(s["len0"].expand_as(s["len"]))
    if case["kind"] == "chunk":
        need = st.st_source_chunk_workspace_bytes(batch, hq, hkv, d, new, s["max_src"] + new)
    else:
        need = st.st_decode_workspace_bytes(batch, hq, hkv, d, new, s["max_src"], s["max_rsn"])
    s["ws"] = torch.empty(max(need, 256), dtype=torch.uint8, device="cuda")
    return s


# ------------------------------------------------------------------ one pass
def run(state):
    return (_run_layer if state["case"]["kind"] in TOKEN_KINDS else _run_cached)(state)


def _run_layer(s):
    """A batch arrives: its segment tables, then the layer -- rotation, attention, for training also the gradients."""
    case = s["case"]
    s["turn"] ^= 1
    plan = s["plans"][s["turn"]] = st.st_plan_create(*s["ids"], s["cu"], workspace=s["plan_ws"][s["turn"]])
    q, k, v, positions = s["q"], s["k"], s["v"], s["ids"][2]
    lse = torch.empty(q.shape[:2], dtype=torch.float32, device="cuda")
    if case["fused_rope"]:
        return {"out": st.st_attn_prefill_rope(q, k, v, positions, THETA, plan, lse=lse), "lse": lse}
    q, k = st.st_rope_apply_qk(q, k, positions, THETA, q_out=torch.empty_like(q), k_out=torch.empty_like(k))
    out = st.st_attn_prefill(q, k, v, plan, lse=lse)
    if case["kind"] == "prefill":
        return {"out": out, "lse": lse}
    dq, dk, dv = st.st_attn_prefill_bwd(s["d_out"], q, k, v, out, lse, plan)
    return {"out": out, "lse": lse, "dq": dq, "dk": dk, "dv": dv}


def _run_cached(s):
    """The pass's tokens go through every layer.  The caches' lengths are set back first: each pass is the same step."""
    case, side = s["case"], s["stream"]
    new, kind = case["new"], case["kind"]
    if kind != "decode_fp8":
        s["len"].copy_(s["len0"].expand_as(s["len"]))
    if side is not None:
        main = torch.cuda.current_stream()
        side.wait_stream(main)
    for layer in s["layers"]:
        caches = layer["caches"]
        if side is not None:
            st.st_kv_append_rope(caches, st.ST_SOURCE, layer["side_k"], layer["side_v"], THETA,
                                 host_len_upper_bound=s["max_src"] + case["side"], stream=side)
        if kind == "decode":
            st.st_attn_decode_dual_append(layer["q"], layer["k"], layer["v"], caches, s["src"], s["rsn"], s["max_src"], s["max_rsn"],
                                          theta_base=THETA, workspace=s["ws"], out=layer["out"])
        elif kind == "decode_fp8":
            st.st_attn_decode_dual_rope(layer["q"], caches, s["src"], s["rsn"], s["max_src"], s["max_rsn"], THETA, workspace=s["ws"], out=layer["out"])
        elif kind == "decode_many":
            st.st_kv_append_rope(caches, st.ST_REASONING, layer["k"], layer["v"], THETA, host_len_upper_bound=s["max_rsn"])
            st.st_attn_decode_dual_rope(layer["q"], caches, s["src"], s["rsn"], s["max_src"], s["max_rsn"], THETA, workspace=s["ws"], out=layer["out"])
        else:
            st.st_kv_append_rope(caches, st.ST_SOURCE, layer["k"], layer["v"], THETA, host_len_upper_bound=s["max_src"] + new)
            st.st_attn_source_chunk_rope(layer["q"], caches, s["src_after"], s["max_src"] + new, THETA, workspace=s["ws"], out=layer["out"])
    if side is not None:
        main.wait_stream(side)
    # what the pass has written: the results, the lengths, and the pools that tokens were stored in
    return {"out": s["out"], "len": s["len"], "stored": s["stored"]}


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    hq, hkv, d = case["q_heads"], case["kv_heads"], case["head_dim"]
    if case["kind"] in TOKEN_KINDS:
        seqs, pairs = _structure(case)
        n = sum(int(s.sum() + r.sum()) for s, r in seqs)
        size = 4 if case["dtype"] == "f32" else 2
        rows, keys = n * hq * d * size, n * hkv * d * size          # q or out; k or v
        forward = 2 * rows + 2 * keys + n * (12 + 4 * hq)           # three ids and the log-sum-exps
        flops = 4.0 * d * hq * pairs
        if case["kind"] == "train":                                 # d_out in, dq, dk, dv out; five products instead of two
            return {"bytes": float(forward + 2 * rows + 2 * keys), "flops": 3.5 * flops}
        return {"bytes": float(forward), "flops": flops}
    src, rsn = _lengths(case)
    new, batch, layers = case["new"], case["batch"], case["layers"]
    row = hkv * (2 * d + 8) if case["fp8"] else hkv * 4 * d         # key and value of one cached token
    fresh = batch * new * (hq * 4 * d + hkv * 4 * d)                # q, k, v in, out back
    if case["kind"] == "chunk":
        seen = int(src.sum()) + batch * new
        pairs = new * int(src.sum()) + batch * new * (new + 1) // 2
    else:
        seen = int(src.sum()) + int(rsn.sum())
        pairs = new * (seen - batch * new) + batch * new * (new + 1) // 2
    beside = batch * case["side"] * hkv * 8 * d                     # read and stored
    return {"bytes": float(layers * (seen * row + fresh + beside)), "flops": 4.0 * d * hq * pairs * layers}


def tolerance(case):
    # Four times what the path differs by from the same in 64 bits.  bf16: 2.2e-3 to 3.1e-3 in the 2-norm (the rounding
    # of the results, of the probabilities and dS and of the prescaled queries), 0.125 at most in one gradient value;
    # fp32: 1.0e-6 and 1.1e-5 (the order of the sums).
    if case.get("dtype") == "f32":
        return {"rel": 4e-6, "max": 5e-5}
    return {"rel": 1.2e-2, "max": 0.5}

"""The work that a user of this library has it do, as cases that can be timed and compared.

Four kinds of work, all through the public entry points of ``paper_2605_13111_amd.binding``:

  denoise   one denoising pass: the attention of ``layers`` layers for the chunk being generated, history and frame index
            already there (they change once per chunk, and a chunk takes several passes)
  rollout   a video from its first frame on: per chunk ``passes`` attention passes over the layers, then every layer's
            write-back (append) and the next chunk's frame index
  history   an existing video taken into the cache chunk by chunk (to continue it), then the frame index
  classify  the offline classification of the heads from their historical attention sequences

Fields: heads, head_dim, tpf (tokens per latent frame), chunk (frames generated at a time), frames (history length; of a
rollout, its end), policy / policy_seed (which frames a head keeps is fixed per model, so it belongs to the case and not
to the inputs), layout ("packed": tensors per head; "model": [tokens][heads][head_dim], the strided entry points).
"""
import math

import torch

from paper_2605_13111_amd import binding as B
from paper_2605_13111_amd import synth

DEV = "cuda:0"


def listed():
    return [
        # the smallest calls, where latency and launches are all there is: the tiny configuration (16-token frames), as one
        # attention call and as a whole short rollout
        dict(name="tiny_layer", kind="denoise", layers=1, heads=4, head_dim=64, tpf=16, chunk=3, frames=12, policy="thirds",
             policy_seed=0, layout="packed"),
        dict(name="tiny_rollout", kind="rollout", layers=1, heads=4, head_dim=64, tpf=16, chunk=3, frames=12, passes=4,
             policy="thirds", policy_seed=0, layout="packed"),
        # a small picture: frames and chunk that are multiples of nothing
        dict(name="odd_layer", kind="denoise", layers=2, heads=5, head_dim=128, tpf=333, chunk=2, frames=9, policy="drawn",
             policy_seed=7000, layout="packed"),
        # the first chunk of every video: the chunk attends to itself only
        dict(name="first_chunk", kind="denoise", layers=2, heads=12, head_dim=128, tpf=1560, chunk=3, frames=0,
             policy="drawn", policy_seed=7000, layout="model"),
        # one layer at model shape with a short history (one-layer workload of the benchmark)
        dict(name="short_layer", kind="denoise", layers=1, heads=12, head_dim=128, tpf=1560, chunk=3, frames=18,
             policy="thirds", policy_seed=0, layout="packed"),
        # the benchmark's denoising step at a one-minute horizon: eight of its thirty layers (each has its own policy
        # table), the tensors as the model holds them
        dict(name="long_step", kind="denoise", layers=8, heads=12, head_dim=128, tpf=1560, chunk=3, frames=57,
             policy="drawn", policy_seed=7000, layout="model"),
        # many heads whose key lengths are far apart (skewed workload of the benchmark)
        dict(name="skewed_layer", kind="denoise", layers=1, heads=40, head_dim=128, tpf=1560, chunk=3, frames=60,
             policy="skewed", policy_seed=0, layout="packed"),
        # a pass in the middle of a streaming rollout: one-frame chunks
        dict(name="stream_pass", kind="denoise", layers=6, heads=12, head_dim=128, tpf=1560, chunk=1, frames=20,
             policy="drawn", policy_seed=7000, layout="packed"),
        # the other head size that the library takes, at a size of real use
        dict(name="d64_layer", kind="denoise", layers=1, heads=16, head_dim=64, tpf=1560, chunk=3, frames=18,
             policy="thirds", policy_seed=0, layout="model"),
        # a rollout under the paper's own policy set (strided Anchor, capped Wave, merging Veil heads)
        dict(name="paper_rollout", kind="rollout", layers=1, heads=12, head_dim=128, tpf=1560, chunk=3, frames=30, passes=4,
             policy="paper", policy_seed=8000, layout="model"),
        # a video of 57 frames taken into the cache of one layer: appends that evict and pack
        dict(name="long_history", kind="history", layers=1, heads=12, head_dim=128, tpf=1560, chunk=3, frames=57,
             policy="drawn", policy_seed=7000, layout="packed"),
        # head classification at the paper's analysis size: 256 prompts, 30 layers x 12 heads
        dict(name="classify", kind="classify", prompts=256, heads=360, hist=69),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges, no dearer than the dearest listed one."""
    most = max(_cost(c) for c in listed())
    while True:
        kind = rng.choices(["denoise", "rollout", "history", "classify"], [6, 3, 2, 1])[0]
        if kind == "classify":
            c = dict(kind=kind, prompts=_log_int(rng, 4, 256), heads=_log_int(rng, 12, 360), hist=_log_int(rng, 24, 240))
        else:
            c = dict(kind=kind, layers=rng.randint(1, 8) if kind == "denoise" else 1, heads=_log_int(rng, 4, 40),
                     head_dim=rng.choice([128, 128, 128, 64]), tpf=_log_int(rng, 16, 1560) if rng.random() < 0.6 else 1560,
                     chunk=rng.randint(1, 3), frames=0, policy=rng.choice(["thirds", "drawn", "drawn", "paper", "windows", "skewed"]),
                     policy_seed=rng.randint(0, 9999), layout=rng.choice(["packed", "model"]))
            if kind == "rollout":
                c["passes"] = rng.choice([2, 4])
                c["frames"] = c["chunk"] * rng.randint(3, 12)
            elif kind == "history":
                c["frames"] = c["chunk"] * rng.randint(4, 20)
            else:
                c["frames"] = rng.randint(0, 60)
        if _cost(c) <= most:
            return c


def _policies(c, layer):
    """One layer's policy table, its pool regions exactly as large as the history needs."""
    H, T, seed = c["heads"], max(c["frames"], 1), c["policy_seed"] + layer
    if c["policy"] == "thirds":                       # Anchor (all) / Wave (every 2nd) / Veil (first + last 3)
        third = (H + 2) // 3
        pols = ([synth.anchor_all(T)] * third + [synth.wave(2, T)] * third + [synth.veil(1, 3)] * third)[:H]
    elif c["policy"] == "skewed":                     # one head in five keeps everything
        n_all = max(1, H // 5)
        pols = [synth.anchor_all(T)] * n_all + [synth.veil(1, 3)] * (H - n_all)
    elif c["policy"] == "drawn":
        pols = synth.drawn_policies(H, seed, T)
    elif c["policy"] == "windows":
        pols = synth.head_window_policies(H, seed)
    else:
        pols = synth.paper_default_policies(H, seed, T, lambda p: B.slots_needed(p, T))
    return [p._replace(slots=max(1, B.slots_needed(p, T))) for p in pols]


def _tokens(shape, seed, layout):
    """bf16 N(0, 1) of logical shape [..., heads, tokens, head_dim]; layout "model" holds [..., tokens, heads, head_dim]."""
    if layout == "packed":
        return synth.randn_bf16(shape, seed, device=DEV)
    return synth.randn_bf16(shape[:-3] + (shape[-2], shape[-3], shape[-1]), seed, device=DEV).transpose(-3, -2)


def _frames(t, tpf):
    """[heads, tokens, head_dim] -> [heads, frames, tpf, head_dim], no copy."""
    return t.unflatten(1, (-1, tpf))


def _append(c):
    return B.pf_cache_append_strided if c["layout"] == "model" else B.pf_cache_append


def _attn(c):
    return B.pf_ragged_attn_fwd_strided if c["layout"] == "model" else B.pf_ragged_attn_fwd


def prepare(case, seed):
    c = case
    base = 1000003 * (int(seed) % (1 << 31))
    if c["kind"] == "classify":
        logits, _ = synth.head_logits(c["prompts"], c["heads"], c["hist"], base)
        return {"case": c, "logits": logits.to(DEV)}
    H, D, tpf, n = c["heads"], c["head_dim"], c["tpf"], c["chunk"]
    Lq = n * tpf
    layers, ws_bytes = [], 0
    for layer in range(c["layers"]):
        s0 = base + 100000 * (layer + 1)
        pool = B.Pool(_policies(c, layer), tpf, D, device=DEV)
        L = {"pool": pool}
        B.pf_pool_reset(pool)
        if c["kind"] == "denoise":
            for t0 in range(0, c["frames"], n):
                k, v = (_tokens((H, min(n, c["frames"] - t0) * tpf, D), s0 + 10 * t0 + i, c["layout"]) for i in (0, 1))
                score = synth.frame_scores(H, k.shape[1] // tpf, s0 + 10 * t0 + 2, device=DEV)
                _append(c)(pool, _frames(k, tpf), _frames(v, tpf), score)
            L["q"], L["k"], L["v"] = (_tokens((H, Lq, D), s0 + 5000 + i, c["layout"]) for i in (0, 1, 2))
        else:
            n_chunks = c["frames"] // n
            tensors = (n_chunks, c.get("passes", 1))
            if c["kind"] == "rollout":
                L["q"] = _tokens(tensors + (H, Lq, D), s0, c["layout"])
            L["k"], L["v"] = (_tokens(tensors + (H, Lq, D), s0 + 1 + i, c["layout"]) for i in (0, 1))
            L["score"] = synth.frame_scores(n_chunks * H, n, s0 + 3, device=DEV).unflatten(0, (n_chunks, H))
        if "q" in L:
            L["out"] = torch.empty_like(L["q"])        # keeps the strides
            ws_bytes = max(ws_bytes, B.pf_attn_workspace_bytes(pool, Lq))
        L["index"] = B.Index(pool, Lq)
        if c["kind"] == "denoise":
            B.pf_build_index(pool, L["index"], Lq)
        layers.append(L)
    # the layers run one after another and share one workspace
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device=DEV) if ws_bytes else None
    return {"case": c, "layers": layers, "workspace": ws, "Lq": Lq}


def _cache_state(L):
    pool, index = L["pool"], L["index"]
    return [pool.k_pool.view(torch.int16), pool.v_pool.view(torch.int16), pool.n_frames, pool.frame_ids, pool.frame_score,
            index.sel_count, index.sel_frames, index.sel_slots, index.cu_seqlens]


def run(state):
    c = state["case"]
    if c["kind"] == "classify":
        return B.pf_classify_heads(state["logits"])
    layers, ws, Lq = state["layers"], state["workspace"], state["Lq"]
    attn, append = _attn(c), _append(c)
    if c["kind"] == "denoise":
        for L in layers:
            attn(L["pool"], L["index"], L["q"], L["k"], L["v"], L["out"], ws)
        return [L["out"] for L in layers]
    for L in layers:                                   # a new video starts from empty pools
        B.pf_pool_reset(L["pool"])
        if c["kind"] == "rollout":
            B.pf_build_index(L["pool"], L["index"], Lq)
    for ci in range(c["frames"] // c["chunk"]):
        for p in range(c.get("passes", 0)):
            for L in layers:
                attn(L["pool"], L["index"], L["q"][ci, p], L["k"][ci, p], L["v"][ci, p], L["out"][ci, p], ws)
        for L in layers:
            append(L["pool"], _frames(L["k"][ci, -1], c["tpf"]), _frames(L["v"][ci, -1], c["tpf"]), L["score"][ci])
            if c["kind"] == "rollout":
                B.pf_build_index(L["pool"], L["index"], Lq)
    if c["kind"] == "history":
        for L in layers:
            B.pf_build_index(L["pool"], L["index"], Lq)
    return [([L["out"]] if "out" in L else []) + _cache_state(L) for L in layers]


def work(case):
    c = case
    if c["kind"] == "classify":
        n = c["prompts"] * c["heads"]
        # sequences in, types and periods out; a real spectrum of hist-1 points per sequence (5 N log2 N / 2)
        N = max(c["hist"] - 1, 2)
        return {"bytes": n * (4.0 * c["hist"] + 12) + 4.0 * c["heads"], "flops": n * 2.5 * N * math.log2(N)}
    H, D, tpf, n = c["heads"], c["head_dim"], c["tpf"], c["chunk"]
    Lq, frame = n * tpf, tpf * D * 2.0
    bytes_, flops = 0.0, 0.0
    for layer in range(c["layers"]):
        pols = _policies(c, layer)

        def attention(T):                              # q in, out written, every attended key and value read once
            keys = sum(B.pf_selected_count(p, T) * tpf + Lq for p in pols)
            return 2.0 * 2 * H * Lq * D + 2.0 * 2 * keys * D, 4.0 * Lq * keys * D

        if c["kind"] == "denoise":
            b, f = attention(c["frames"])
            bytes_, flops = bytes_ + b, flops + f
            continue
        for T in range(0, c["frames"], n):
            if c["kind"] == "rollout":
                b, f = attention(T)
                bytes_, flops = bytes_ + c["passes"] * b, flops + c["passes"] * f
            bytes_ += 2.0 * 2 * H * n * frame          # K and V of the new frames, read and written
    return {"bytes": bytes_, "flops": flops}


def _cost(c):
    w = work(c)
    return w["bytes"] / 4e12 + w["flops"] / 0.8e15


def tolerance(case):
    """Attention: bf16 in and out, fp32 accumulation, softmax weights rounded to bf16.  Measured over the listed cases:
    the path against itself with its sums cut elsewhere differs by rel 2.6e-3 .. 3.1e-3, max 1.5e-2 .. 3.1e-2, and against
    the same attention in 64 bits by rel 2.4e-3, max 9e-3; stated are about three to four times as much.  Cache and index contents are
    copies and whole numbers: the same bits.  The classification takes its decisions in 64 bits; its periods are exact
    quotients of whole numbers."""
    if case["kind"] in ("history", "classify"):
        return "exact"
    return {"rel": 1e-2, "max": 1e-1, "differ": 0.0}

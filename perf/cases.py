"""The work that a program using this library has it do, as cases that can be timed and compared.

Every case is one pass through public entry points of the ctypes binding: a whole denoising step or
denoising loop of a small model, single bf16 blocks, the layers of an FP8 block, the cache-update
pass, the block-causal attention on its own, and the parts of a step that are called on their own
(the timestep's embedding, the patch and action embedding, the output head).

`listed` gives the cases, `draw` more of the same ranges; `prepare` builds what a program holds
before the call (weights, caches, plans, workspaces), `run` is the pass, `exact` the same outputs in
64 bits from plain torch, `work` the bytes and operations a pass cannot do without.
"""
import math

import torch

import paper_2602_15922_amd as wam

LATENT_CH, ACT_DIM, FREQ_DIM, EPS = 16, 16, 256, 1e-6
PATCH = LATENT_CH * 4
V_SCALE = 16.0 / 448.0  # an FP8 value cache's calibrated scale: these values stay below 16

# width -> (heads, head size, FFN width): the small test model, two generic mid sizes and the 14B class
MODELS = {512: (8, 64, 2048), 1536: (12, 128, 8960), 3072: (24, 128, 12288), 5120: (40, 128, 13824)}


def listed():
    return [
        # a small policy's whole denoising step for two robots: latency, launches
        dict(name="step_d512", kind="step", d=512, layers=3, B=2, F=2, Hl=16, Wl=16, A=16, cached=1, Lc=32,
             text_dim=512, text_cached=False),
        # its whole action chunk: four guided UniPC steps, the text projected once
        dict(name="denoise_d512", kind="denoise", d=512, layers=3, B=2, F=2, Hl=16, Wl=16, A=16, cached=1, Lc=32,
             text_dim=512, steps=4, order=2, cfg_scale=3.0),
        # one block of a mid-size model, odd row counts, a short instruction
        dict(name="block_d1536_odd", kind="block", d=1536, B=1, F=2, Hl=30, Wl=38, A=17, cached=2, Lc=77),
        # one 14B-class block for a single 256-pixel camera (two latent frames of 32 x 32)
        dict(name="block_14b_256px", kind="block", d=5120, B=1, F=2, Hl=32, Wl=32, A=32, cached=2, Lc=512),
        # one 14B-class block at 480p (60 x 104 latents), two cached chunks
        dict(name="block_14b_480p", kind="block", d=5120, B=1, F=2, Hl=60, Wl=104, A=32, cached=2, Lc=512),
        # FP8 deployment, layer by layer (a whole FP8 block amplifies one changed rounding into the size of its
        # quantization error, so only single layers can be compared): the QKV projection into the FP8 cache ...
        dict(name="qkv_14b_fp8_480p", kind="qkv8", d=5120, B=1, F=2, Hl=60, Wl=104, A=32, cached=2),
        # ... the attention over that cache ...
        dict(name="attn_14b_fp8_480p", kind="attn", B=1, H=40, Dh=128, chunk=3152, cached=2, chunks=1, fp8=True),
        # ... and the FFN, here for the 256-pixel camera
        dict(name="ffn_14b_fp8_256px", kind="ffn8", d=5120, B=1, F=2, Hl=32, Wl=32, A=32),
        # the context prefill: one clean 480p frame into an empty cache
        dict(name="prefill_14b_frame", kind="update", d=5120, layers=2, B=1, F=1, Hl=60, Wl=104, A=0, cached=0,
             chunks=1, Lc=512, text_dim=4096),
        # block-causal attention of a small model over a masked five-chunk history of odd chunk sizes
        dict(name="attn_masked_odd", kind="attn", B=2, H=8, Dh=64, chunk=141, cached=1, chunks=4, fp8=False),
        # the two ends of a 480p step: patches and actions in, velocities out
        dict(name="ends_14b_480p", kind="ends", d=5120, B=1, F=2, Hl=60, Wl=104, A=32),
        # the timestep's modulation, once per denoising step
        dict(name="time_14b", kind="time", d=5120, B=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any kind, sizes over the whole range (over their logarithm), odd ones among them."""
    most = max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(["step", "step", "denoise", "block", "block", "qkv8", "ffn8", "update", "attn", "ends", "time"])
        d = rng.choice([m for m in sorted(MODELS) if kind != "qkv8" or MODELS[m][1] == 128])
        grid = dict(F=rng.randint(1, 3), Hl=2 * _log(rng, 5, 30), Wl=2 * _log(rng, 5, 52), A=rng.randint(5, 48))
        text = dict(Lc=_log(rng, 24, 512), text_dim=512 if d == 512 else 4096)
        B, cached = rng.choice([1, 1, 2]), rng.randint(0, 3)
        if kind == "step":
            c = dict(kind=kind, d=d, layers=rng.randint(1, 3), B=B, **grid, cached=cached, **text,
                     text_cached=rng.random() < 0.5)
        elif kind == "denoise":
            d = 512
            c = dict(kind=kind, d=d, layers=rng.randint(1, 4), B=2, F=2, Hl=2 * rng.randint(5, 12),
                     Wl=2 * rng.randint(5, 12), A=rng.randint(5, 48), cached=cached, Lc=_log(rng, 24, 128),
                     text_dim=512, steps=rng.randint(2, 5), order=rng.randint(1, 2), cfg_scale=3.0)
        elif kind == "block":
            c = dict(kind=kind, d=d, B=B, **grid, cached=cached, Lc=text["Lc"])
        elif kind == "update":
            c = dict(kind=kind, d=d, layers=rng.randint(1, 2), B=B, **dict(grid, A=0), cached=cached,
                     chunks=rng.randint(1, 3), **text)
            c["F"] *= c["chunks"]
        elif kind == "attn":
            H, Dh = rng.choice([(8, 64), (12, 128), (24, 128), (40, 128)])
            c = dict(kind=kind, B=B, H=H, Dh=Dh, chunk=_log(rng, 60, 3200), cached=cached, chunks=rng.randint(1, 4),
                     fp8=Dh == 128 and rng.random() < 0.5)
        elif kind == "qkv8":
            c = dict(kind=kind, d=d, B=B, **grid, cached=cached)
        elif kind in ("ffn8", "ends"):
            c = dict(kind=kind, d=d, B=B, **grid)
        else:
            c = dict(kind=kind, d=d, B=rng.randint(1, 4))
        if _cost(c) <= most:
            return c


# ------------------------------------------------------------------------------------------ sizes
def _rows(c):
    lv = c["F"] * (c["Hl"] // 2) * (c["Wl"] // 2)
    return lv, lv + c["A"]


def _chunk_rows(c):
    """Rows of one chunk: those of a denoising call, or those of each chunk an update pass appends."""
    return _rows(c)[1] // c.get("chunks", 1)


def _frames(c):
    """Latent frames of one chunk."""
    return c["F"] // c.get("chunks", 1)


def _layout(c):
    """(current rows, cached rows, visible keys summed over the current rows)."""
    if c["kind"] == "time":
        return 0, 0, 0
    n = c["chunk"] if c["kind"] == "attn" else _chunk_rows(c)
    chunks, cached = c.get("chunks", 1), c.get("cached", 0)
    return n * chunks, n * cached, sum(n * n * (cached + i + 1) for i in range(chunks))


def _block_work(c, ctx_kv=False):
    d = c["d"]
    ffn = MODELS[d][2]
    L, cached, seen = _layout(c)
    B, Lc = c["B"], c["Lc"]
    params = 6 * d * d + 2 * d * ffn
    flops = 2 * B * L * params + 4 * B * d * seen + 4 * B * d * L * Lc
    size = 2 * params + 4 * B * d * (cached + L) + 8 * B * L * d
    if ctx_kv:
        size += 4 * B * Lc * d
    else:
        flops += 4 * B * Lc * d * d
        size += 4 * d * d + 2 * B * Lc * d
    return size, flops


def _time_work(c):
    d, B = c["d"], c["B"]
    return 2 * (FREQ_DIM * d + 7 * d * d) + 28 * B * d, 2 * B * (FREQ_DIM * d + 7 * d * d)


def _text_work(c):
    d, n, t = c["d"], c["B"] * c["Lc"], c["text_dim"]
    return 2 * (t * d + d * d + n * t + n * d), 2 * n * (t * d + d * d)


def _ends_work(c, keep_x, head=True):
    d, B = c["d"], c["B"]
    lv, L = _rows(c)
    size = 2 * d * (PATCH + ACT_DIM) * (2 if head else 1) + (2 + 4 * head) * B * (lv * PATCH + c["A"] * ACT_DIM)
    if keep_x:
        size += 8 * B * L * d  # the residual goes out and comes in again
    return size, 2 * B * d * (lv * PATCH + c["A"] * ACT_DIM) * (2 if head else 1)


def work(case):
    c, kind = case, case["kind"]
    if kind == "attn":
        L, cached, seen = _layout(c)
        d = c["H"] * c["Dh"]
        wide = 1 if c["fp8"] else 2
        size = c["B"] * d * (wide * (L + 2 * (cached + L)) + 2 * L)
        flops = 4 * c["B"] * d * seen
    elif kind == "block":
        size, flops = _block_work(c)
    elif kind == "qkv8":  # the bf16 projection is an output too
        d, M = c["d"], c["B"] * _rows(c)[1]
        size, flops = 3 * d * d + M * d * (4 + 6 + 3), 6 * M * d * d
    elif kind == "ffn8":
        d, M, ffn = c["d"], c["B"] * _rows(c)[1], MODELS[c["d"]][2]
        size, flops = 2 * d * ffn + 8 * M * d, 4 * M * d * ffn
    elif kind == "ends":
        size, flops = _ends_work(c, keep_x=True)
    elif kind == "time":
        size, flops = _time_work(c)
    else:
        n = c["layers"]
        bs, bf = _block_work(c, ctx_kv=c.get("text_cached", False))
        bs -= 8 * c["B"] * _layout(c)[0] * c["d"]  # between layers the residual is the framework's own
        parts = [_time_work(c), _ends_work(c, keep_x=False, head=kind != "update")]
        if kind == "update":  # the last layer stops after its K|V projection, and no text reaches it
            d, L = c["d"], _layout(c)[0]
            parts.append((4 * d * d + 4 * c["B"] * L * d, 4 * c["B"] * L * d * d))
            n -= 1
        if n and not c.get("text_cached", False):
            parts.append(_text_work(c))
        size = n * bs + sum(p[0] for p in parts)
        flops = n * bf + sum(p[1] for p in parts)
        if kind == "denoise":  # the text is projected once; every step runs the rest
            ts, tf = _text_work(c)
            ck = 4 * c["B"] * c["Lc"] * c["d"] ** 2 * n
            flops = c["steps"] * (flops - tf - ck) + tf + ck
            size = c["steps"] * (size - ts) + ts
    return {"bytes": size, "flops": flops}


def _cost(c):
    w = work(c)
    return w["flops"] / 2.5e15 + w["bytes"] / 8e12


def tolerance(case):
    """About four times what these paths change by when all their sums run in another order (the same network with
    its channels, heads and FFN columns permuted), or what the result's own rounding allows."""
    kind = case["kind"]
    if kind == "attn":  # probabilities in bf16, or in E4M3 relative to a running maximum
        return {"rel": 3e-2 if case["fp8"] else 6e-3}
    return {"time": {"rel": 2e-6}, "ends": {"rel": 4e-3}, "qkv8": {"rel": 1.2e-3, "max": 0.06, "differ": 6e-3},
            "ffn8": {"rel": 4e-3, "max": 0.2}, "step": {"rel": 1.6e-2}, "block": {"rel": 1e-2}, "denoise": {"rel": 1.2e-2},
            "update": {"rel": 1.6e-2}}[kind]


# ------------------------------------------------------------------------------------------ inputs
class _Draws:
    """Normal values on the GPU from one seeded stream."""

    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(int(seed))

    def __call__(self, shape, std=1.0, dtype=torch.bfloat16, mean=0.0):
        return torch.empty(shape, dtype=dtype, device="cuda").normal_(mean, std, generator=self.gen)

    def f32(self, shape, std=1.0, mean=0.0):
        return self(shape, std, torch.float32, mean)

    def uniform(self, shape):
        return torch.empty(shape, device="cuda").uniform_(0.02, 0.98, generator=self.gen)


def _block_inputs(rnd, d):
    ffn = MODELS[d][2]
    shapes = dict(w_qkv=(3 * d, d), w_o=(d, d), w_cq=(d, d), w_ckv=(2 * d, d), w_co=(d, d), w_f1=(ffn, d), w_f2=(d, ffn))
    t = {n: rnd(s, 0.02) for n, s in shapes.items()}
    for n, s in shapes.items():
        t["b" + n[1:]] = rnd.f32(s[0], 0.05)
    t["mod6"] = rnd.f32((6, d), 0.1)
    t["lnc_gamma"], t["lnc_beta"] = rnd.f32(d, 0.1, 1.0), rnd.f32(d, 0.1)
    return t


def _top_inputs(rnd, d, text_dim, parts):
    shapes = {}
    if "time" in parts:
        shapes.update(w_t1=(d, FREQ_DIM), w_t2=(d, d), w_t6=(6 * d, d))
    if "text" in parts:
        shapes.update(w_x1=(d, text_dim), w_x2=(d, d))
    if "ends" in parts:
        shapes.update(w_patch=(d, PATCH), w_ain=(d, ACT_DIM), w_hv=(PATCH, d), w_ha=(ACT_DIM, d))
    t = {n: rnd(s, 0.02) for n, s in shapes.items()}
    for n, s in shapes.items():
        t["b" + n[1:]] = rnd.f32(s[0], 0.05)
    if "ends" in parts:
        t["head_mod2"] = rnd.f32((2, d), 0.1)
    return t


def _inputs(case, seed):
    """The seeded tensors of a case (made the same way for the pass and for its 64-bit value)."""
    c, kind, rnd = case, case["kind"], _Draws(seed)
    s = {}
    if kind == "attn":
        L, cached, _ = _layout(c)
        s["q"] = rnd((c["B"], L, c["H"], c["Dh"]))
        s["k"] = rnd((c["B"], cached + L, c["H"], c["Dh"]))
        s["v"] = rnd((c["B"], cached + L, c["H"], c["Dh"]))
        return s
    d, B = c["d"], c["B"]
    H, Dh, ffn = MODELS[d]
    if kind == "time":
        s["top"], s["t"] = _top_inputs(rnd, d, 0, ("time",)), rnd.uniform((B,))
        return s
    if kind == "ends":
        s["top"], s["e"] = _top_inputs(rnd, d, 0, ("ends",)), rnd.f32((B, d), 0.5)
    if kind in ("ends", "step", "denoise", "update"):
        s["z"] = rnd((B, LATENT_CH, c["F"], c["Hl"], c["Wl"]))
        s["a"] = rnd((B, c["A"], ACT_DIM))
    if kind == "ends":
        return s
    L, cached, _ = _layout(c)
    if kind in ("block", "qkv8", "ffn8"):
        s["x"] = rnd.f32((B, L, d))
        s["e0"] = rnd.f32((B, 6, d), 0.5)
    if kind in ("qkv8", "ffn8"):
        s["mod6"] = rnd.f32((6, d), 0.1)
        for n, shape in {"qkv8": [("w", (3 * d, d))], "ffn8": [("w1", (ffn, d)), ("w2", (d, ffn))]}[kind]:
            s[n], s["b" + n[1:]] = rnd(shape, 0.02), rnd.f32(shape[0], 0.05)
        return s
    n = 1 if kind == "block" else c["layers"]
    s["blocks"] = [_block_inputs(rnd, d) for _ in range(n)]
    s["kc"] = [rnd((B, cached + L, H, Dh)) for _ in range(n)]
    s["vc"] = [rnd((B, cached + L, H, Dh)) for _ in range(n)]
    if kind == "block":
        s["ctx"] = rnd((B, c["Lc"], d))
        return s
    s["top"] = _top_inputs(rnd, d, c["text_dim"], ("time", "text", "ends"))
    s["t"] = torch.ones(B, device="cuda") if kind == "update" else rnd.uniform((B,))
    s["text"] = rnd((B, c["Lc"], c["text_dim"]))
    if c.get("text_cached"):
        s["ctx_kv"] = [rnd((B, c["Lc"], 2 * d)) for _ in range(n)]
    if kind == "denoise":
        s["x0"] = rnd.f32((1, s["z"][0].numel() + s["a"][0].numel()))
    return s


def _positions(c):
    """Positions of the current rows: chunk after chunk, after the cached ones."""
    import numpy as np

    f, chunks = _frames(c), c.get("chunks", 1)
    return np.concatenate([wam.wam_chunk_positions(c["cached"] + i, f, c["Hl"] // 2, c["Wl"] // 2, c["A"])
                           for i in range(chunks)])


def _workspace(n):
    return torch.empty(max(int(n), 256), dtype=torch.uint8, device="cuda")


def _schedule(c):
    n = c["steps"]
    return [0.02 + 0.98 * i / n for i in range(n + 1)]


def _rope(c, Dh):
    return [torch.from_numpy(t).cuda() for t in wam.wam_rope_tables(_positions(c), Dh)]


def _mx(x):
    """E4M3 codes of a [B][L][H][128] tensor in blocks of 32 with their exponent words."""
    B, n, H, Dh = x.shape
    codes = torch.empty(x.shape, dtype=torch.uint8, device="cuda")
    exps = torch.empty((B, n, H), dtype=torch.int32, device="cuda")
    wam.wam_quantize_mx_fp8(x.view(B * n, H * Dh), codes.view(B * n, H * Dh), exps.view(torch.uint8).view(B * n, H * 4))
    return codes, exps


def _rows8(w):
    """E4M3 codes of a weight matrix with one scale per row."""
    codes = torch.empty(w.shape, dtype=torch.uint8, device="cuda")
    scale = torch.empty(w.shape[0], device="cuda")
    wam.wam_quantize_rows_fp8(w, codes, scale)
    return codes, scale


# ------------------------------------------------------------------------------------------ the pass
def prepare(case, seed):
    c, kind = case, case["kind"]
    s = _inputs(c, seed)
    s["case"] = c
    if kind == "attn":
        s["o"] = torch.empty_like(s["q"])
        s["layout"] = wam.append_chunks([c["chunk"]] * c["cached"], [c["chunk"]] * c["chunks"])
        if c["fp8"]:
            s["q8"], s["k8"] = _mx(s["q"]), _mx(s["k"])
            s["v8"] = torch.empty(s["v"].shape, dtype=torch.uint8, device="cuda")
            wam.wam_quantize_scaled_fp8(s["v"], V_SCALE, s["v8"])
        return s
    d, B = c["d"], c["B"]
    H, Dh, ffn = MODELS[d]
    L, cached, _ = _layout(c)
    if kind in ("qkv8", "ffn8"):
        M = B * L
        s["q8"], s["qs"] = torch.empty((M, d), dtype=torch.uint8, device="cuda"), torch.empty(M, device="cuda")
        if kind == "ffn8":
            s["w1"], s["w2"] = _rows8(s["w1"]), _rows8(s["w2"])
            s["u8"] = torch.empty((M, ffn), dtype=torch.uint8, device="cuda")
            s["ue"] = torch.empty(ffn // 128 * 4 * M, dtype=torch.uint8, device="cuda")
            return s
        s["w"] = _rows8(s["w"])
        s["cos"], s["sin"] = _rope(c, Dh)
        s["qkv"] = torch.empty((B, L, 3 * d), dtype=torch.bfloat16, device="cuda")
        # the caches' earlier rows are not read here
        codes, words = (B, cached + L, H, Dh), (B, cached + L, H)
        s["k8"], s["v8"] = (torch.zeros(codes, dtype=torch.uint8, device="cuda") for _ in range(2))
        s["ke"] = torch.zeros(words, dtype=torch.int32, device="cuda")
        s["rot8"] = torch.empty((B, L, H, Dh), dtype=torch.uint8, device="cuda")
        s["rote"] = torch.empty((B, L, H), dtype=torch.int32, device="cuda")
        return s
    dims = wam.make_dims(d, H, Dh, ffn, len(s.get("blocks", ())), LATENT_CH, ACT_DIM, c.get("text_dim", 4096), FREQ_DIM, EPS)
    if kind == "block":
        s["cos"], s["sin"] = _rope(c, Dh)
        s["dims"], s["weights"] = dims, wam.make_block_weights(s["blocks"][0])
        s["layout"] = wam.cached_chunks(cached, L)
        s["ws"] = _workspace(wam.wam_block_workspace_bytes(dims, B, L, c["Lc"]))
        return s
    m = s["model"] = wam.make_model(dims, s["top"], s.get("blocks", []))
    if kind == "time":
        s["e"], s["e0"] = torch.empty((B, d), device="cuda"), torch.empty((B, 6, d), device="cuda")
        s["ws"] = _workspace(wam.wam_time_embed_workspace_bytes(dims, B))
        return s
    s["vv"] = torch.empty(s["z"].shape, device="cuda")
    s["va"] = torch.empty(s["a"].shape, device="cuda")
    if kind == "ends":
        s["x"] = torch.empty((B, L, d), device="cuda")
        s["ws"] = _workspace(max(wam.wam_embed_workspace_bytes(dims, B, c["F"], c["Hl"], c["Wl"]),
                                 wam.wam_head_workspace_bytes(dims, B, c["F"], c["Hl"], c["Wl"], c["A"])))
        return s
    s["cos"], s["sin"] = _rope(c, Dh)
    n = _chunk_rows(c)
    layout = wam.append_chunks([n] * c["cached"], [n] * c.get("chunks", 1))
    head = kind != "update"
    s["io"] = wam.make_step_io(s["z"], s["a"], s["t"], s["text"], s["kc"], s["vc"], s["cos"], s["sin"], cached, layout,
                               s["vv"] if head else None, s["va"] if head else None, ctx_kv=s.get("ctx_kv"))
    if kind == "denoise":
        s["x"] = torch.empty_like(s["x0"])
        s["params"] = wam.make_denoise_params(_schedule(c), s["x"], cfg=True, cfg_scale=c["cfg_scale"],
                                              solver=wam.WAM_SOLVER_UNIPC, order=c["order"])
        s["ws"] = _workspace(wam.wam_denoise_workspace_bytes(m, s["io"], s["params"]))
    elif kind == "update":
        s["ws"] = _workspace(wam.wam_update_workspace_bytes(m, s["io"]))
    else:
        s["ws"] = _workspace(wam.wam_step_workspace_bytes(m, s["io"]))
    return s


def _norm8(s, first):
    """The modulated LayerNorm before an FP8 projection: rows first .. first + 1 of the modulation."""
    c, m, e = s["case"], s["mod6"], s["e0"]
    wam.wam_adaln_ln_mod_fp8(s["x"], s["q8"], s["qs"], EPS, s["x"].shape[1], shift_a=m[first], shift_v=e[:, first],
                             scale_a=m[first + 1], scale_v=e[:, first + 1], mod_stride=6 * c["d"])


def run(state):
    s, c = state, state["case"]
    kind = c["kind"]
    if kind == "attn":
        if c["fp8"]:
            wam.wam_attn_blockcausal_fp8(*s["q8"], *s["k8"], s["v8"], V_SCALE, s["o"], s["layout"])
        else:
            wam.wam_attn_blockcausal(s["q"], s["k"], s["v"], s["o"], s["layout"])
        return s["o"]
    if kind == "time":
        wam.wam_time_embed_fwd(s["model"], s["t"], s["e"], s["e0"], s["ws"])
        return s["e"], s["e0"]
    if kind == "ends":
        wam.wam_embed_fwd(s["model"], s["z"], s["a"], s["x"], s["ws"])
        wam.wam_head_fwd(s["model"], s["x"], s["e"], s["vv"], s["va"], s["ws"])
        return s["x"], s["vv"], s["va"]
    L, cached, _ = _layout(c)
    if kind == "qkv8":
        H, Dh, _ = MODELS[c["d"]]
        _norm8(s, 0)
        wam.wam_gemm_fp8(s["q8"], s["w"][0], s["qkv"].view(-1, 3 * c["d"]), wam.WAM_EPI_BF16, s["qs"], s["w"][1], bias=s["b"])
        wam.wam_rope_qkv_fp8(s["qkv"], s["cos"], s["sin"], s["rot8"], s["rote"], s["k8"], s["ke"], s["v8"], V_SCALE,
                             cached, H, Dh)
        return s["qkv"], s["rot8"], s["rote"], s["k8"][:, cached:], s["ke"][:, cached:], s["v8"][:, cached:]
    if kind == "ffn8":  # x += gate (gelu(LN(x) W1^T + b1) W2^T + b2), in place
        M = s["q8"].shape[0]
        _norm8(s, 3)
        wam.wam_gemm_fp8_mx(s["q8"], s["w1"][0], s["u8"], wam.WAM_EPI_GELU_BF16, s["w1"][1], a_scale=s["qs"],
                            out_exp=s["ue"], o_lde=4 * M, bias=s["b1"])
        wam.wam_gemm_fp8_mx(s["u8"], s["w2"][0], s["x"].view(M, -1), wam.WAM_EPI_RESID_F32, s["w2"][1], a_exp=s["ue"],
                            a_lde=4 * M, bias=s["b2"], gate_a=s["mod6"][5], gate_v=s["e0"][:, 5],
                            gate_stride=6 * c["d"], gate_rows=L)
        return s["x"]
    if kind == "block":  # the residual is updated in place, as in a stack of blocks
        wam.wam_dit_block_fwd(s["dims"], s["weights"], s["x"], s["e0"], s["cos"], s["sin"], s["kc"][0], s["vc"][0],
                              cached, s["layout"], ctx=s["ctx"], ws=s["ws"])
        return s["x"], s["kc"][0][:, cached:], s["vc"][0][:, cached:]
    new = [t[:, cached:] for t in s["kc"] + s["vc"]]
    if kind == "step":
        wam.wam_dit_step_fwd(s["model"], s["io"], s["ws"])
        return [s["vv"], s["va"]] + new
    if kind == "update":
        wam.wam_dit_update_fwd(s["model"], s["io"], s["ws"])
        return new
    s["x"].copy_(s["x0"])  # the chunk starts from its noise
    wam.wam_denoise_chunk(s["model"], s["io"], s["params"], s["ws"])
    return s["x"], s["vv"], s["va"]


# ------------------------------------------------------------------------------------------ 64 bits
def _lin(x, w, b):
    return x @ w.double().T + b.double()


def _gelu(x):
    return 0.5 * x * (1 + torch.tanh(math.sqrt(2 / math.pi) * (x + 0.044715 * x ** 3)))


def _silu(x):
    return x / (1 + torch.exp(-x))


def _norm(x):
    m = x.mean(-1, keepdim=True)
    return (x - m) / torch.sqrt(((x - m) ** 2).mean(-1, keepdim=True) + EPS)


def _attend(q, k, v, spans):
    """q [B][L][H][Dh]; spans: (first query, last query, visible keys)."""
    o = torch.empty_like(q)
    for b in range(q.shape[0]):
        for h in range(q.shape[2]):
            for i, j, n in spans:
                p = torch.softmax(q[b, i:j, h] @ k[b, :n, h].T / math.sqrt(q.shape[3]), -1)
                o[b, i:j, h] = p @ v[b, :n, h]
    return o


def _spans(c):
    n = c["chunk"] if c["kind"] == "attn" else _chunk_rows(c)
    return [(i * n, (i + 1) * n, (c["cached"] + i + 1) * n) for i in range(c.get("chunks", 1))]


def _angles(c, Dh):
    f, hg, wg, A = _frames(c), c["Hl"] // 2, c["Wl"] // 2, c["A"]
    pos = []
    for chunk in range(c["cached"], c["cached"] + c.get("chunks", 1)):
        pos += [(f * chunk + i, r, s) for i in range(f) for r in range(hg) for s in range(wg)]
        pos += [(f * chunk + f + j, 0, 0) for j in range(A)]
    pos = torch.tensor(pos, dtype=torch.float64, device="cuda")
    side = 2 * (Dh // 6)
    parts = []
    for axis, n in enumerate((Dh - 2 * side, side, side)):
        w = 10000.0 ** (-2 * torch.arange(n // 2, dtype=torch.float64, device="cuda") / n)
        parts.append(pos[:, axis:axis + 1] * w)
    return torch.cat(parts, 1)


def _rotate(x, ang):
    """x [B][L][H][Dh], adjacent pairs turned by ang [L][Dh/2]."""
    cs, sn = torch.cos(ang)[None, :, None], torch.sin(ang)[None, :, None]
    a, b = x[..., 0::2], x[..., 1::2]
    return torch.stack((a * cs - b * sn, a * sn + b * cs), -1).flatten(-2)


def _e4m3(x):
    return x.clamp(-448, 448).to(torch.float8_e4m3fn).double()


def _as_fp8_rows(w):
    """A weight matrix as its E4M3 codes say: one scale per row."""
    top = w.float().abs().amax(1, keepdim=True)
    return _e4m3(w.float() * (448.0 / top)) * (top.double() / 448.0)


def _as_mx(x):
    """A tensor as its block-scaled codes say: a power of two per 32 elements."""
    x = x.double().unflatten(-1, (-1, 32))
    top = x.abs().amax(-1, keepdim=True)
    e = torch.ceil(torch.log2(top / 448.0))
    e = torch.where(top > 448.0 * 2.0 ** e, e + 1, torch.where(top <= 448.0 * 2.0 ** (e - 1), e - 1, e))
    return (_e4m3(x * 2.0 ** -e) * 2.0 ** e).flatten(-2)


def _as_scaled(x):
    """A tensor as its codes with the value cache's one scale say."""
    return _e4m3(x.float() * (1.0 / V_SCALE)) * V_SCALE


def _block64(c, w, x, e0, kc, vc, ctx, ctx_kv=None, kv_only=False):
    """One block in 64 bits: (x, appended k, appended v)."""
    H, Dh, _ = MODELS[c["d"]]
    L, cached, _ = _layout(c)
    B = x.shape[0]
    sh1, sc1, g1, sh2, sc2, g2 = (w["mod6"].double() + e0).unbind(1)
    h = _norm(x) * (1 + sc1[:, None]) + sh1[:, None]
    q, k, v = (_lin(h, w["w_qkv"], w["b_qkv"])).view(B, L, 3, H, Dh).unbind(2)
    ang = _angles(c, Dh)
    q, k = _rotate(q, ang), _rotate(k, ang)
    if kv_only:
        return None, k, v
    o = _attend(q, torch.cat((kc[:, :cached].double(), k), 1), torch.cat((vc[:, :cached].double(), v), 1), _spans(c))
    x = x + g1[:, None] * _lin(o.flatten(2), w["w_o"], w["b_o"])
    h = _norm(x) * w["lnc_gamma"].double() + w["lnc_beta"].double()
    cq = _lin(h, w["w_cq"], w["b_cq"]).view(B, L, H, Dh)
    kv = ctx_kv.double() if ctx_kv is not None else _lin(ctx, w["w_ckv"], w["b_ckv"])
    ck, cv = kv.view(B, -1, 2, H, Dh).unbind(2)
    o = _attend(cq, ck, cv, [(0, L, ck.shape[1])])
    x = x + _lin(o.flatten(2), w["w_co"], w["b_co"])
    h = _norm(x) * (1 + sc2[:, None]) + sh2[:, None]
    x = x + g2[:, None] * _lin(_gelu(_lin(h, w["w_f1"], w["b_f1"])), w["w_f2"], w["b_f2"])
    return x, k, v


def _time64(top, t):
    half = FREQ_DIM // 2
    w = 10000.0 ** (-torch.arange(half, dtype=torch.float64, device="cuda") / half)
    arg = 1000.0 * t.double()[:, None] * w
    e = _lin(_silu(_lin(torch.cat((torch.cos(arg), torch.sin(arg)), 1), top["w_t1"], top["b_t1"])), top["w_t2"], top["b_t2"])
    return e, _lin(_silu(e), top["w_t6"], top["b_t6"]).view(len(t), 6, -1)


def _text64(top, text):
    return _lin(_gelu(_lin(text.double(), top["w_x1"], top["b_x1"])), top["w_x2"], top["b_x2"])


def _embed64(top, z, a):
    B, C, F, Hl, Wl = z.shape
    tok = z.double().view(B, C, F, Hl // 2, 2, Wl // 2, 2).permute(0, 2, 3, 5, 1, 4, 6).reshape(B, -1, C * 4)
    x = _lin(tok, top["w_patch"], top["b_patch"])
    return torch.cat((x, _lin(a.double(), top["w_ain"], top["b_ain"])), 1) if a.shape[1] else x


def _head64(top, x, e, z):
    B, C, F, Hl, Wl = z.shape
    lv = F * (Hl // 2) * (Wl // 2)
    m = top["head_mod2"].double()
    h = _norm(x) * (1 + m[1] + e)[:, None] + (m[0] + e)[:, None]
    tok = _lin(h[:, :lv], top["w_hv"], top["b_hv"])
    vv = tok.view(B, F, Hl // 2, Wl // 2, C, 2, 2).permute(0, 4, 1, 2, 5, 3, 6).reshape(B, C, F, Hl, Wl)
    return vv, _lin(h[:, lv:], top["w_ha"], top["b_ha"])


def _step64(c, s, z, a, t, update=False):
    """(v_video, v_action, appended keys, appended values) of one call of the network."""
    top = s["top"]
    e, e0 = _time64(top, t)
    ctx = None if c.get("text_cached") else _text64(top, s["text"])
    x, ks, vs = _embed64(top, z, a), [], []
    for i, w in enumerate(s["blocks"]):
        last = update and i + 1 == len(s["blocks"])
        x, k, v = _block64(c, w, x, e0, s["kc"][i], s["vc"][i], ctx, s["ctx_kv"][i] if ctx is None else None, last)
        ks.append(k)
        vs.append(v)
    return (None, None) + (ks, vs) if update else _head64(top, x, e, z) + (ks, vs)


def _unipc(ts, t, others):
    """Weights of x, of the data prediction at ts and of those at `others` in UniPC's update from ts to t: the
    integral of e^lambda m over the step, with m through the given points in lambda."""
    if t >= 1.0:
        return 0.0, 1.0, []
    lam = lambda u: math.log(u / (1 - u))  # noqa: E731
    h = lam(t) - lam(ts)
    i0 = -math.expm1(-h)
    rhs, ik = [], i0
    for k in range(1, len(others) + 1):
        ik = h ** k / math.factorial(k) - ik
        rhs.append(math.factorial(k) * ik / (h ** k * i0))
    if not others:
        return (1 - t) / (1 - ts), t * i0, []
    r = torch.tensor([(lam(u) - lam(ts)) / h for u in others], dtype=torch.float64)
    R = torch.stack([r ** k for k in range(len(others))])
    w = (t * i0 * torch.linalg.solve(R, torch.tensor(rhs, dtype=torch.float64)) / r).tolist()
    return (1 - t) / (1 - ts), t * i0 - sum(w), w


def _denoise64(c, s):
    sched = [float(torch.tensor(t, dtype=torch.float32)) for t in _schedule(c)]
    n, x = c["steps"], s["x0"].double()
    nv = s["z"][0].numel()
    ms, prev, x_last = [], 0, None
    vv = va = None
    for i in range(n):
        xb = x.to(torch.float32).bfloat16()  # the network reads the state in bf16
        z = xb[:, :nv].view(1, *s["z"].shape[1:]).expand_as(s["z"])
        a = xb[:, nv:].view(1, *s["a"].shape[1:]).expand_as(s["a"])
        t = sched[i]
        vv, va, _, _ = _step64(c, s, z, a, torch.full((2,), t, device="cuda", dtype=torch.float64))
        both = torch.cat((vv.flatten(1), va.flatten(1)), 1)
        v = both[1:] + c["cfg_scale"] * (both[:1] - both[1:])
        m = x + (1 - t) * v
        if i:  # correct the state at t with the new prediction
            pts = [sched[i - 1 - k] for k in range(1, prev)] + [t]
            wx, w0, w = _unipc(sched[i - 1], t, pts)
            x = wx * x_last + w0 * ms[-1] + sum(w[k - 1] * ms[-1 - k] for k in range(1, prev)) + w[-1] * m
        p = 1 if sched[i + 1] >= 1.0 else min(c["order"], i + 1)
        wx, w0, w = _unipc(t, sched[i + 1], [sched[i - k] for k in range(1, p)])
        x_last = x
        x = wx * x + w0 * m + sum(w[k - 1] * ms[-k] for k in range(1, p))
        ms.append(m)
        prev = p
    return x, vv, va


def exact(case, seed):
    """What run() returns, in 64 bits; an FP8 layer's weights, keys and values are what their codes say."""
    c, kind = case, case["kind"]
    s = _inputs(c, seed)
    if kind == "attn":
        q, k, v = (_as_mx(s["q"]), _as_mx(s["k"]), _as_scaled(s["v"])) if c["fp8"] else (s[n].double() for n in "qkv")
        return _attend(q, k, v, _spans(c))
    if kind == "time":
        return _time64(s["top"], s["t"])
    if kind == "ends":
        x = _embed64(s["top"], s["z"], s["a"])
        return (x,) + _head64(s["top"], x, s["e"].double(), s["z"])
    if kind in ("qkv8", "ffn8"):
        m, x = (s["mod6"].double() + s["e0"].double())[:, :, None], s["x"].double()
        if kind == "qkv8":
            h = _norm(x) * (1 + m[:, 1]) + m[:, 0]
            return (_lin(h, _as_fp8_rows(s["w"]), s["b"]),) + (None,) * 5
        u = _gelu(_lin(_norm(x) * (1 + m[:, 4]) + m[:, 3], _as_fp8_rows(s["w1"]), s["b1"]))
        return x + m[:, 5] * _lin(u, _as_fp8_rows(s["w2"]), s["b2"])
    if kind == "block":
        return _block64(c, s["blocks"][0], s["x"].double(), s["e0"].double(), s["kc"][0], s["vc"][0], s["ctx"].double())
    if kind == "denoise":
        return _denoise64(c, s)
    vv, va, ks, vs = _step64(c, s, s["z"], s["a"], s["t"].double(), update=kind == "update")
    return ([] if kind == "update" else [vv, va]) + ks + vs

"""Workloads whose speed this library is judged by, each one call of a public entry point.

The listed cases follow what a sampling program has the library do.  A program either
runs a whole schedule (bc_sample), drives the blocks of a stack by itself
(bc_dit_block_forward), or calls single operations (bc_linear, bc_attention,
bc_bary_extrapolate).  Sizes are those of the four synthetic workloads (tiny, DiT-XL/2,
PixArt, the video model) and of other resolutions and batches of the same models.
"""
import math
import types

import torch

import paper_2608_28670_amd as bc
from paper_2608_28670_amd import loader

DEV = "cuda:0"
KINDS = {"dit": bc.BLOCK_DIT, "pixart": bc.BLOCK_PIXART, "dual": bc.BLOCK_DUAL, "single": bc.BLOCK_SINGLE}
THETA = 256.0   # rotary base of the video model


def listed():
    return [
        # The smallest whole call: a tiny fp32 model's schedule, all launches and latency.
        dict(name="sample_tiny_f32", op="sample", B=2, depth=2, D=128, heads=4, mlp=512, in_ch=4, out_ch=4, patch=1,
             side=8, classes=0, steps=10, K=3, interval=3, dtype="f32"),
        # A class-conditional batch through the whole schedule: conditioning, 14 full steps, 36 forecast steps.
        dict(name="sample_dit_xl2_b16", op="sample", B=16, depth=28, D=1152, heads=16, mlp=4608, in_ch=4, out_ch=8,
             patch=2, side=32, classes=1000, steps=50, K=3, interval=4, dtype="bf16"),
        # One image at a time: 256 rows, where a block is latency and its weights' bytes.
        dict(name="block_dit_b1", op="block", kind="dit", B=1, T=256, D=1152, heads=16, mlp=4608, dtype="bf16"),
        # The ordinary class-conditional batch.
        dict(name="block_dit_b16", op="block", kind="dit", B=16, T=256, D=1152, heads=16, mlp=4608, dtype="bf16"),
        # Text-to-image at 1024 x 1024: long self-attention and cross-attention to the caption.
        dict(name="block_pixart_b4", op="block", kind="pixart", B=4, T=4096, Tc=120, D=1152, heads=16, mlp=4608,
             dtype="bf16"),
        # The same at one 480 x 544 image (30 x 34 patches): ragged tiles, one sample.
        dict(name="block_pixart_1020", op="block", kind="pixart", B=1, T=1020, Tc=120, D=1152, heads=16, mlp=4608,
             dtype="bf16"),
        # The video model at its full size: joint attention over 14 310 + 256 tokens.
        dict(name="block_dual_video", op="block", kind="dual", B=1, grid_f=9, grid_h=30, grid_w=53, Tt=256, D=3072,
             heads=24, mlp=12288, dtype="bf16"),
        dict(name="block_single_video", op="block", kind="single", B=1, grid_f=9, grid_h=30, grid_w=53, Tt=256, D=3072,
             heads=24, mlp=12288, dtype="bf16"),
        # The video model on a single frame: 1590 + 256 tokens, too few rows to fill many rounds of large tiles.
        dict(name="block_single_frame", op="block", kind="single", B=1, grid_f=1, grid_h=30, grid_w=53, Tt=256, D=3072,
             heads=24, mlp=12288, dtype="bf16"),
        # Attention called alone, unscaled queries, ragged query and key counts.
        dict(name="attention_d64", op="attention", B=2, H=16, Tq=2050, Tk=2050, d=64, prescaled=False, dtype="bf16"),
        # A projection called alone, rows not a multiple of any tile.
        dict(name="linear_gelu", op="linear", M=5000, N=4608, K=1152, epi="gelu", dtype="bf16"),
        # The forecast over three cached features of [8, 16384, 3072]: memory alone.
        dict(name="forecast_k3", op="forecast", K=3, n=8 * 16384 * 3072, dtype="bf16", out="bf16"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["block", "block", "block", "block", "linear", "linear", "attention", "attention", "forecast",
                     "sample"])
    if op == "block":
        kind = rng.choice(["dit", "pixart", "dual", "single"])
        if kind in ("dual", "single"):
            D, heads = rng.choice([(3072, 24), (1024, 8), (1536, 24)])
            return dict(op=op, kind=kind, B=1 if D == 3072 else rng.randint(1, 2), grid_f=rng.randint(1, 9),
                        grid_h=rng.randint(8, 30), grid_w=rng.randint(8, 53), Tt=rng.randint(16, 256), D=D, heads=heads,
                        mlp=4 * D, dtype="bf16")
        f32 = rng.random() < 0.15
        D, heads = (384, 6) if f32 else rng.choice([(1152, 16), (1152, 16), (768, 12), (1024, 16)])
        T = _log(rng, 32, 4096 if kind == "pixart" else 1024)
        c = dict(op=op, kind=kind, B=max(1, min(16, 16384 // T, _log(rng, 1, 32))), T=T, D=D, heads=heads, mlp=4 * D,
                 dtype="f32" if f32 else "bf16")
        if kind == "pixart":
            c["Tc"] = rng.randint(16, 300)
        return c
    if op == "linear":
        f32 = rng.random() < 0.15
        epi = rng.choice(["bias", "gelu", "gated"])
        K = rng.choice([64 * rng.randint(2, 96), 8 * rng.randint(16, 300)])
        N = rng.choice([64 * rng.randint(1, 96), 8 * rng.randint(1, 600), rng.randint(16, 3000)])
        return dict(op=op, M=_log(rng, 16, 2048 if f32 else 16384), N=min(N, 1500) if f32 else N, K=K, epi=epi,
                    dtype="f32" if f32 else "bf16")
    if op == "attention":
        f32 = rng.random() < 0.1
        d = rng.choice([32, 64] if f32 else [64, 72, 128])
        Tq = _log(rng, 32, 1024 if f32 else 8192)
        return dict(op=op, B=rng.randint(1, 3), H=rng.randint(4, 24), Tq=Tq,
                    Tk=Tq if rng.random() < 0.6 else rng.randint(16, 600), d=d, prescaled=not f32 and rng.random() < 0.5,
                    dtype="f32" if f32 else "bf16")
    if op == "forecast":
        return dict(op=op, K=rng.randint(1, 5), n=_log(rng, 50_000, 200_000_000), dtype=rng.choice(["bf16", "bf16", "f32"]),
                    out=rng.choice(["bf16", "f32"]))
    D, heads = rng.choice([(1152, 16), (384, 6), (768, 12)])
    return dict(op=op, B=rng.randint(1, 12), depth=rng.randint(2, 8), D=D, heads=heads, mlp=4 * D, in_ch=4, out_ch=8,
                patch=2, side=rng.choice([16, 24, 32]), classes=1000, steps=rng.randint(10, 30), K=rng.randint(2, 4),
                interval=rng.randint(2, 6), dtype="bf16")


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _dt(name):
    return torch.bfloat16 if name == "bf16" else torch.float32


def _randn(g, shape, scale=1.0, dtype=torch.float32):
    return torch.empty(shape, device=DEV, dtype=torch.float32).normal_(0.0, scale, generator=g).to(dtype)


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _stream_shapes(kind, D, F):
    """Parameters of one stream of a block, by the binding's names."""
    if kind == "single":
        return {"w_mod": (3 * D, D), "b_mod": (3 * D,), "w_qkv": (3 * D + F, D), "b_qkv": (3 * D + F,),
                "w_o": (D, D + F), "b_o": (D,)}
    s = {"w_mod": (6, D)} if kind == "pixart" else {"w_mod": (6 * D, D), "b_mod": (6 * D,)}
    s.update({"w_qkv": (3 * D, D), "b_qkv": (3 * D,), "w_o": (D, D), "b_o": (D,), "w_fc1": (F, D), "b_fc1": (F,),
              "w_fc2": (D, F), "b_fc2": (D,)})
    return s


def _cross_shapes(D):
    return {"wx_q": (D, D), "bx_q": (D,), "wx_kv": (2 * D, D), "bx_kv": (2 * D,), "wx_o": (D, D), "bx_o": (D,)}


def _tokens(case):
    return case["T"] if "T" in case else case["grid_f"] * case["grid_h"] * case["grid_w"]


def _block_inputs(case, seed):
    g, D, F, dt = _gen(seed), case["D"], case["mlp"], _dt(case["dtype"])
    kind, B, T, Tt = case["kind"], case["B"], _tokens(case), case.get("Tt", 0)
    hd = D // case["heads"]
    p = {"img": {n: _randn(g, s, 0.02, dt) for n, s in _stream_shapes(kind, D, F).items()}}
    if kind == "dual":
        p["txt"] = {n: _randn(g, s, 0.02, dt) for n, s in _stream_shapes(kind, D, F).items()}
    if kind == "pixart":
        p["cross"] = {n: _randn(g, s, 0.02, dt) for n, s in _cross_shapes(D).items()}
    if kind in ("dual", "single"):
        for s in p.values():
            s["q_norm"] = (1.0 + _randn(g, (hd,), 0.02)).to(dt)
            s["k_norm"] = (1.0 + _randn(g, (hd,), 0.02)).to(dt)
    p["x"] = _randn(g, (B, T + (Tt if kind == "single" else 0), D))
    p["x_txt"] = _randn(g, (B, Tt, D)) if kind == "dual" else None
    p["c"] = _randn(g, (B, 6 * D if kind == "pixart" else D), 0.3 if kind == "pixart" else 1.0)
    p["ctx"] = _randn(g, (B, case["Tc"], D), 1.0, dt) if kind == "pixart" else None
    return p


def _sample_cfg(case):
    D, side = case["D"], case["side"]
    return types.SimpleNamespace(
        kind="dit", depth=case["depth"], depth_single=0, hidden=D, heads=case["heads"], head_dim=D // case["heads"],
        mlp=case["mlp"], in_ch=case["in_ch"], out_ch=case["out_ch"], p=case["patch"], latent=(case["in_ch"], side, side),
        n_classes=case["classes"], ctx_tokens=0, ctx_dim=0, txt_tokens=0, freq_dim=256, dtype=case["dtype"],
        sampler="ddim", K=case["K"], tokens=(side // case["patch"]) ** 2)


def _sample_shapes(case):
    D, F, p2 = case["D"], case["mlp"], case["patch"] ** 2
    s = {"t_w1": (D, 256), "t_b1": (D,), "t_w2": (D, D), "t_b2": (D,), "patch_w": (D, case["in_ch"] * p2), "patch_b": (D,),
         "pos": ((case["side"] // case["patch"]) ** 2, D), "final_w_mod": (2 * D, D), "final_b_mod": (2 * D,),
         "final_w": (case["out_ch"] * p2, D), "final_b": (case["out_ch"] * p2,)}
    if case["classes"]:
        s["y_table"] = (case["classes"] + 1, D)
    for l in range(case["depth"]):
        for n, shape in _stream_shapes("dit", D, F).items():
            s["blocks.%d.%s" % (l, n)] = shape
    return s


def _sample_inputs(case, seed):
    g, dt = _gen(seed), _dt(case["dtype"])
    p = {n: _randn(g, s, 0.02, dt) for n, s in _sample_shapes(case).items()}
    x = _randn(g, (case["B"], case["in_ch"], case["side"], case["side"]))
    lab = torch.randint(0, case["classes"], (case["B"],), device=DEV, generator=g) if case["classes"] else None
    return p, x, lab


def _op_inputs(case, seed):
    g, dt = _gen(seed), _dt(case["dtype"])
    if case["op"] == "linear":
        M, N, K = case["M"], case["N"], case["K"]
        s = dict(A=_randn(g, (M, K), 1.0, dt), W=_randn(g, (N, K), 0.02, dt), bias=_randn(g, (N,), 0.02, dt))
        if case["epi"] == "gated":
            s["rows"] = max(1, M // 4)
            s["res"] = _randn(g, (M, N))
            s["gate"] = _randn(g, (-(-M // s["rows"]), N), 0.3)
        return s
    if case["op"] == "attention":
        B, H, d = case["B"], case["H"], case["d"]
        q = _randn(g, (B, case["Tq"], H, d))
        if case["prescaled"]:
            q = q * (math.log2(math.e) / math.sqrt(d))
        return dict(q=q.to(dt), k=_randn(g, (B, case["Tk"], H, d), 1.0, dt), v=_randn(g, (B, case["Tk"], H, d), 1.0, dt))
    K, n = case["K"], case["n"]
    feats = torch.empty((K, n), device=DEV, dtype=dt)
    for j in range(K):
        feats[j].normal_(0.0, 1.0, generator=g)
    return dict(feats=feats)


def prepare(case, seed):
    op = case["op"]
    if op == "sample":
        p, x, lab = _sample_inputs(case, seed)
        cfg = _sample_cfg(case)
        m = loader.DeviceModel(cfg, {}, device=DEV, dev_params=p)
        mask = bc.make_mask(case["steps"], case["interval"])
        m.buffers(case["B"], case["K"], case["steps"])
        m.ring(case["B"], case["K"]).storage.zero_()
        return dict(op=op, model=m, xT=x, x=torch.empty_like(x), labels=lab, mask=mask)
    if op == "block":
        p = _block_inputs(case, seed)
        D, rope = case["D"], None
        if case["kind"] in ("dual", "single"):
            rope = (case["grid_f"], case["grid_h"], case["grid_w"], THETA)
        desc = bc.block_desc(KINDS[case["kind"]], case["B"], _tokens(case), D, case["heads"], D // case["heads"],
                             case["mlp"], bc.BF16 if case["dtype"] == "bf16" else bc.F32, T_txt=case.get("Tt", 0),
                             T_ctx=case.get("Tc", 0), rope=rope)
        w = bc.block_weights(p["img"], p.get("txt"), p.get("cross"))
        ws = torch.empty(bc.block_workspace_size(desc), dtype=torch.uint8, device=DEV)
        return dict(op=op, p=p, desc=desc, w=w, ws=ws)
    s = _op_inputs(case, seed)
    s["op"] = op
    if op == "linear":
        s["epi"] = {"bias": bc.EPI_BIAS, "gelu": bc.EPI_BIAS_GELU, "gated": bc.EPI_GATE_RES}[case["epi"]]
        s["out"] = torch.empty((case["M"], case["N"]), device=DEV, dtype=torch.float32 if case["epi"] == "gated" else _dt(case["dtype"]))
    elif op == "attention":
        s["prescaled"] = case["prescaled"]
        s["out"] = torch.empty_like(s["q"])
    else:
        K = case["K"]
        s["ring"] = bc.CacheRing(K, s["feats"])
        for j in range(K):
            s["ring"].push(None, float(4 * j))
        s["wts"] = bc.bary_weights([4.0 * j for j in reversed(range(K))], 4.0 * K - 2.0)
        s["out"] = torch.empty(case["n"], device=DEV, dtype=_dt(case["out"]))
    return s


def run(s):
    op = s["op"]
    if op == "sample":
        s["x"].copy_(s["xT"])
        ring = s["model"].sample(s["x"], s["mask"], labels=s["labels"])
        return {"latents": s["x"], "ring": ring.storage}
    if op == "block":
        p = s["p"]
        bc.dit_block_forward(s["desc"], s["w"], p["x"], p["c"], s["ws"], x_txt=p["x_txt"], ctx=p["ctx"])
        return {"x": p["x"]} if p["x_txt"] is None else {"x": p["x"], "x_txt": p["x_txt"]}
    if op == "linear":
        bc.linear(s["A"], s["W"], s["bias"], s["out"], s["epi"], s.get("res"), s.get("gate"), s.get("rows", 1))
    elif op == "attention":
        bc.attention(s["q"], s["k"], s["v"], s["out"], prescaled=s["prescaled"])
    else:
        bc.bary_extrapolate(s["ring"], s["wts"], s["out"])
    return s["out"]


# ---------------------------------------------------------------------------
# What a pass cannot do without, and how exactly it can be done
# ---------------------------------------------------------------------------
def _block_work(case, e, B, T):
    """(flops, weight elements) of one block without its modulation."""
    D, F, kind = case["D"], case["mlp"], case.get("kind", "dit")
    if kind == "single":
        L = T + case["Tt"]
        return 2.0 * B * L * D * (4 * D + 2 * F) + 4.0 * B * L * L * D, D * (4 * D + 2 * F)
    Tt = case.get("Tt", 0)
    fl = 2.0 * B * (T + Tt) * D * (4 * D + 2 * F) + 4.0 * B * (T + Tt) ** 2 * D
    wt = D * (4 * D + 2 * F) * (2 if kind == "dual" else 1)
    if kind == "pixart":
        Tc = case["Tc"]
        fl += 2.0 * B * T * D * 2 * D + 4.0 * B * T * Tc * D + 2.0 * B * Tc * D * 2 * D
        wt += 4 * D * D
    return fl, wt


def work(case):
    op, e = case["op"], 2 if case["dtype"] == "bf16" else 4
    if op == "sample":
        S = case["steps"]
        full = len({k for k in range(S) if k % case["interval"] == 0} | {S - 1})
        T, D, B = (case["side"] // case["patch"]) ** 2, case["D"], case["B"]
        fl, _ = _block_work(case, e, B, T)
        fl = full * case["depth"] * (fl + 2.0 * B * 6 * D * D)
        fl += 2.0 * S * B * T * D * case["out_ch"] * case["patch"] ** 2
        wt = sum(math.prod(s) for s in _sample_shapes(case).values())
        lat = B * case["in_ch"] * case["side"] ** 2 * 4
        return {"bytes": float(wt * e + 2 * lat + min(full, case["K"]) * B * T * D * e), "flops": fl}
    if op == "block":
        B, T, D, Tt = case["B"], _tokens(case), case["D"], case.get("Tt", 0)
        fl, wt = _block_work(case, e, B, T)
        if case["kind"] != "pixart":
            nm = 3 if case["kind"] == "single" else 12 if case["kind"] == "dual" else 6
            fl += 2.0 * B * nm * D * D
            wt += nm * D * D
        by = wt * e + 2 * B * (T + Tt) * D * 4 + B * case.get("Tc", 0) * D * e
        return {"bytes": float(by), "flops": fl}
    if op == "linear":
        M, N, K = case["M"], case["N"], case["K"]
        by = (M * K + N * K) * e + M * N * (8 if case["epi"] == "gated" else e)
        return {"bytes": float(by), "flops": 2.0 * M * N * K}
    if op == "attention":
        B, H, Tq, Tk, d = (case[n] for n in ("B", "H", "Tq", "Tk", "d"))
        return {"bytes": float(B * H * d * 2 * (Tq + Tk) * e), "flops": 4.0 * B * H * Tq * Tk * d}
    K, n = case["K"], case["n"]
    return {"bytes": float(n * (K * e + (2 if case["out"] == "bf16" else 4))), "flops": 2.0 * K * n}


def tolerance(case):
    """About four times the error that the path shows against 64 bits.  One bf16 rounding of an
    output is 1.7e-3 (2-norm); attention rounds its probabilities too (2.3e-3).  A block returns
    the fp32 stream, whose bf16-computed update is small beside it for the DiT and PixArt blocks
    (5e-4 to 1e-3) and not for the video model's wider ones (2.8e-3).  A whole bf16 run shows
    1.2e-3 (latents) and 2.0e-3 (cached features), fp32 ones 1e-7."""
    op, f32 = case["op"], case["dtype"] == "f32"
    if op == "sample":
        return {"rel": 1e-5, "max": 1e-3} if f32 else {"rel": 1e-2, "max": 0.3}
    if op == "block":
        if f32:
            return {"rel": 1e-5, "max": 1e-3}
        return {"rel": 1.1e-2, "max": 0.2} if case["kind"] in ("dual", "single") else {"rel": 4e-3, "max": 0.1}
    if op == "linear":
        return {"rel": 1e-5, "max": 1e-4} if f32 or case["epi"] == "gated" else {"rel": 7e-3, "max": 0.02}
    if op == "attention":
        return {"rel": 1e-5, "max": 1e-3} if f32 else {"rel": 1e-2, "max": 0.1}
    return {"rel": 1e-6, "max": 1e-4} if case["out"] == "f32" else {"rel": 7e-3, "max": 0.02}


# ---------------------------------------------------------------------------
# The same in 64 bits, plain torch
# ---------------------------------------------------------------------------
def _gelu(x):
    return torch.nn.functional.gelu(x, approximate="tanh")


def _lin(x, w, b):
    return torch.addmm(b.double(), x.reshape(-1, x.shape[-1]), w.double().t().contiguous()).reshape(*x.shape[:-1], w.shape[0])


def _ln(x, shift, scale):
    h = torch.nn.functional.layer_norm(x, x.shape[-1:], eps=1e-6)
    return h * (1.0 + scale[:, None, :]) + shift[:, None, :]


def _attend(q, k, v, scale):
    """softmax(scale q k^T) v over [B, T, H, d], a bounded number of scores at a time."""
    B, Tq, H, d = q.shape
    Tk = k.shape[1]
    qs, ks, vs = (t.permute(0, 2, 1, 3).reshape(B * H, t.shape[1], d).contiguous() for t in (q, k, v))
    out = torch.empty_like(qs)
    step = max(1, (1 << 28) // (Tq * Tk))
    for i in range(0, B * H, step):
        s = torch.bmm(qs[i:i + step], ks[i:i + step].transpose(1, 2).contiguous()) * scale
        out[i:i + step] = torch.bmm(torch.softmax(s, dim=-1), vs[i:i + step])
        del s
    return out.reshape(B, H, Tq, d).permute(0, 2, 1, 3)


def _heads(x, H):
    return x.reshape(x.shape[0], x.shape[1], H, x.shape[2] // H)


def _rms(x, w):
    return x / torch.sqrt(x.square().mean(-1, keepdim=True) + 1e-6) * w.double()


def _rope(x, grid):
    """Rotates the first f*h*w tokens of x [B, T, H, d]: d/8 dims by frame, the rest by row and column."""
    f, h, w = grid
    d, n = x.shape[-1], f * h * w
    pos = torch.cartesian_prod(*(torch.arange(m, device=DEV, dtype=torch.float64) for m in (f, h, w)))
    ang = []
    for a, da in enumerate((d // 8, (d - d // 8) // 2, d - d // 8 - (d - d // 8) // 2)):
        ang.append(pos[:, a:a + 1] * THETA ** (-torch.arange(0, da, 2, device=DEV, dtype=torch.float64) / da))
    ang = torch.cat(ang, 1)[None, :, None, :]
    c, s, x0, x1 = ang.cos(), ang.sin(), x[:, :n, :, 0::2], x[:, :n, :, 1::2]
    y = x.clone()
    y[:, :n, :, 0::2] = x0 * c - x1 * s
    y[:, :n, :, 1::2] = x0 * s + x1 * c
    return y


def _exact_dit(p, cross, x, mod, heads, ctx):
    D = x.shape[-1]
    m = [mod[:, i * D:(i + 1) * D] for i in range(6)]
    qkv = _lin(_ln(x, m[0], m[1]), p["w_qkv"], p["b_qkv"])
    q, k, v = (_heads(qkv[..., i * D:(i + 1) * D], heads) for i in range(3))
    scale = 1.0 / math.sqrt(D // heads)
    x = x + m[2][:, None, :] * _lin(_attend(q, k, v, scale).reshape(x.shape), p["w_o"], p["b_o"])
    if cross:
        q = _heads(_lin(x, cross["wx_q"], cross["bx_q"]), heads)
        kv = _lin(ctx, cross["wx_kv"], cross["bx_kv"])
        a = _attend(q, _heads(kv[..., :D], heads), _heads(kv[..., D:], heads), scale)
        x = x + _lin(a.reshape(x.shape), cross["wx_o"], cross["bx_o"])
    h = _gelu(_lin(_ln(x, m[3], m[4]), p["w_fc1"], p["b_fc1"]))
    return x + m[5][:, None, :] * _lin(h, p["w_fc2"], p["b_fc2"])


def _exact_block(case, seed):
    p, D, H, kind = _block_inputs(case, seed), case["D"], case["heads"], case["kind"]
    x, c, scale = p["x"].double(), p["c"].double(), 1.0 / math.sqrt(case["D"] // case["heads"])
    silu = torch.nn.functional.silu
    if kind == "pixart":
        return {"x": _exact_dit(p["img"], p["cross"], x, c + p["img"]["w_mod"].double().reshape(1, -1), H, p["ctx"].double())}
    if kind == "dit":
        return {"x": _exact_dit(p["img"], None, x, _lin(silu(c), p["img"]["w_mod"], p["img"]["b_mod"]), H, None)}
    grid = (case["grid_f"], case["grid_h"], case["grid_w"])

    def qkv_of(y, w, rope):
        q, k, v = (_heads(y[..., i * D:(i + 1) * D], H) for i in range(3))
        q, k = _rms(q, w["q_norm"]), _rms(k, w["k_norm"])
        return (_rope(q, grid), _rope(k, grid), v) if rope else (q, k, v)

    if kind == "single":
        w = p["img"]
        m = _lin(silu(c), w["w_mod"], w["b_mod"])
        y = _lin(_ln(x, m[:, :D], m[:, D:2 * D]), w["w_qkv"], w["b_qkv"])
        a = _attend(*qkv_of(y, w, True), scale).reshape(x.shape)
        z = torch.cat([a, _gelu(y[..., 3 * D:])], -1)
        return {"x": x + m[:, None, 2 * D:] * _lin(z, w["w_o"], w["b_o"])}
    xs, ws = (x, p["x_txt"].double()), (p["img"], p["txt"])
    ms = [_lin(silu(c), w["w_mod"], w["b_mod"]).reshape(-1, 6, D) for w in ws]
    t = [qkv_of(_lin(_ln(xx, m[:, 0], m[:, 1]), w["w_qkv"], w["b_qkv"]), w, i == 0)
         for i, (xx, m, w) in enumerate(zip(xs, ms, ws))]
    a = _attend(*(torch.cat([t[0][i], t[1][i]], 1) for i in range(3)), scale)
    a, out = a.reshape(a.shape[0], a.shape[1], D), []
    for xx, m, w, at in zip(xs, ms, ws, (a[:, :x.shape[1]], a[:, x.shape[1]:])):
        xx = xx + m[:, None, 2] * _lin(at, w["w_o"], w["b_o"])
        h = _gelu(_lin(_ln(xx, m[:, 3], m[:, 4]), w["w_fc1"], w["b_fc1"]))
        out.append(xx + m[:, None, 5] * _lin(h, w["w_fc2"], w["b_fc2"]))
    return {"x": out[0], "x_txt": out[1]}


def _weights(nodes, t):
    """The barycentric weights of the nodes (newest first) at t, at the default parameters."""
    K = len(nodes)
    u = [(0.5 if j in (0, K - 1) else 1.0) * (-1.0) ** (j + 1) / (t - s) for j, s in enumerate(nodes)]
    u = [max(-10.0, min(10.0, v)) for v in u]
    v = [math.copysign((abs(z) + 1e-12) ** {1: 1.0, 2: 1.0, 3: 0.95}.get(K, 0.7), z) for z in u]
    return [z / sum(v) for z in v]


def _exact_sample(case, seed):
    p, x, lab = _sample_inputs(case, seed)
    x, S, D, B, ps = x.double(), case["steps"], case["D"], case["B"], case["patch"]
    C, side, silu = case["in_ch"], case["side"], torch.nn.functional.silu
    n = side // ps
    betas = 1e-4 + (0.02 - 1e-4) * torch.arange(1000, dtype=torch.float64) / 999
    ab = torch.cumprod(1.0 - betas, 0).tolist()
    tau = [999 - 1000 * k // S for k in range(S)]
    ring, head, nodes = torch.zeros((case["K"], B * n * n * D), dtype=torch.float64, device=DEV), -1, []
    for k in range(S):
        f = torch.exp(-math.log(10000.0) * torch.arange(128, device=DEV, dtype=torch.float64) / 128) * tau[k]
        t = _lin(silu(_lin(torch.cat([f.cos(), f.sin()])[None], p["t_w1"], p["t_b1"])), p["t_w2"], p["t_b2"])
        c = silu(t.expand(B, D) + (p["y_table"][lab].double() if lab is not None else 0.0))
        if k % case["interval"] == 0 or k == S - 1:
            tok = x.reshape(B, C, n, ps, n, ps).permute(0, 2, 4, 3, 5, 1).reshape(B, n * n, ps * ps * C)
            feat = _lin(tok, p["patch_w"], p["patch_b"]) + p["pos"].double()
            for l in range(case["depth"]):
                w = {m: p["blocks.%d.%s" % (l, m)] for m in _stream_shapes("dit", D, case["mlp"])}
                feat = _exact_dit(w, None, feat, _lin(c, w["w_mod"], w["b_mod"]), case["heads"], None)
            head = (head + 1) % case["K"]
            ring[head] = feat.reshape(-1)
            nodes = [k] + nodes[:case["K"] - 1]
        else:
            wts = _weights([float(s) for s in nodes], float(k))
            feat = sum(w * ring[(head - j) % case["K"]] for j, w in enumerate(wts)).reshape(B, n * n, D)
        m = _lin(c, p["final_w_mod"], p["final_b_mod"])
        out = _lin(_ln(feat, m[:, :D], m[:, D:]), p["final_w"], p["final_b"])
        out = out.reshape(B, n, n, ps, ps, case["out_ch"]).permute(0, 5, 1, 3, 2, 4).reshape(B, case["out_ch"], side, side)
        a, a2, eps = ab[tau[k]], ab[tau[k + 1]] if k + 1 < S else 1.0, out[:, :C]
        x = math.sqrt(a2) * (x - math.sqrt(1.0 - a) * eps) / math.sqrt(a) + math.sqrt(1.0 - a2) * eps
    return {"latents": x, "ring": ring}


def exact(case, seed):
    op = case["op"]
    if op == "sample":
        return _exact_sample(case, seed)
    if op == "block":
        return _exact_block(case, seed)
    s = _op_inputs(case, seed)
    if op == "linear":
        y = _lin(s["A"].double(), s["W"], s["bias"])
        if case["epi"] == "gelu":
            y = _gelu(y)
        if case["epi"] == "gated":
            row = torch.arange(case["M"], device=DEV) // s["rows"]
            y = s["res"].double() + s["gate"].double()[row] * y
        return y
    if op == "attention":
        scale = math.log(2.0) if case["prescaled"] else 1.0 / math.sqrt(case["d"])
        return _attend(s["q"].double(), s["k"].double(), s["v"].double(), scale)
    K = case["K"]
    wts = _weights([4.0 * j for j in reversed(range(K))], 4.0 * K - 2.0)
    acc = torch.zeros(case["n"], device=DEV, dtype=torch.float64)
    for j, w in enumerate(wts):
        acc += w * s["feats"][K - 1 - j].double()
    return acc

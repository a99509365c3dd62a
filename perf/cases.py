"""The work that users have this decoder do, as cases that can be timed and checked.

A case is one decode call of a named stream or clip (``KvCache.decode_chunk``, or
``decode_chunks`` for several streams at once): a model shape, its operand
precision, a token grid, the latent frames of the call, the attention window and
the pixel format. Streams are measured steady: the frames that fill the window are
decoded beforehand, so a pass is the next chunk of a running stream. Clips start
from a reset, which is part of the pass.

One decoder (weights) serves every stream of a case, as in a program that decodes
one video after another with one model; the seed gives the latents. Most cases
hold a few blocks of each stack (one or two backbone blocks, one refinement block,
and with them the embedding, the temporal upsampling and the pixel head); some are
whole decoders. Pixels are returned as fp32 or bf16: in uint8 a rounding anywhere in the
network moves whole codes, which says nothing about the kernels.
"""
from __future__ import annotations

import math

import torch

from paper_2607_14898_amd import flashdecoder as fdb
from paper_2607_14898_amd.flops import call_flops
from paper_2607_14898_amd.workloads import ModelConfig, param_specs

_DEV = "cuda"


# ------------------------------------------------------------------ the cases

# (D, query heads, KV groups) of the decoder sizes: the narrow soak decoder, then S, B, L, XL
_WIDTHS = {"narrow": (256, 4, 2), "s": (512, 8, 2), "b": (768, 12, 3), "l": (1024, 16, 4), "xl": (1536, 24, 3)}


def _case(name, width, gh, gw, **kw):
    d, n, g = _WIDTHS[width] if isinstance(width, str) else width
    c = {"name": name, "dtype": "f16", "mlp": "f16", "dim": d, "heads": n, "groups": g, "grid_h": gh, "grid_w": gw,
         "patch": 2, "channels": 16, "bb": 2, "rf": 1, "frames": 1, "window": 2, "batch": 1, "streams": 1,
         "plain": False, "clip": False, "s_out": 16, "pixels": "f32"}
    c.update(kw)
    return c


def listed():
    return [
        # a two-frame clip of the tiny decoder in fp32: what unit checks and first trials of the library run
        _case("tiny-f32-clip", (128, 4, 2), 8, 8, dtype="f32", patch=1, rf=2, frames=2, clip=True, s_out=8),
        # the same as the workload list words it: LayerNorm, GELU, plain multi-head attention, one linear head
        _case("tiny-plain-f32-clip", (128, 4, 4), 8, 8, dtype="f32", patch=1, rf=0, frames=2, window=1, plain=True,
              clip=True, s_out=8),
        # the fp32 path at full width on a small picture: a checkpoint is validated with it before 16-bit serving
        _case("xl-f32-small-stream", "xl", 10, 13, dtype="f32"),
        # a thumbnail stream through the whole XL decoder (20 + 2 blocks): the latency of one small call
        _case("xl-thumb-stream", "xl", 6, 10, bb=20, rf=2),
        # several small ragged streams in one batch, two frames a call, wider window (narrow decoder)
        _case("narrow-batch4", "narrow", 10, 13, frames=2, window=3, batch=4),
        # the S decoder on Wan2.2 latents (48 channels, no PixelUnshuffle) at 480p, whole depth
        _case("s-480p-stream", "s", 30, 52, bb=12, rf=2, patch=1, channels=48),
        # the 480p stream of the XL decoder, one latent frame a call
        _case("xl-480p-stream", "xl", 30, 52),
        # a 4-frame clip at 480p in one call, bf16 operands and pixels
        _case("xl-480p-clip4-bf16", "xl", 30, 52, dtype="bf16", bb=1, frames=4, clip=True, pixels="bf16"),
        # two 480p streams served at once with the per-token FP8 MLP, one backbone block (see _FP8_BLOCKS)
        _case("xl-480p-fp8-2streams", "xl", 30, 52, mlp="fp8", bb=1, rf=0, streams=2),
        # the 720p stream with the static-calibrated FP8 MLP, one refinement block
        _case("xl-720p-fp8s-stream", "xl", 45, 80, mlp="fp8s", bb=0, rf=1),
        # the headline: one chunk of the 720p stream through the whole XL decoder
        _case("xl-720p-stream", "xl", 45, 80, bb=20, rf=2),
        # the 1080p stream (padded to a 68 x 120 token grid)
        _case("xl-1080p-stream", "xl", 68, 120, bb=1),
    ]


# FP8 decoders are measured by single blocks: an E4M3 code moves a whole step (2^-4 of its value) when its
# input's rounding moves, and with every further quantised block such moves travel on and grow
_FP8_BLOCKS = [(1, 0), (0, 1)]
_LARGEST = 17.7e12  # operations of the largest listed case's pass


def draw(rng):
    while True:
        logu = lambda a, b: math.exp(rng.uniform(math.log(a), math.log(b)))  # noqa: E731
        f32 = rng.random() < 0.25
        if f32:
            plain = rng.random() < 0.4
            width = rng.choice([(128, 4, 2), (128, 4, 4), (256, 4, 2), (256, 8, 4), (512, 8, 2), (1536, 24, 3)])
            tokens = logu(24, 600)
        else:
            plain = rng.random() < 0.08
            width = _WIDTHS[rng.choice(["narrow", "s", "b", "l", "xl", "xl", "xl"])]
            tokens = logu(24, 8160)
        asp = rng.uniform(1.0, 2.0)
        gh = max(3, round(math.sqrt(tokens / asp)))
        gw = max(3, round(gh * asp))
        clip = rng.random() < 0.3
        patch = rng.choice([1, 2])
        kw = dict(dtype="f32" if f32 else rng.choice(["f16", "f16", "f16", "bf16"]), patch=patch,
                  channels=16 if patch == 2 else rng.choice([16, 48]), bb=rng.choice([1, 2]), rf=0 if plain else 1,
                  frames=rng.choice([1, 1, 1, 2, 3, 4]) if not plain else 2 * rng.choice([1, 2]),
                  window=rng.choice([1, 2, 2, 2, 3, 4]) if not plain else rng.choice([1, 2]), plain=plain, clip=clip,
                  s_out=8 if f32 else 16, pixels="f32" if f32 else rng.choice(["f32", "f32", "bf16"]))
        if not f32 and not plain and kw["dtype"] == "f16" and rng.random() < 0.3:
            bb, rf = rng.choice(_FP8_BLOCKS)
            kw.update(mlp=rng.choice(["fp8", "fp8s"]), bb=bb, rf=rf)
        if tokens < 800 and rng.random() < 0.3:
            kw["batch"] = rng.choice([2, 3, 4])
        elif not f32 and rng.random() < 0.2:
            kw["streams"] = rng.choice([2, 3])
        c = _case("", width, gh, gw, **kw)
        del c["name"]
        if work(c)["flops"] <= (0.025 if f32 else 1.0) * _LARGEST:
            return c


# ------------------------------------------------------------------ model, weights, inputs

def _model(c):
    plain = c["plain"]
    return ModelConfig(
        compute_dtype=c["dtype"], latent_channels=c["channels"], latent_h=c["grid_h"] * c["patch"],
        latent_w=c["grid_w"] * c["patch"], patch=c["patch"], dim=c["dim"], n_heads=c["heads"], n_kv_groups=c["groups"],
        n_backbone_blocks=c["bb"], n_refine_blocks=c["rf"], mlp_hidden=4 * c["dim"],
        head_hidden=0 if plain else 4 * c["dim"], mlp_kind="gelu" if plain else "swiglu",
        norm_kind="ln" if plain else "rms", head_kind="linear" if plain else "temporal_first", kv_norm=not plain,
        rope=not plain, norm_eps=1e-5 if plain else 1e-6, s_out=c["s_out"], window=c["window"],
        unit_frames=2 if plain else 1, mlp_precision=c["mlp"])


def _history(c):
    """Calls decoded before the measured one: those that fill the window."""
    if c["clip"]:
        return 0
    unit = 2 if c["plain"] else 1
    return -(-(c["window"] - 1) * unit // c["frames"])


def _round(x, c):
    return x if c["dtype"] == "f32" else x.bfloat16().float()


def _weights(m, c):
    """The model's weights, on the GPU in fp32 (rounded to bf16 for 16-bit compute)."""
    g = torch.Generator(_DEV).manual_seed(0)
    w = {}
    for name, shape, kind in param_specs(m):
        a = torch.randn(shape, generator=g, device=_DEV) * 0.02
        w[name] = _round(a + 1.0 if kind == "g" else a, c)
    return w


def _latents(m, c, seed):
    """[streams] latents [batch, C', history and measured frames, H', W']."""
    g = torch.Generator(_DEV).manual_seed(1000 + seed)
    t = (_history(c) + 1) * c["frames"]
    z = [torch.randn((c["batch"], m.latent_channels, t, m.latent_h, m.latent_w), generator=g, device=_DEV)
         for _ in range(c["streams"])]
    return [_round(x, c) for x in z]


_AMAX = (6.0, 10.0)  # static FP8 amplitudes of every block (MLP input, SwiGLU output)
_kept = {}           # the decoder in use: one, of the case at hand


def _decoder(m, c):
    key = repr(sorted((k, v) for k, v in c.items() if k != "name"))
    if key not in _kept:
        _kept.clear()
        w = {k: v.cpu().numpy() for k, v in _weights(m, c).items()}
        dec = fdb.Decoder(m, w, max_batch=c["batch"], max_frames_per_call=c["frames"])
        if c["mlp"] == "fp8s":
            fdb.fd_set_fp8_act_amax(dec.handle, list(_AMAX) * (c["bb"] + c["rf"]))
        _kept[key] = dec
    return _kept[key]


_PIXELS = {"f32": fdb.FD_PIXELS_F32, "bf16": fdb.FD_PIXELS_BF16}


def prepare(case, seed):
    m = _model(case)
    dec = _decoder(m, case)
    fmt = _PIXELS[case["pixels"]]
    caches = [fdb.KvCache(dec, case["batch"]) for _ in range(case["streams"])]
    F, zs = case["frames"], _latents(m, case, seed)
    for cache, z in zip(caches, zs):
        for k in range(_history(case)):
            cache.decode_chunk(z[:, :, k * F:(k + 1) * F].contiguous())
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    last = [z[:, :, -F:].to(dt).contiguous() for z in zs]
    outs = [torch.empty(dec.output_shape(case["batch"], F), dtype=fdb.pixel_torch_dtype(fmt), device=_DEV)
            for _ in caches]
    return {"caches": caches, "latents": last, "outs": outs, "fmt": fmt, "clip": case["clip"]}


def run(state):
    caches, z, outs, fmt = state["caches"], state["latents"], state["outs"], state["fmt"]
    if state["clip"]:
        for cache in caches:
            cache.reset()
    if len(caches) > 1:
        return fdb.decode_chunks(caches, z, outs, out_format=fmt)
    return [caches[0].decode_chunk(z[0], outs[0], out_format=fmt)]


def work(case):
    m = _model(case)
    F, B, n = case["frames"], case["batch"], case["streams"]
    L, uf, es = m.tokens_per_frame, m.unit_frames, 4 if case["dtype"] == "f32" else 2
    t0 = _history(case) * F
    gemm, attn = call_flops(m, F, t0, B)
    params = 0.0
    for name, shape, _ in param_specs(m):
        size = math.prod(shape)
        mlp8 = case["mlp"] != "f16" and name.endswith((".w13", ".w2"))
        params += size * (4 if len(shape) == 1 else 1 if mlp8 else es)
    # rings: the window's earlier keys and values read, the call's own written
    kv = 2.0 * B * m.n_kv_groups * m.head_dim * es
    old = min(t0, (m.window - 1) * uf)
    ring = kv * L * (old + F) * (m.n_backbone_blocks + m.r_t * m.n_refine_blocks)
    pix = B * F * m.r_t * L * m.pix_per_token * (4 if case["pixels"] == "f32" else 2)
    return {"bytes": params + n * (ring + B * F * L * m.embed_in * es + pix), "flops": n * (gemm + attn)}


def tolerance(case):
    # about four times what the decode differs from exact() by (relative 2-norm)
    if case["dtype"] == "f32":
        return {"rel": 1e-5}
    if case["mlp"] != "f16":
        return {"rel": 0.03, "max": 0.6}  # an E4M3 code moves a whole step when its input's rounding moves
    return {"rel": 2e-2 if case["dtype"] == "bf16" else 6e-3, "max": 0.2 if case["dtype"] == "bf16" else 0.06}


# ------------------------------------------------------------------ the same in 64 bits

def _e4m3(x):
    """The nearest E4M3 value of fp32 x (ties to even), saturating."""
    return x.clamp(-448.0, 448.0).to(torch.float8_e4m3fn).double()


def _rows_e4m3(x, amax=None):
    """E4M3 values and scales of rows, by row maximum or at a fixed amplitude, scaled back."""
    x = x.float()
    a = x.abs().amax(-1, keepdim=True) if amax is None else torch.full_like(x[..., :1], amax)
    a = torch.where(a > 0, a, torch.full_like(a, 448.0))
    return _e4m3(x * (torch.full_like(a, 448.0) / a)) * (a / 448.0).double()


def _norm(x, w, p, m):
    if m.norm_kind == "ln":
        x = x - x.mean(-1, keepdim=True)
    x = x * torch.rsqrt((x * x).mean(-1, keepdim=True) + m.norm_eps) * w[p + ".g"]
    return x + w[p + ".b"] if m.norm_kind == "ln" else x


def _rotate(x, pos, m):
    """3D-RoPE of x [rows, vectors, D_h] at pos [rows, 3] (t, h, w), interleaved pairs."""
    if not m.rope:
        return x
    dh = m.head_dim
    sec = [dh // 4, 3 * dh // 8, dh - dh // 4 - 3 * dh // 8]
    ang = torch.cat([pos[:, a:a + 1] * m.rope_theta ** (-2.0 * torch.arange(s // 2, device=_DEV, dtype=torch.float64) / s)
                     for a, s in enumerate(sec)], 1)[:, None]
    a, b, cs, sn = x[..., 0::2], x[..., 1::2], torch.cos(ang), torch.sin(ang)
    return torch.stack([a * cs - b * sn, a * sn + b * cs], -1).flatten(-2)


def _attend(q, k, v, m):
    """q [N, rows, D_h] against k, v [G, keys, D_h], a slice of query rows at a time."""
    out = torch.empty_like(q)
    step = max(64, int(2e8 // k.shape[1]))
    for n in range(m.n_heads):
        kt, vn = k[n * m.n_kv_groups // m.n_heads].t().contiguous(), v[n * m.n_kv_groups // m.n_heads]
        for r in range(0, q.shape[1], step):
            s = torch.softmax(q[n, r:r + step] @ kt / math.sqrt(m.head_dim), -1)
            out[n, r:r + step] = s @ vn
    return out


def _stack(x, w, name, blocks, m, unit, pos):
    """A transformer stack over the units of one stream: x, pos [units, unit, ...]."""
    dh, G, N = m.head_dim, m.n_kv_groups, m.n_heads
    for i in range(blocks):
        p = "%s.%d" % (name, i)
        y = _norm(x, w, p + ".norm1", m) @ w[p + ".wqkv"].t() + w[p + ".bqkv"]
        qs, ks, vs, o = [], [], [], []
        for u in range(x.shape[0]):
            z = y[u].reshape(unit, N + 2 * G, dh)
            q, k, v = z[:, :N], z[:, N:N + G], z[:, N + G:]
            if m.kv_norm:
                k, v = [t * torch.rsqrt((t * t).mean(-1, keepdim=True) + m.norm_eps) * w["%s.%snorm.g" % (p, s)]
                        for t, s in ((k, "k"), (v, "v"))]
            qs.append(_rotate(q, pos[u], m).transpose(0, 1).contiguous())
            ks.append(_rotate(k, pos[u], m).transpose(0, 1).contiguous())
            vs.append(v.transpose(0, 1).contiguous())
        for u in range(x.shape[0]):
            lo = max(0, u - m.window + 1)
            a = _attend(qs[u], torch.cat(ks[lo:u + 1], 1), torch.cat(vs[lo:u + 1], 1), m)
            o.append(a.transpose(0, 1).reshape(unit, N * dh))
        x = x + torch.stack(o) @ w[p + ".wo"].t() + w[p + ".bo"]
        h = _norm(x, w, p + ".norm2", m)
        if m.mlp_kind == "gelu":
            h = torch.nn.functional.gelu(h @ w[p + ".w1"].t() + w[p + ".b1"])
            x = x + h @ w[p + ".w2"].t() + w[p + ".b2"]
            continue
        fp8, static = m.mlp_precision != "f16", m.mlp_precision == "fp8s"
        q8 = lambda t, a: _rows_e4m3(t, _AMAX[a] if static else None) if fp8 else t  # noqa: E731
        w13, w2 = (_rows_e4m3(w[p + s]) if fp8 else w[p + s] for s in (".w13", ".w2"))
        gate, up = (q8(h, 0) @ w13.t() + w[p + ".b13"]).chunk(2, -1)
        h = torch.nn.functional.silu(gate) * up
        x = x + q8(h.half() if fp8 else h, 1) @ w2.t() + w[p + ".b2"]
    return _norm(x, w, name + ".norm_f", m)


def exact(case, seed):
    m = _model(case)
    w = {k: v.double() for k, v in _weights(m, case).items()}
    L, gh, gw, s, F, r = m.tokens_per_frame, m.grid_h, m.grid_w, m.s_out, case["frames"], m.r_t
    hw = torch.stack(torch.meshgrid(torch.arange(gh), torch.arange(gw), indexing="ij"), -1).reshape(L, 2).to(_DEV)

    def positions(n):  # [n frames, L, 3]
        t = torch.arange(n, device=_DEV).view(n, 1, 1).expand(n, L, 1)
        return torch.cat([t, hw.expand(n, L, 2)], -1).double()

    outs = []
    for zs in _latents(m, case, seed):
        rows = []
        for z in zs.double():
            T = z.shape[1]
            x = torch.nn.functional.pixel_unshuffle(z.transpose(0, 1), m.patch) if m.patch > 1 else z.transpose(0, 1)
            x = x.reshape(T, m.embed_in, L).transpose(1, 2) @ w["embed.w"].t() + w["embed.b"]
            U = m.unit_frames
            x = _stack(x.reshape(T // U, U * L, m.dim), w, "bb", m.n_backbone_blocks, m, U * L,
                       positions(T).reshape(T // U, U * L, 3))
            x = x.reshape(T, L, m.dim)
            if m.head_kind == "temporal_first":
                x = (x @ w["tup.w"].t() + w["tup.b"]).reshape(T, L, r, m.dim).transpose(1, 2)
                x = _stack(x.reshape(T // U, U * r * L, m.dim), w, "rf", m.n_refine_blocks, m, U * r * L,
                           positions(T * r).reshape(T // U, U * r * L, 3))
                x = x.reshape(T, r, L, m.dim)[-F:]
                x = torch.nn.functional.silu(x @ w["head1.w"].t() + w["head1.b"]) @ w["head2.w"].t() + w["head2.b"]
            else:
                x = (x[-F:] @ w["head.w"].t() + w["head.b"]).reshape(F, L, r, -1).transpose(1, 2)
            # [F, r, L, C s^2] -> [C, F r, gh s, gw s]
            x = x.reshape(F * r, gh, gw, m.out_channels, s, s).permute(3, 0, 1, 4, 2, 5)
            rows.append(x.reshape(m.out_channels, F * r, gh * s, gw * s).clamp(-1.0, 1.0))
        outs.append(torch.stack(rows))
    return outs

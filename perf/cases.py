"""The work this framework does for a program that uses it, as measurable cases.

A case is one pass through the public entry points of `paper_2609_34144_amd` on inputs
of the shapes, types and distributions of a reconstruction-coupled DiT block: routing
over the historical KV, routed attention of the anchor frames, Phase-Aware
Reconstruction of the skipped frames, and control-aware frame selection.  Buffers and
workspaces are allocated once, as a serving loop keeps them.

`kind` of a case:
  step     one block step: routing, attention, PAR update of the residual site
  attn     cast_anchor_attn          route    cast_route_kv
  coupled  cast_route_coupled        par      cast_par_reconstruct
  select   cast_frame_select
"""
import math

import torch

import paper_2609_34144_amd as cast

DEV = "cuda"


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------

def _block(kind, **kw):
    c = {"kind": kind}
    c.update(kw)
    return c


def listed():
    # the two backbones of the benchmark: 704x1280 chunks (30x52 tokens, 12 heads) and
    # 480x832 chunks at the wider model (44x80 tokens, 24 heads), dh = 128
    matrix = dict(n_a=3, S=1560, H=12, dh=128, M=16, Bv=1560, topk=4, n0=0)
    hy = dict(n_a=4, S=3520, H=24, dh=128, M=32, Bv=3520, topk=8, n0=0)
    return [
        # the smallest whole step: what counts is launches and latency
        _block("step", name="step_tiny", frames=4, Hg=8, Wg=8, anchors="0,3", coupled=False,
               n_a=2, S=64, H=2, dh=32, M=4, Bv=64, topk=2, n0=0),
        # an ordinary step of the smaller backbone, edge tiles and ragged chunks
        _block("step", name="step_matrix", frames=8, Hg=30, Wg=52, anchors="0,3,7", coupled=False, **matrix),
        # the largest attention: four anchors over 8 of 32 historical frames
        _block("attn", name="attn_hy", **hy),
        # with the always-attended segment: one current frame and 77 text tokens
        _block("attn", name="attn_current", **dict(matrix, n0=1637)),
        # history routed in blocks of 8x8 tokens (a fifth of them kept) and a text
        # segment, on a backbone with 64-wide heads
        _block("attn", name="attn_blocks_dh64", n_a=3, S=1560, H=24, dh=64, M=390, Bv=64, topk=78, n0=77),
        # routing over whole-frame chunks, the bandwidth-bound scan
        _block("route", name="route_hy", **hy),
        # routing over 8x8-token blocks: 32 frames of 55 blocks, a fifth of them kept
        _block("route", name="route_blocks", **dict(hy, M=1760, Bv=64, topk=352)),
        # reconstruction-coupled routing on both granularities
        _block("coupled", name="coupled_hy", frames=16, anchors="0,4,8,12", **hy),
        _block("coupled", name="coupled_blocks", frames=8, anchors="0,3,7",
               **dict(matrix, M=390, Bv=64, topk=78)),
        # the residual update of a chunk (three anchor pairs, extrapolated tail)
        _block("par", name="par_hy", frames=16, Hg=44, Wg=80, D=3072, anchors="0,4,8,12", tile_h=8,
               tile_w=8, accumulate=1, update_anchors=0),
        # one long interval: 64 frames between two anchors
        _block("par", name="par_stress", frames=66, Hg=64, Wg=64, D=3072, anchors="0,65", tile_h=8,
               tile_w=8, accumulate=1, update_anchors=0),
        # the next block's anchors from both control branches
        _block("select", name="select_hy", frames=16, S=3520, D=3072, anchors="0,4,8,12", k_f=4,
               branches=2, fp32=False),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _anchors(rng, frames, n_a):
    """n_a strictly increasing frames, the first near the chunk's start."""
    rest = sorted(rng.sample(range(1, frames), n_a - 1))
    return ",".join(str(a) for a in [0 if rng.random() < 0.8 else rng.randrange(0, rest[0])] + rest)


def draw(rng):
    """A case of the same kinds over the ranges between the listed ones."""
    kind = rng.choice(["step", "step", "attn", "attn", "attn", "route", "coupled", "par", "par", "par", "select"])
    Hg, Wg = rng.randint(8, 64), rng.randint(8, 80)
    frames = rng.randint(4, 16)
    n_a = rng.randint(2, min(4, frames - 1))
    if kind == "par":
        if rng.random() < 0.3:
            frames = rng.randint(17, 66)
        th, tw = (8, 8) if rng.random() < 0.75 else (rng.randint(4, 8), rng.randint(4, 8))
        acc = int(rng.random() < 0.7)
        c = _block("par", frames=frames, Hg=Hg, Wg=Wg, D=rng.choice([64, 128]) * rng.randint(1, 24),
                   anchors=_anchors(rng, frames, n_a), tile_h=th, tile_w=tw, accumulate=acc,
                   update_anchors=int(rng.random() < 0.4))
    elif kind == "select":
        c = _block("select", frames=frames, S=Hg * Wg, D=rng.choice([64, 128]) * rng.randint(1, 24),
                   anchors=_anchors(rng, frames, n_a), k_f=n_a, branches=rng.choice([1, 2, 2]),
                   fp32=rng.random() < 0.3)
    else:
        S, H, dh = Hg * Wg, rng.randint(1, 24), rng.choice([32, 64, 64, 128, 128, 128])
        grain = rng.random()
        if grain < 0.5:            # a whole frame per chunk
            Bv, M = S, _logint(rng, 4, 32)
        elif grain < 0.85:         # 8x8-token blocks
            Bv, M = 64, _logint(rng, 32, 1760)
        else:                      # other granularities
            Bv, M = _logint(rng, 16, 1024), _logint(rng, 8, 128)
        topk = max(1, min(M, 1000, int(round(M * rng.uniform(0.1, 0.35)))))
        n0 = 0 if kind in ("route", "coupled") or rng.random() < 0.5 else rng.choice([77, 77 + S, rng.randint(1, 512)])
        c = _block(kind, n_a=n_a, S=S, H=H, dh=dh, M=M, Bv=Bv, topk=topk, n0=n0)
        if kind in ("step", "coupled"):
            c.update(frames=frames, anchors=_anchors(rng, frames, n_a))
        if kind == "step":
            c.update(Hg=Hg, Wg=Wg, coupled=rng.random() < 0.5)
    # never dearer than the largest listed cases
    while work(c)["flops"] > 4.8e12 or work(c)["bytes"] > 6.5e9:
        if "H" in c:
            c["H"] = max(1, c["H"] // 2)
        else:
            c["D"] = max(1, c["D"] // 2)
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed & ((1 << 62) - 1))
    return g


def _anchor_list(c):
    return [int(x) for x in c["anchors"].split(",")]


def _bf16(g, *shape, mean=None):
    x = torch.randn(shape, generator=g, device=DEV)
    if mean is not None:
        x += mean
    return x.to(torch.bfloat16)


def _qkv(c, g, s):
    n_a, S, H, dh, M, Bv = (c[k] for k in ("n_a", "S", "H", "dh", "M", "Bv"))
    # keys differ by chunk (a mean per chunk, head and channel), so routing has a signal
    mu = 0.5 * torch.randn((M, 1, H, dh), generator=g, device=DEV)
    s["q"] = _bf16(g, n_a, S, H, dh, mean=0.5 * torch.randn((n_a, 1, H, dh), generator=g, device=DEV))
    s["k"] = _bf16(g, M, Bv, H, dh, mean=mu)
    s["v"] = _bf16(g, M, Bv, H, dh)
    s["kc"] = s["vc"] = None
    if c["n0"] > 0:
        s["kc"], s["vc"] = _bf16(g, c["n0"], H, dh), _bf16(g, c["n0"], H, dh)


def _field(g, Hg, Wg, D):
    """A smooth periodic field per channel (power 1/f^2, unit RMS), as its spectrum."""
    fy = torch.fft.fftfreq(Hg, device=DEV)[:, None]
    fx = torch.fft.rfftfreq(Wg, device=DEV)[None, :]
    f = torch.sqrt(fy * fy + fx * fx)
    amp = torch.where(f > 0, 1.0 / f.clamp_min(1e-6), torch.zeros_like(f))
    spec = torch.fft.rfft2(torch.randn((Hg, Wg, D), generator=g, device=DEV), dim=(0, 1)) * amp[:, :, None]
    x = torch.fft.irfft2(spec, s=(Hg, Wg), dim=(0, 1))
    return spec / x.square().mean(dim=(0, 1)).sqrt().clamp_min(1e-12)


def _resid(c, g, s):
    """Anchor residuals: one field in translation, partly coherent per channel."""
    Hg, Wg, D = c["Hg"], c["Wg"], c.get("D") or c["H"] * c["dh"]
    base = _field(g, Hg, Wg, D)
    coh = torch.rand((D,), generator=g, device=DEV)
    fy = torch.fft.fftfreq(Hg, device=DEV)[:, None]
    fx = torch.fft.rfftfreq(Wg, device=DEV)[None, :]
    s["resid"] = torch.zeros((c["frames"], Hg, Wg, D), device=DEV)
    for a in _anchor_list(c):
        d = 8 * torch.rand((2,), generator=g, device=DEV) - 4
        shift = torch.polar(torch.ones_like(fy + fx), -2 * math.pi * (fy * d[0] + fx * d[1]))
        spec = coh * (base * shift[:, :, None]) + torch.sqrt(1 - coh * coh) * _field(g, Hg, Wg, D)
        s["resid"][a] = torch.fft.irfft2(spec, s=(Hg, Wg), dim=(0, 1))


def _ws(nbytes):
    return torch.empty(max(nbytes, 256), dtype=torch.uint8, device=DEV)


def _prepare_route(c, s):
    n_a, S, H, dh, M, Bv = (c[k] for k in ("n_a", "S", "H", "dh", "M", "Bv"))
    s["idx"] = torch.empty((n_a, H, min(c["topk"], M)), dtype=torch.int32, device=DEV)
    if c["kind"] == "coupled" or c.get("coupled"):
        s["u"] = torch.empty((n_a, H, M), device=DEV)
        s["route_ws"] = _ws(cast.cast_route_coupled_workspace_bytes(n_a, S, H, dh, M, Bv))
    else:
        s["scores"] = torch.empty((n_a, H, M), device=DEV)
        s["route_ws"] = _ws(cast.cast_route_kv_workspace_bytes(n_a, S, H, dh, M, Bv))


def _prepare_attn(c, s):
    n_a, S, H, dh = (c[k] for k in ("n_a", "S", "H", "dh"))
    s["out"] = torch.empty((n_a, S, H, dh), dtype=torch.bfloat16, device=DEV)
    s["attn_ws"] = _ws(cast.cast_anchor_attn_workspace_bytes(n_a, S, H, dh, min(c["topk"], c["M"]), c["n0"], c["Bv"]))


def _prepare_par(c, g, s):
    D = c.get("D") or c["H"] * c["dh"]
    s["prm"] = cast.cast_par_params_default(
        tile_h=c.get("tile_h", 8), tile_w=c.get("tile_w", 8), accumulate=c.get("accumulate", 1),
        update_anchors=c.get("update_anchors", 1))
    _resid(c, g, s)
    if s["prm"].accumulate:
        s["x"] = torch.randn(s["resid"].shape, generator=g, device=DEV)
    else:
        s["x"] = torch.zeros_like(s["resid"])
    s["par_ws"] = _ws(cast.cast_par_workspace_bytes(c["frames"], len(_anchor_list(c)), c["Hg"], c["Wg"], D, s["prm"]))


def prepare(case, seed):
    c, g = case, _gen(seed)
    s = {"c": c, "scale": 1.0 / math.sqrt(c.get("dh", 1))}
    if "anchors" in c:
        s["anchors"] = _anchor_list(c)
    if "H" in c:
        _qkv(c, g, s)
    if c["kind"] in ("step", "route", "coupled"):
        _prepare_route(c, s)
    if c["kind"] == "coupled" or c.get("coupled"):
        D = c["H"] * c["dh"]
        s["gram"] = cast.cast_wo_gram(_bf16(g, D, D) / math.sqrt(D), c["H"], c["dh"])
    if c["kind"] in ("step", "attn"):
        _prepare_attn(c, s)
    if c["kind"] == "attn":
        # the budget's chunks per (anchor, head), ascending, as routing writes them
        pick = torch.rand((c["n_a"], c["H"], c["M"]), generator=g, device=DEV).topk(min(c["topk"], c["M"])).indices
        s["idx"] = pick.sort().values.to(torch.int32)
    if c["kind"] in ("step", "par"):
        _prepare_par(c, g, s)
    if c["kind"] == "select":
        shape, n = (c["frames"], c["S"], c["D"]), c["frames"]
        s["delta"] = []
        for b in range(c["branches"]):
            mag = 0.3 + 2.7 * torch.rand((n, 1, 1), generator=g, device=DEV)
            x = torch.randn(shape, generator=g, device=DEV) * mag
            s["delta"].append(x if c["fp32"] else x.to(torch.bfloat16))
        s["ages0"] = torch.randint(0, 4, (n,), generator=g, device=DEV, dtype=torch.int32)
        s["ages"] = s["ages0"].clone()
        s["r"] = torch.zeros((2, n), device=DEV)
        s["score"] = torch.empty((n,), device=DEV)
        s["next"] = torch.empty((c["k_f"],), dtype=torch.int32, device=DEV)
        s["sel_ws"] = _ws(cast.cast_frame_select_workspace_bytes(n, c["S"], c["D"]))
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def _route(c, s):
    if c["kind"] == "coupled" or c.get("coupled"):
        _, k, _ = cast.cast_route_coupled(s["q"], s["k"], s["v"], s["gram"], s["anchors"], c["frames"], c["topk"],
                                          s["scale"], u_out=s["u"], idx_out=s["idx"], workspace=s["route_ws"])
        return k, {"idx": s["idx"], "u": s["u"]}
    _, k, _ = cast.cast_route_kv(s["q"], s["k"], c["topk"], s["scale"], scores_out=s["scores"], idx_out=s["idx"],
                                 workspace=s["route_ws"])
    return k, {"idx": s["idx"], "scores": s["scores"]}


def _attn(c, s, k_eff):
    cast.cast_anchor_attn(s["q"], s["k"], s["v"], s["idx"], k_eff, s["scale"], k_cur=s["kc"], v_cur=s["vc"],
                          out=s["out"], workspace=s["attn_ws"])
    return {"out": s["out"]}


def _par(c, s):
    cast.cast_par_reconstruct(s["resid"], s["anchors"], s["prm"], out=s["x"], workspace=s["par_ws"])
    return {"x": s["x"]}


def run(state):
    s, c = state, state["c"]
    kind = c["kind"]
    if kind in ("route", "coupled"):
        return _route(c, s)[1]
    if kind == "attn":
        return _attn(c, s, s["idx"].shape[2])
    if kind == "par":
        return _par(c, s)
    if kind == "select":
        d = s["delta"] + [None] * (2 - len(s["delta"]))
        cast.cast_frame_select(d[0], d[1], s["anchors"], c["k_f"], s["ages"], r_out=s["r"], score_out=s["score"],
                               anchors_out=s["next"], workspace=s["sel_ws"])
        return {"next": s["next"], "ages": s["ages"], "r": s["r"], "score": s["score"]}
    k_eff, got = _route(c, s)
    got.update(_attn(c, s, k_eff))
    got.update(_par(c, s))
    return got


# ---------------------------------------------------------------------------
# what a pass cannot do without, and how exactly it can be said
# ---------------------------------------------------------------------------

def work(case):
    c = case
    kind, b, f = c["kind"], 0.0, 0.0
    if kind in ("step", "route", "coupled"):
        D = c["H"] * c["dh"]
        kv = 2 if kind == "coupled" or c.get("coupled") else 1
        b += 2.0 * D * (c["n_a"] * c["S"] + kv * c["M"] * c["Bv"]) + 4.0 * c["n_a"] * c["H"] * (c["M"] + c["topk"])
        f += 2.0 * D * (c["n_a"] * c["S"] + kv * c["M"] * c["Bv"])
        if kv == 2:
            b += 4.0 * D * c["dh"]
            f += 2.0 * c["n_a"] * c["M"] * D * c["dh"]
    if kind in ("step", "attn"):
        k = min(c["topk"], c["M"])
        L, D = c["n0"] + k * c["Bv"], c["H"] * c["dh"]
        f += 4.0 * c["n_a"] * c["S"] * L * D
        b += 2.0 * D * (2.0 * c["n_a"] * c["S"] + 2.0 * (c["n0"] + min(c["n_a"] * k, c["M"]) * c["Bv"]))
    if kind in ("step", "par"):
        D, n_a = c.get("D") or c["H"] * c["dh"], len(_anchor_list(c))
        S, skip = c["Hg"] * c["Wg"], c["frames"] - len(_anchor_list(c))
        written = skip + (n_a if c.get("update_anchors", 1) else 0)
        b += 4.0 * S * D * (n_a + written * (2 if c.get("accumulate", 1) else 1))
        f += 30.0 * S * D * (n_a + skip)         # transforms and blend per element
    if kind == "select":
        n = float(c["frames"]) * c["S"] * c["D"] * c["branches"]
        b += n * (4 if c["fp32"] else 2)
        f += 2.0 * n
    return {"bytes": b, "flops": f}


def tolerance(case):
    # Measured against the 64-bit results, times about four.  Attention: bf16 outputs and
    # probabilities, 2.4e-3.  Pooled means, scores, omission proxies and tile transforms:
    # 32-bit sums.  Indices may differ where two scores agree to 32-bit rounding.
    if case["kind"] in ("attn", "step"):
        return {"rel": 1e-2, "max": 0.2, "differ": 0.002}
    if case["kind"] in ("route", "coupled"):
        return {"rel": 1e-5, "max": 4e-4, "differ": 0.002}
    return {"rel": 2e-6, "max": 1e-3}


# ---------------------------------------------------------------------------
# the same results in 64 bits, by plain torch
# ---------------------------------------------------------------------------

def _pooled(x):
    return torch.stack([y.double().mean(dim=0) for y in x])      # [n, H, dh]


def _ex_route(c, s):
    scores = s["scale"] * torch.einsum("ihd,mhd->ihm", _pooled(s["q"]), _pooled(s["k"]))
    return scores, scores.topk(min(c["topk"], c["M"])).indices.sort().values


def _ex_omission(c, s):
    qb, kb, vb = _pooled(s["q"]), _pooled(s["k"]), _pooled(s["v"])
    pi = torch.softmax(s["scale"] * torch.einsum("ihd,mhd->ihm", qb, kb), dim=-1)
    ob = torch.einsum("ihm,mhd->ihd", pi, vb)
    u = torch.empty_like(pi)
    for h in range(c["H"]):
        d = ob[:, h, None, :] - vb[None, :, h, :]
        u[:, h] = ((d @ s["gram"][h].double()) * d).sum(-1)
    return u * (pi / (1 - pi + 1e-8)) ** 2


def _ex_attn(c, s, idx):
    out = torch.empty(s["q"].shape, dtype=torch.float64, device=DEV)
    for i in range(c["n_a"]):
        for h in range(c["H"]):
            j = idx[i, h].long()
            k = s["k"][j, :, h].reshape(-1, c["dh"]).double()
            v = s["v"][j, :, h].reshape(-1, c["dh"]).double()
            if s["kc"] is not None:
                k, v = torch.cat([s["kc"][:, h].double(), k]), torch.cat([s["vc"][:, h].double(), v])
            p = torch.softmax(s["scale"] * (s["q"][i, :, h].double() @ k.t().contiguous()), dim=-1)
            out[i, :, h] = p @ v
    return out


def _gate(F_a, F_b, hp, wp):
    """theta and g of every stored bin [tiles..., ky, kx] from the two anchors' spectra
    [tiles..., ky, kx, channel]."""
    Z, W = (F_b * F_a.conj()).sum(-1), (F_b.abs() * F_a.abs()).sum(-1)
    nk = wp // 2 + 1
    ky = torch.arange(hp, device=DEV)[:, None].expand(hp, nk)
    kx = torch.arange(nk, device=DEV)[None, :].expand(hp, nk)
    own = (kx == 0) | (2 * kx == wp)                       # columns that hold their conjugates
    mirror = own & (2 * ky > hp)
    real = own & ((ky == 0) | (2 * ky == hp))
    # a mirror is the conjugate of its representative
    Z = torch.where(mirror, Z[..., (-torch.arange(hp, device=DEV)) % hp, :].conj(), Z)
    eta = 1e-6 * W.amax(dim=(-2, -1), keepdim=True) + 1e-8
    rel = (W > eta) & (Z.abs() > eta)
    theta = torch.where(rel & ~real, torch.angle(Z), torch.zeros_like(W))
    plus = rel & ~((ky == 0) & (kx == 0))
    kap = torch.where(own, 1.0, 2.0).double() * plus
    conf = torch.where(plus.any(-1).any(-1), (kap * Z.abs()).sum((-2, -1)) / ((kap * W).sum((-2, -1)) + 1e-8), 0.0)
    fy = torch.where(2 * ky <= hp, ky, ky - hp).double() / hp
    nu = torch.sqrt(fy * fy + (kx.double() / wp) ** 2)
    nu = nu / nu.max() if float(nu.max()) > 0 else nu
    f32 = lambda v: float(torch.tensor(v, dtype=torch.float32))  # noqa: E731  (the parameters are 32-bit)
    tau = 0.25 + 0.5 * nu ** 2
    return theta, torch.sigmoid((conf[..., None, None] - tau) / f32(0.10))


def _ex_par(c, s):
    Hg, Wg, th, tw = c["Hg"], c["Wg"], s["prm"].tile_h, s["prm"].tile_w
    anchors, frames, x = s["anchors"], c["frames"], s["x"].double()
    add = 1.0 if s["prm"].accumulate else 0.0
    if s["prm"].update_anchors:
        for a in anchors:
            x[a] = add * x[a] + s["resid"][a].double()
    ys = [(0, Hg // th, th)] if Hg >= th else []
    ys += [(Hg - Hg % th, 1, Hg % th)] if Hg % th else []
    xs = [(0, Wg // tw, tw)] if Wg >= tw else []
    xs += [(Wg - Wg % tw, 1, Wg % tw)] if Wg % tw else []
    for y0, ny, hp in ys:
        for x0, nx, wp in xs:
            rows, cols = slice(y0, y0 + ny * hp), slice(x0, x0 + nx * wp)

            def spectrum(a):
                r = s["resid"][a, rows, cols].double().reshape(ny, hp, nx, wp, -1).permute(0, 2, 1, 3, 4)
                return torch.fft.rfft2(r, dim=(2, 3), norm="ortho")
            for p in range(len(anchors) - 1):
                fa, fb = anchors[p], anchors[p + 1]
                targets = list(range(fa + 1, fb))
                targets += list(range(0, fa)) if p == 0 else []
                targets += list(range(fb + 1, frames)) if p == len(anchors) - 2 else []
                if not targets:
                    continue
                A, B = spectrum(fa), spectrum(fb)
                theta, g = _gate(A, B, hp, wp)
                for t in targets:
                    al = (t - fa) / (fb - fa)
                    wa = torch.polar((1 - al) * torch.ones_like(theta), g * al * theta)[..., None]
                    wb = torch.polar(al * torch.ones_like(theta), -g * (1 - al) * theta)[..., None]
                    r = torch.fft.irfft2(wa * A + wb * B, s=(hp, wp), dim=(2, 3), norm="ortho")
                    r = r.permute(0, 2, 1, 3, 4).reshape(ny * hp, nx * wp, -1)
                    x[t, rows, cols] = add * x[t, rows, cols] + r
    return x


def _ex_select(c, s):
    r = torch.zeros((2, c["frames"]), dtype=torch.float64, device=DEV)
    d = torch.zeros((c["frames"],), dtype=torch.float64, device=DEV)
    for b, x in enumerate(s["delta"]):
        r[b] = torch.stack([f.double().square().mean().sqrt() for f in x])
        d += (r[b] - r[b].min()) / (r[b].max() - r[b].min() + 1e-8) / len(s["delta"])
    h = s["ages0"].double() + 1
    h[s["anchors"]] = 0
    return {"next": None, "ages": None, "r": r, "score": d + 0.5 * h / math.ceil(c["frames"] / c["k_f"])}


def exact(case, seed):
    c, s = case, prepare(case, seed)
    kind = c["kind"]
    if kind == "select":
        return _ex_select(c, s)
    if kind == "attn":
        return {"out": _ex_attn(c, s, s["idx"])}
    if kind == "par":
        return {"x": _ex_par(c, s)}
    if kind == "coupled":
        return {"idx": None, "u": _ex_omission(c, s)}
    if kind == "route":
        return {"idx": None, "scores": _ex_route(c, s)[0]}
    # a step: the attention that follows the 64-bit routing; coupled masks come from a
    # search, so what depends on them has no such value here
    if c["coupled"]:
        return {"idx": None, "u": _ex_omission(c, s), "out": None, "x": _ex_par(c, s)}
    scores, idx = _ex_route(c, s)
    return {"idx": None, "scores": scores, "out": _ex_attn(c, s, idx), "x": _ex_par(c, s)}

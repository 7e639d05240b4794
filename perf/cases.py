"""The calls whose speed matters: what one image or batch takes through the framework.

A user's program condenses an image (density, resize, or the preview block and the density of its
embeddings), runs the vision encoder's window and full attention, the language model's prefill
attention before and after pruning, and the selection with its gather.  Each case is one of these
calls through ``paper_2608_27206_amd.pace``, with outputs and workspaces that the program keeps.
Shapes are those of ``paper_2608_27206_amd.workloads``: 14-pixel patches, 8x8-patch windows, 2x2
merge, 16 heads of 80 in the encoder, 28/4 heads of 128 and rows of 3584 in the language model.
"""
import functools
import math

import numpy as np
import torch

from paper_2608_27206_amd import pace
from paper_2608_27206_amd import workloads as wl

DEV = "cuda"
DIM, FFN = 1280, 3420          # the preview block of the encoder
EXACT_ROWS = 2048              # query rows that exact() handles at a time


def listed():
    batch = wl.varlen_resolutions(4)
    nv = [(h // 28) * (w // 28) for h, w in batch]
    return [
        # one small photo's density: the shortest call of the front end, launches and latency
        {"name": "density_448", "kind": "density", "H": 448, "W": 448},
        # a 4K frame's density and its 2x shrink, before the encoder sees it
        {"name": "density_4k", "kind": "density", "H": 2156, "W": 3836},
        {"name": "resize_4k", "kind": "resize", "H": 2156, "W": 3836, "oH": 1078, "oW": 1918},
        # the same frame scored with the encoder's first block as the preview
        {"name": "preview_4k", "kind": "preview", "H": 2156, "W": 3836},
        # the window attention of an encoder layer at 4K, with ragged windows at two edges
        {"name": "window_4k", "kind": "window", "grids": "154x274", "mass": True},
        # the full-attention layer whose key mass the selection reads: a small photo, a packed
        # batch of eight images of odd sizes, and the 4K frame (the largest call there is)
        {"name": "full_448", "kind": "full", "lens": "1024", "heads": 16, "d": 80, "mass": True},
        {"name": "full_varlen8", "kind": "full", "lens": ",".join(str(4 * n) for n in nv), "heads": 16, "d": 80,
         "mass": True},
        {"name": "full_4k", "kind": "full", "lens": "42196", "heads": 16, "d": 80, "mass": True},
        # the prefill of the shortened context after pruning (no mass), and the layer at full
        # length whose text rows give the language model's mass
        {"name": "prefill_pruned", "kind": "prefill", "vis": "1055", "text": "128", "hq": 28, "hkv": 4, "d": 128,
         "rows": "none"},
        {"name": "prefill_4k", "kind": "prefill", "vis": "10549", "text": "128", "hq": 28, "hkv": 4, "d": 128,
         "rows": "text"},
        # fusion, top-K and gather for one 4K frame, and for a batch of sixteen
        {"name": "select_4k", "kind": "select", "grids": "154x274", "keep": 0.10, "mode": 0, "hidden": 3584},
        {"name": "select_x16", "kind": "select", "grids": ",".join(["154x274"] * 16), "keep": 0.10, "mode": 0,
         "hidden": 3584},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["density", "resize", "preview", "window", "full", "full", "prefill", "prefill", "select"])
    side = lambda lo, hi, m: max(1, _log(rng, lo, hi) // m) * m   # noqa: E731
    if kind == "density":
        return {"kind": kind, "H": side(224, 2156, 14), "W": side(224, 3836, 14)}
    if kind == "resize":
        # what the area ratio and the pixel budget ask for: 1x to 4.5x per side
        H, W, s = _log(rng, 300, 2156), _log(rng, 300, 3836), rng.uniform(1.0, 4.5)
        return {"kind": kind, "H": H, "W": W, "oH": max(1, int(H / s)), "oW": max(1, int(W / s))}
    if kind == "preview":
        return {"kind": kind, "H": side(224, 2156, 28), "W": side(224, 3836, 28)}
    if kind in ("window", "select"):
        n = _log(rng, 1, 8)
        grids = ",".join(f"{2 * _log(rng, 5, 77)}x{2 * _log(rng, 5, 137)}" for _ in range(n))
        if kind == "window":
            return {"kind": kind, "grids": grids, "mass": rng.random() < 0.5}
        return {"kind": kind, "grids": grids, "keep": rng.uniform(0.03, 0.3), "mode": rng.randrange(2),
                "hidden": rng.choice([2048, 3584])}
    n = _log(rng, 1, 8)
    if kind == "full":
        # mostly the encoder's heads of 80; merged grids give multiples of four patches, crops do not
        lens = [_log(rng, 100, 30000 // n) for _ in range(n)]
        if rng.random() < 0.5:
            lens = [x // 4 * 4 for x in lens]
        return {"kind": kind, "lens": ",".join(map(str, lens)), "heads": 16, "d": 128 if rng.random() < 0.15 else 80,
                "mass": rng.random() < 0.8}
    vis = ",".join(str(_log(rng, 49, 9000 // n)) for _ in range(n))
    text = ",".join(str(rng.randrange(16, 257)) for _ in range(n))
    hq, hkv = rng.choice([(28, 4), (28, 4), (8, 2), (16, 16)])
    return {"kind": kind, "vis": vis, "text": text, "hq": hq, "hkv": hkv, "d": 128,
            "rows": rng.choice(["text", "text", "all", "none"])}


# ---------------------------------------------------------------- inputs
def _ints(s):
    return [int(x) for x in s.split(",")]


def _pairs(s):
    return [tuple(int(y) for y in x.split("x")) for x in s.split(",")]


def _cu(lens):
    return torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32, device=DEV)


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _normal(g, shape, dtype=torch.bfloat16, scale=1.0):
    return (torch.randn(shape, generator=g, device=DEV) * scale).to(dtype)


def _empty(*shape, dtype=torch.float32):
    return torch.empty(shape, dtype=dtype, device=DEV)


@functools.lru_cache(maxsize=64)
def _layout(gh, gw):
    return wl.vit_layout(gh, gw)


def _image(g, H, W):
    """Smooth per-channel waves with a fifth of the patches replaced by texture."""
    r = torch.rand((3, 3), generator=g, device=DEV)
    y = torch.arange(H, device=DEV)[:, None, None] / H
    x = torch.arange(W, device=DEV)[None, :, None] / W
    v = 127.5 + 100.0 * torch.sin(2 * math.pi * ((0.5 + 1.5 * r[0]) * x + (0.5 + 1.5 * r[1]) * y + r[2]))
    tex = torch.randint(0, 256, (H, W, 3), generator=g, device=DEV)
    gh, gw = -(-H // wl.PATCH), -(-W // wl.PATCH)
    pick = (torch.rand((gh, gw, 1), generator=g, device=DEV) < 0.2).repeat_interleave(wl.PATCH, 0)
    pick = pick.repeat_interleave(wl.PATCH, 1)[:H, :W]
    return torch.where(pick, tex, (v + 0.5).floor().long()).clamp(0, 255).to(torch.uint8).contiguous()


def _preview_weights(g):
    """Device weights in the layout of pace.preview_weights_to_device."""
    kin = 3 * wl.PATCH ** 2
    kp, f8 = -(-kin // 8) * 8, -(-FFN // 8) * 8
    mat = lambda n, k: _normal(g, (n, k), scale=k ** -0.5)   # noqa: E731
    vec = lambda n, s: torch.randn(n, generator=g, device=DEV) * s   # noqa: E731
    w = {"dim": DIM, "ffn": f8, "pe": torch.zeros((DIM, kp), dtype=torch.bfloat16, device=DEV)}
    w["pe"][:, :kin] = mat(DIM, kin)
    for k in "qkvo":
        w["w" + k], w["b" + k] = mat(DIM, DIM), vec(DIM, 0.02)
    w["g1"], w["g2"] = 1 + vec(DIM, 0.1), 1 + vec(DIM, 0.1)
    w["wgu"] = torch.zeros((2 * f8, DIM), dtype=torch.bfloat16, device=DEV)
    w["wgu"][:2 * FFN] = mat(2 * FFN, DIM)
    w["bgu"] = torch.zeros(2 * f8, device=DEV)
    w["bgu"][:2 * FFN] = vec(2 * FFN, 0.02)
    w["wd"] = torch.zeros((DIM, f8), dtype=torch.bfloat16, device=DEV)
    w["wd"][:, :FFN] = mat(DIM, FFN)
    w["bd"] = vec(DIM, 0.02)
    return w


def prepare(case, seed):
    g, s = _gen(seed), dict(case)
    L = pace.lib()
    ws = lambda n: torch.empty(max(1, int(n)), dtype=torch.uint8, device=DEV)   # noqa: E731
    kind = case["kind"]
    if kind in ("density", "resize", "preview"):
        H, W = case["H"], case["W"]
        s["img"] = _image(g, H, W)
        N = (H // wl.PATCH) * (W // wl.PATCH)
        if kind == "resize":
            s["dst"] = _empty(case["oH"], case["oW"], 3, dtype=torch.uint8)
            return s
        s["d_out"], s["rho"] = _empty(N), _empty(3)
        if kind == "density":
            s["ws"] = ws(L.pace_apc_density_workspace_size(H, W, wl.PATCH))
            return s
        lay = _layout(H // wl.PATCH, W // wl.PATCH)
        s["order"] = torch.tensor(lay.order, dtype=torch.int32, device=DEV)
        s["cu"], s["max"] = torch.tensor(lay.cu_windows, device=DEV), int(max(lay.window_sizes))
        s["w"] = _preview_weights(g)
        s["emb"] = _empty(N, DIM, dtype=torch.bfloat16)
        s["ws"] = ws(L.pace_apc_preview_workspace_size(N, DIM, s["w"]["ffn"], wl.PATCH))
        s["ws2"] = ws(L.pace_apc_density_features_workspace_size(N, DIM))
        return s
    if kind in ("window", "full"):
        if kind == "window":
            lens, heads, d = [n for gh, gw in _pairs(case["grids"]) for n in _layout(gh, gw).window_sizes], 16, 80
        else:
            lens, heads, d = _ints(case["lens"]), case["heads"], case["d"]
        N = sum(lens)
        s["lens"], s["cu"], s["max"] = lens, _cu(lens), max(lens)
        s["q"], s["k"], s["v"] = (_normal(g, (N, heads, d)) for _ in range(3))
        s["o"], s["lse"] = torch.empty_like(s["q"]), _empty(heads, N)
        s["m"] = _empty(heads, N) if case["mass"] else None
        s["ws"] = ws(L.pace_vit_attention_workspace_size(N, heads, d, len(lens), max(lens)))
        return s
    if kind == "prefill":
        vis, text = _ints(case["vis"]), _ints(case["text"])
        hq, hkv, d = case["hq"], case["hkv"], case["d"]
        lens = [a + b for a, b in zip(vis, text)]
        N = sum(lens)
        q, k, v = _normal(g, (N, hq, d)), _normal(g, (N, hkv, d), torch.float32), _normal(g, (N, hkv, d))
        # a twentieth of the visual keys stand out along one direction per head
        u = torch.randn((hkv, d), generator=g, device=DEV)
        u = 3.0 * u / u.norm(dim=1, keepdim=True)
        off = 0
        for nv, n in zip(vis, lens):
            k[off:off + nv] += (torch.rand((nv, 1, 1), generator=g, device=DEV) < 0.05) * u
            off += n
        s["q"], s["k"], s["v"] = q, k.to(torch.bfloat16), v
        s["lens"], s["vis_l"], s["cu"], s["max"] = lens, vis, _cu(lens), max(lens)
        s["vis_len"], s["cu_vis"] = torch.tensor(vis, dtype=torch.int32, device=DEV), _cu(vis)
        rows = [(0, n) if case["rows"] == "all" else (nv, n - nv) for nv, n in zip(vis, lens)]
        s["rows_l"] = rows
        s["mq_start"], s["mq_len"] = (torch.tensor(x, dtype=torch.int32, device=DEV) for x in zip(*rows))
        s["o"], s["lse"] = torch.empty_like(q), _empty(hq, N)
        s["m"] = _empty(hq, sum(vis)) if case["rows"] != "none" else None
        return s
    lays = [_layout(gh, gw) for gh, gw in _pairs(case["grids"])]
    nv = [x.n_vis for x in lays]
    n = sum(nv)
    s["nv"], s["k_l"] = nv, [pace.keep_count(case["keep"], x) for x in nv]
    s["perm"] = torch.tensor(np.concatenate([x.vis_perm for x in lays]), dtype=torch.int32, device=DEV)
    # masses are positive and long-tailed; a few tokens collect several times the mean
    s["vis"] = torch.randn((16, 4 * n), generator=g, device=DEV).mul_(0.5).exp_()
    s["llm"] = torch.randn((28, n), generator=g, device=DEV).mul_(0.7).exp_()
    s["rows"] = _normal(g, (n, case["hidden"]))
    kt = max(1, sum(s["k_l"]))
    s["idx"], s["score"] = _empty(kt, dtype=torch.int32), _empty(n)
    s["fuse"], s["out"] = _empty(len(nv), 4), _empty(kt, case["hidden"], dtype=torch.bfloat16)
    s["ws"] = ws(L.pace_ddae_select_workspace_size(n, len(nv)))
    return s


def run(s):
    kind = s["kind"]
    if kind == "density":
        return pace.apc_density(s["img"], d_out=s["d_out"], rho_out=s["rho"], workspace=s["ws"])
    if kind == "resize":
        return pace.apc_downsample(s["img"], s["oH"], s["oW"], dst=s["dst"])
    if kind == "preview":
        emb = pace.apc_preview(s["img"], wl.PATCH, s["order"], s["cu"], s["max"], s["w"], out=s["emb"],
                               workspace=s["ws"])
        return (emb,) + pace.apc_density_features(emb, d_out=s["d_out"], rho_out=s["rho"], workspace=s["ws2"])
    if kind in ("window", "full"):
        return pace.vit_attention(s["q"], s["k"], s["v"], s["cu"], s["max"], want_mass=s["mass"], o=s["o"],
                                  lse=s["lse"], mass=s["m"], workspace=s["ws"])
    if kind == "prefill":
        return pace.prefill_attention_with_mass(
            s["q"], s["k"], s["v"], s["cu"], s["max"], s["vis_len"], s["cu_vis"], sum(s["vis_l"]), max(s["vis_l"]),
            s["mq_start"], s["mq_len"], max(b for _, b in s["rows_l"]), want_mass=s["m"] is not None, o=s["o"],
            lse=s["lse"], mass=s["m"])
    return pace.ddae_select(s["vis"], 4, s["perm"], s["llm"], s["nv"], s["k_l"], mode=s["mode"], hidden=s["rows"],
                            idx_out=s["idx"], score_out=s["score"], fuse_out=s["fuse"], out=s["out"],
                            workspace=s["ws"])


# ---------------------------------------------------------------- what a pass cannot do without
def work(case):
    kind = case["kind"]
    if kind in ("density", "resize", "preview"):
        H, W = case["H"], case["W"]
        N = (H // wl.PATCH) * (W // wl.PATCH)
        if kind == "density":
            return {"bytes": 3 * H * W + 4 * N + 12, "flops": 0}
        if kind == "resize":
            return {"bytes": 3 * (H * W + case["oH"] * case["oW"]), "flops": 0}
        kin = 3 * wl.PATCH ** 2
        weights = DIM * (kin + 4 * DIM + 3 * FFN)
        pairs = sum(x * x for x in _layout(H // wl.PATCH, W // wl.PATCH).window_sizes)
        return {"bytes": 3 * H * W + 2 * weights + 2 * N * DIM + 4 * N, "flops": 2 * N * weights + 4 * DIM * pairs}
    if kind in ("window", "full"):
        lens = ([n for gh, gw in _pairs(case["grids"]) for n in _layout(gh, gw).window_sizes] if kind == "window"
                else _ints(case["lens"]))
        heads, d = case.get("heads", 16), case.get("d", 80)
        N = sum(lens)
        return {"bytes": 8 * N * heads * d + 4 * N * heads * (1 + case["mass"]),
                "flops": 4 * d * heads * sum(n * n for n in lens)}
    if kind == "prefill":
        vis, text = _ints(case["vis"]), _ints(case["text"])
        lens, hq, hkv, d = [a + b for a, b in zip(vis, text)], case["hq"], case["hkv"], case["d"]
        N = sum(lens)
        return {"bytes": 4 * N * d * (hq + hkv) + 4 * N * hq + (4 * sum(vis) * hq if case["rows"] != "none" else 0),
                "flops": 2 * d * hq * sum(n * (n + 1) for n in lens)}
    nv = [(gh // 2) * (gw // 2) for gh, gw in _pairs(case["grids"])]
    kt = sum(pace.keep_count(case["keep"], x) for x in nv)
    return {"bytes": sum(nv) * 4 * (16 * 4 + 28 + 1 + 1) + 4 * kt + 4 * kt * case["hidden"], "flops": 0}


def tolerance(case):
    kind = case["kind"]
    if kind == "density":
        return {"rel": 4e-6}      # sums of 588 products in 32 bits: 8e-7 off the 64-bit values
    if kind == "resize":
        return {"rel": 0.0, "differ": 1e-5}   # bytes: only where a 32-bit sum lies on a rounding boundary
    if kind == "select":
        return {"rel": 2e-6}      # sums over the heads in 32 bits: 2.4e-7 off
    if kind == "preview":
        return {"rel": 1.5e-2}    # ten activations stored in bf16, one after the other: 4.4e-3 off
    return {"rel": 8e-3}          # bf16 products and outputs: 2.1e-3 off


# ---------------------------------------------------------------- the same in 64 bits
def _density64(T):
    c = T.mean(0)
    phi = (c * c).sum()
    nc = c.norm()
    d = (T - (c / nc if nc > 1e-5 else 0 * c)).norm(dim=1)
    tail = d.topk(max(1, math.ceil(0.10 * len(d) - 1e-9))).values.mean()
    rho_g, rho_d = 1 - phi, (tail / 1.5).clamp(max=1.0)
    return torch.stack([rho_g, rho_d, 0.6 * rho_g + 0.4 * rho_d]), d


def _patches64(img):
    H, W, _ = img.shape
    P = wl.PATCH
    x = img.double() / 127.5 - 1.0
    return x.view(H // P, P, W // P, P, 3).permute(0, 2, 1, 3, 4).reshape(-1, 3 * P * P)


def _attend64(q, k, v, causal, rows, keys):
    """One head's O, LSE and the mass of keys [keys) over query rows [rows), in 64 bits."""
    n, scale = len(q), 1.0 / math.sqrt(q.shape[1])
    o, lse, mass = torch.empty_like(q), q.new_empty(n), q.new_zeros(keys[1] - keys[0])
    for r0 in range(0, n, EXACT_ROWS):
        r1 = min(n, r0 + EXACT_ROWS)
        end = r1 if causal else n
        sc = (q[r0:r1] @ k[:end].T).mul_(scale)
        if causal:
            sc.masked_fill_(torch.arange(end, device=DEV)[None, :] > torch.arange(r0, r1, device=DEV)[:, None],
                            -math.inf)
        lse[r0:r1] = torch.logsumexp(sc, 1)
        p = sc.sub_(lse[r0:r1, None]).exp_()
        o[r0:r1] = p @ v[:end]
        a, b = max(r0, rows[0]), min(r1, rows[1])
        if a < b and keys[0] < end:
            c = p[a - r0:b - r0, keys[0]:min(end, keys[1])].sum(0)
            mass[:len(c)] += c
    return o, lse, mass


def _windows64(q, k, v, lens):
    """All windows at once, padded to the longest: O, LSE [heads, N] and mass [heads, N]."""
    N, H, d = q.shape
    ln = torch.tensor(lens, device=DEV)
    col = torch.arange(int(ln.max()), device=DEV)[None, :]
    ok = col < ln[:, None]
    at = torch.where(ok, (ln.cumsum(0) - ln)[:, None] + col, 0)
    o, lse, mass = q.new_empty((N, H, d)), q.new_empty((H, N)), q.new_empty((H, N))
    for h in range(H):
        qh, kh, vh = (t[:, h][at] for t in (q, k, v))
        s = (qh @ kh.transpose(1, 2).contiguous()) / math.sqrt(d)
        s.masked_fill_(~ok[:, None, :], -math.inf)
        lw = torch.logsumexp(s, 2)
        p = (s - lw[..., None]).exp()
        o[:, h] = (p @ vh)[ok]
        lse[h] = lw[ok]
        mass[h] = (p * ok[..., None]).sum(1)[ok]
    return o, lse, mass


def exact(case, seed):
    s = prepare(case, seed)
    kind = case["kind"]
    if kind == "density":
        x = _patches64(s["img"])
        return _density64(x / x.norm(dim=1, keepdim=True))
    if kind == "resize":
        return None   # bytes
    if kind == "preview":
        w = {a: b.double() for a, b in s["w"].items() if torch.is_tensor(b)}
        norm = lambda t, g: t * (t.square().mean(1, keepdim=True) + 1e-6).rsqrt() * g   # noqa: E731
        x = _patches64(s["img"])[s["order"].long()]
        h0 = x @ w["pe"][:, :x.shape[1]].T
        u = norm(h0, w["g1"])
        q, k, v = ((u @ w["w" + c].T + w["b" + c]).view(-1, DIM // 80, 80) for c in "qkv")
        lens = (s["cu"][1:] - s["cu"][:-1]).tolist()
        h1 = h0 + _windows64(q, k, v, lens)[0].reshape(-1, DIM) @ w["wo"].T + w["bo"]
        u = norm(h1, w["g2"])
        gu = u @ w["wgu"].T + w["bgu"]
        gate, up = gu[:, 0::2], gu[:, 1::2]
        e = h1 + (gate * torch.sigmoid(gate) * up) @ w["wd"].T + w["bd"]
        return (e,) + _density64(e / e.norm(dim=1, keepdim=True).clamp(min=1e-12))
    if kind == "select":
        V, lm = s["vis"].double().sum(0).view(-1, 4).sum(1), s["llm"].double().sum(0)
        scores, fuse, off = [], [], 0
        for n in s["nv"]:
            a, b = V[off:off + n][s["perm"][off:off + n].long()], lm[off:off + n]
            a, b = ((t - t.min()) / (t.max() - t.min()) for t in (a, b))
            sv, sl = a.std(correction=0), b.std(correction=0)
            wl_ = torch.sigmoid((sl - sv) / 0.5) if case["mode"] == 0 else torch.full_like(sv, 0.5)
            scores.append(wl_ * b + (1 - wl_) * a)
            fuse.append(torch.stack([sl, sv, wl_, 1 - wl_]))
            off += n
        return None, torch.cat(scores), torch.stack(fuse), None   # indices and copied rows have none
    q, k, v = (s[c].double() for c in "qkv")
    if kind == "window":
        o, lse, m = _windows64(q, k, v, s["lens"])
        return o, lse, (m if case["mass"] else None)
    causal = kind == "prefill"
    N, H, _ = q.shape
    group = H // k.shape[1]
    vis = s["vis_l"] if causal else s["lens"]
    o, lse, m = torch.empty_like(q), q.new_empty((H, N)), q.new_empty((H, sum(vis)))
    for h in range(H):
        qh, kh, vh = q[:, h].contiguous(), k[:, h // group].contiguous(), v[:, h // group].contiguous()
        t0 = v0 = 0
        for i, n in enumerate(s["lens"]):
            start, count = s["rows_l"][i] if causal else (0, n)
            r = _attend64(qh[t0:t0 + n], kh[t0:t0 + n], vh[t0:t0 + n], causal, (start, start + count), (0, vis[i]))
            o[t0:t0 + n, h], lse[h, t0:t0 + n], m[h, v0:v0 + vis[i]] = r
            t0, v0 = t0 + n, v0 + vis[i]
    return o, lse, (m if s["m"] is not None else None)

"""The work that programs have this library do, as cases to time and compare.

One case is one call sequence of a video diffusion transformer's attention
layer (or of the code around it) through the package's entry points, on
activations of a latent clip: Q, K, V of a T x H x W grid, routed and attended
in 3D boxes or in runs of a Hilbert curve. Buffers and workspaces are made
once, as a model does that runs the same layer shape on every step.

Inputs are seeded synthetic activations: unit normal Q, K, V plus a sinusoidal
position embedding in Q and K whose weight differs from head to head, so that
heads keep anything from a few per cent of the key blocks to most of them.
"""

import math

import numpy as np
import torch

import paper_2607_16190_amd as fva

HEAD_DIM = 128
GAMMA2 = 0.3  # weight of the position embedding at alpha = 1

GRID_480P = (21, 30, 52)
GRID_720P = (21, 45, 80)
GRID_LONG = (31, 45, 80)
BOX = (2, 8, 8)


def _case(name, kind, grid, heads, box=BOX, batch=1, p=0.9, k_min=4, layout="bhnd", alphas="spread", v="bf16", ranks=0):
    """box: block extents (a run of a curve-ordered sequence is (1, 1, n)); layout: order of the tensors' axes in
    memory; alphas: how the heads' position weights are spread ("spread" or "stress": one head in five flat, the
    others concentrated); v: the type V is multiplied in; ranks: ranks that the heads are dealt out to."""
    c = dict(kind=kind, T=grid[0], H=grid[1], W=grid[2], bt=box[0], bh=box[1], bw=box[2], heads=heads, batch=batch,
             p=p, k_min=k_min, layout=layout, alphas=alphas, v=v, ranks=ranks)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest call: a preview-sized clip, two heads. Latency and the number of launches count.
        _case("step_tiny", "step", (3, 16, 16), 2, box=(1, 8, 8), k_min=2),
        # One GPU's five heads of forty when eight GPUs share a 480p clip, in the layout in which a model's
        # projection leaves them (tokens before heads).
        _case("step_480p_share", "step", GRID_480P, 5, layout="bnhd"),
        # The full layer of a 720p, 81-frame clip on one GPU: the workload of bench.py.
        _case("step_720p", "step", GRID_720P, 40),
        # The attention alone on lists that an earlier step routed, for programs that may not allocate
        # (graph capture, serving loops): one GPU's share of 720p.
        _case("noalloc_720p_share", "noalloc", GRID_720P, 5),
        # The largest: a long clip (111,600 tokens, 960 blocks), attention on given lists.
        _case("attn_long", "attn", GRID_LONG, 40),
        # The quantised-V step (V to E4M3 inside the step) of one GPU's share of 480p.
        _case("fp8_480p_share", "step", GRID_480P, 5, v="e4m3"),
        # The same in curve-ordered blocks at the full 720p size: every block full but the last.
        _case("fp8_curve_720p", "step", GRID_720P, 40, box=(1, 1, 128), v="e4m3"),
        # Routing alone: a program that looks at the mask (sharing it between steps, load planning).
        _case("route_720p", "route", GRID_720P, 40),
        # Routing with slack-aware augmentation over 8 ranks of 5 heads, very uneven heads.
        _case("sasa_720p", "sasa", GRID_720P, 40, alphas="stress", ranks=8),
        # V to E4M3 tiles alone, as a program that quantises once for several attention calls does.
        _case("quantize_720p", "quantize", GRID_720P, 40, v="e4m3"),
        # One tensor into curve order and back: what a model pays around its attention layers.
        _case("permute_720p", "permute", GRID_720P, 40, box=(1, 1, 128)),
        # A clip of another size arrives: the token order of its grid, then Q, K and V into it (one GPU's share).
        _case("curve_layout_480p", "curve_layout", GRID_480P, 5, box=(1, 1, 128)),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    """A case of the listed ones' ranges: grids from preview size to the long clip (partial boxes at every end among
    them), 1 to 40 heads, every kind of call, block organisation, layout and V type that the listed cases use."""
    while True:
        kind = rng.choice(("step", "step", "step", "attn", "noalloc", "route", "sasa", "quantize", "permute",
                           "curve_layout"))
        grid = (_log_int(rng, 2, 31), _log_int(rng, 12, 45), _log_int(rng, 12, 80))
        box = rng.choice(((2, 8, 8), (2, 8, 8), (1, 8, 8), (1, 1, 128), (1, 1, 64)))
        if kind in ("permute", "curve_layout"):
            box = (1, 1, 128)
        v = "e4m3" if kind == "quantize" else rng.choice(("bf16", "e4m3")) if kind in ("step", "attn") else "bf16"
        c = _case(None, kind, grid, _log_int(rng, 1, 40), box=box, batch=rng.choice((1, 1, 1, 2)),
                  p=rng.choice((0.8, 0.9, 0.9, 0.95)), k_min=rng.choice((2, 4, 4, 6)),
                  layout=rng.choice(("bhnd", "bnhd")), alphas=rng.choice(("spread", "spread", "stress")), v=v)
        if kind == "sasa":
            c["ranks"] = rng.choice((2, 4, 8))
        nb = _blocks(c)
        heads = c["heads"] * c["batch"]
        # at most 1024 blocks, and no more work than the largest listed case
        if 4 <= nb <= 1024 and heads <= 40 and heads * _tokens(c) ** 2 <= 30 * 111600 ** 2:
            return c


# ---- shapes -----------------------------------------------------------------


def _tokens(c):
    return c["T"] * c["H"] * c["W"]


def _is_curve(c):
    return c["bt"] == 1 and c["bh"] == 1


def _extents(c):
    """The grid that the blocks are cut from: the clip's, or its curve-ordered tokens in one line."""
    return (1, 1, _tokens(c)) if _is_curve(c) else (c["T"], c["H"], c["W"])


def _blocks(c):
    T, H, W = _extents(c)
    return -(-T // c["bt"]) * -(-H // c["bh"]) * -(-W // c["bw"])


def _tiling(c):
    return fva.Tiling(*_extents(c), c["bt"], c["bh"], c["bw"])


# ---- inputs -----------------------------------------------------------------


def _axis(S, b, dims, dev):
    lam = 2.0 * b * (max(S, b) / b) ** (torch.arange(dims // 2, device=dev, dtype=torch.float64) / (dims // 2 - 1))
    ang = 2.0 * math.pi * torch.arange(S, device=dev, dtype=torch.float64)[:, None] / lam
    return torch.stack((torch.cos(ang), torch.sin(ang)), dim=2).reshape(S, dims)


def _embedding(c, dev):
    """[tokens, 128] sinusoidal embedding of (t, y, x), every row of norm sqrt(128)."""
    T, H, W = c["T"], c["H"], c["W"]
    e = torch.empty((T, H, W, HEAD_DIM), device=dev, dtype=torch.float64)
    e[..., :32] = _axis(T, 2, 32, dev)[:, None, None]
    e[..., 32:80] = _axis(H, 8, 48, dev)[None, :, None]
    e[..., 80:] = _axis(W, 8, 48, dev)[None, None]
    return (math.sqrt(2.0) * e).reshape(-1, HEAD_DIM).float()


def _alphas(c, rng):
    """Position weights of the heads: spread evenly over the logarithm of [0.5, 4] in a random order (so that every
    seed keeps about the same share of blocks), or one head in five at 0.3 and the others at 5."""
    n = c["batch"] * c["heads"]
    if c["alphas"] == "stress":
        return np.where(np.arange(n) < max(1, n // 5), 0.3, 5.0)
    return rng.permutation(0.5 * 8.0 ** ((np.arange(n) + rng.uniform(0.25, 0.75, n)) / n))


def _empty(c, dev):
    B, H, N = c["batch"], c["heads"], _tokens(c)
    if c["layout"] == "bnhd":
        return torch.empty((B, N, H, HEAD_DIM), dtype=torch.bfloat16, device=dev).transpose(1, 2)
    return torch.empty((B, H, N, HEAD_DIM), dtype=torch.bfloat16, device=dev)


def _inputs(c, seed, which):
    """The tensors named in `which` ("q", "k", "v"), [batch, heads, tokens, 128] bf16 in the case's layout."""
    dev = torch.device("cuda", torch.cuda.current_device())
    gen = torch.Generator(device=dev).manual_seed(seed)
    alphas = _alphas(c, np.random.default_rng([seed, 100]))
    N = _tokens(c)
    emb = _embedding(c, dev) if "q" in which else None
    if emb is not None and _is_curve(c):
        emb = emb[torch.from_numpy(_curve(c["T"], c["H"], c["W"])).to(dev)]
    out = {n: _empty(c, dev) for n in which}
    for b in range(c["batch"]):
        for h in range(c["heads"]):
            w = math.sqrt(GAMMA2 * float(alphas[b * c["heads"] + h]))
            for n in which:
                x = torch.randn((N, HEAD_DIM), generator=gen, device=dev)
                if n != "v":
                    x += w * emb
                out[n][b, h] = x
    return out


def _curve(T, H, W):
    """Raster ids of the grid's tokens along J. Skilling's 3D Hilbert curve, axes (t, y, x), in numpy."""
    bits = max(0, (max(T, H, W) - 1).bit_length())
    X = [a.reshape(-1).astype(np.int64) for a in np.meshgrid(np.arange(T), np.arange(H), np.arange(W), indexing="ij")]
    for q in (1 << b for b in range(bits - 1, 0, -1)):
        for i in range(3):
            up = (X[i] & q) != 0
            swap = np.where(up, 0, (X[0] ^ X[i]) & (q - 1))
            X[0] = X[0] ^ np.where(up, q - 1, swap)
            if i:
                X[i] = X[i] ^ swap
    X[1] = X[1] ^ X[0]
    X[2] = X[2] ^ X[1]
    fix = np.zeros_like(X[0])
    for q in (1 << b for b in range(bits - 1, 0, -1)):
        fix ^= np.where((X[2] & q) != 0, q - 1, 0)
    X = [a ^ fix for a in X]
    key = np.zeros_like(X[0])
    for b in range(bits - 1, -1, -1):
        for a in X:
            key = (key << 1) | ((a >> b) & 1)
    return np.argsort(key, kind="stable")


# ---- prepare and run --------------------------------------------------------


def prepare(case, seed):
    c, kind = case, case["kind"]
    dev = torch.device("cuda", torch.cuda.current_device())
    s = dict(kind=kind, p=c["p"], k_min=c["k_min"])
    u8 = lambda n: torch.empty(max(n, 1), dtype=torch.uint8, device=dev)
    if kind == "curve_layout":
        s["grid"] = (c["T"], c["H"], c["W"])
        s["perm"] = torch.zeros(_tokens(c), dtype=torch.int32, device=dev)
        s["ws"] = u8(fva.fva_curve_workspace_size(*s["grid"]))
        s.update(_inputs(c, seed, "qkv"))
        s["there"] = {n: _empty(c, dev) for n in "qkv"}
        return s
    if kind == "permute":
        s.update(_inputs(c, seed, "v"))
        s["perm"] = torch.from_numpy(_curve(c["T"], c["H"], c["W"]).astype(np.int32)).to(dev)
        s["there"], s["back"] = _empty(c, dev), _empty(c, dev)
        return s
    B, H, nb = c["batch"], c["heads"], _blocks(c)
    s["tiling"] = _tiling(c)
    s.update(_inputs(c, seed, {"quantize": "v", "route": "qk", "sasa": "qk"}.get(kind, "qkv")))
    desc = fva._desc_of(s["v"] if kind == "quantize" else s["q"])
    if c["v"] == "e4m3":
        s["v8"] = (torch.empty((B, H, nb, 128, 128), dtype=torch.uint8, device=dev),
                   torch.empty((B, H, 128), dtype=torch.int32, device=dev))
        s["ws_v"] = u8(fva.fva_quantize_v_workspace_size(desc, s["tiling"]))
    if kind == "quantize":
        return s
    # the kept lists are filled up to the row's count: the rest of a row stays as it is here
    s["lists"] = (torch.zeros((B, H, nb, nb), dtype=torch.uint8, device=dev),
                  torch.zeros((B, H, nb), dtype=torch.int32, device=dev),
                  torch.zeros((B, H, nb, nb), dtype=torch.int32, device=dev))
    if kind == "sasa":
        heads = torch.arange(B * H, device=dev, dtype=torch.int64)
        s["ranks"] = c["ranks"]
        s["rank_of"] = (heads * c["ranks"] // (B * H)).to(torch.int32)
        s["extra"] = torch.zeros(c["ranks"], dtype=torch.int32, device=dev)
        s["ws_r"] = u8(fva.fva_route_sasa_workspace_size(desc, s["tiling"]))
        return s
    s["ws_r"] = u8(fva.fva_route_workspace_size(desc, s["tiling"]))
    if kind == "route":
        return s
    s["out"] = _empty(c, dev)
    if kind != "noalloc":
        s["ws_a"] = u8(fva.fva_attn_workspace_size(desc, s["tiling"]))
    if kind in ("attn", "noalloc"):
        fva.fva_route(s["q"], s["k"], s["p"], s["k_min"], s["tiling"], out=s["lists"], workspace=s["ws_r"])
        if c["v"] == "e4m3":
            fva.fva_quantize_v(s["v"], s["tiling"], out=s["v8"], workspace=s["ws_v"])
    return s


def run(s):
    kind = s["kind"]
    if kind == "curve_layout":
        perm = fva.fva_curve_order(*s["grid"], out=s["perm"], workspace=s["ws"])
        out = {n: fva.fva_permute_tokens(s[n], perm, fva.FVA_TO_CURVE, out=s["there"][n]) for n in "qkv"}
        return {"perm": perm, **out}
    if kind == "permute":
        fva.fva_permute_tokens(s["v"], s["perm"], fva.FVA_TO_CURVE, out=s["there"])
        fva.fva_permute_tokens(s["there"], s["perm"], fva.FVA_FROM_CURVE, out=s["back"])
        return {"there": s["there"], "back": s["back"]}
    if kind == "quantize":
        v8, vexp = fva.fva_quantize_v(s["v"], s["tiling"], out=s["v8"], workspace=s["ws_v"])
        return {"v8": v8, "v_exp": vexp}
    if kind == "sasa":
        mask, counts, kv, extra = fva.fva_route_sasa(
            s["q"], s["k"], s["p"], s["k_min"], s["tiling"], s["rank_of"], s["ranks"], out=s["lists"],
            rank_extra=s["extra"], workspace=s["ws_r"])
        return {"mask": mask, "counts": counts, "kv_idx": kv, "extra": extra}
    out = {}
    mask, counts, kv = s["lists"]
    if kind in ("step", "route"):
        if kind == "step" and "v8" in s:
            fva.fva_quantize_v(s["v"], s["tiling"], out=s["v8"], workspace=s["ws_v"])
        fva.fva_route(s["q"], s["k"], s["p"], s["k_min"], s["tiling"], out=s["lists"], workspace=s["ws_r"])
        out.update(mask=mask, counts=counts, kv_idx=kv)
        if kind == "route":
            return out
    if kind == "noalloc":
        fva.fva_attn_noalloc(s["q"], s["k"], s["v"], s["tiling"], counts, kv, s["out"])
    elif "v8" in s:
        fva.fva_attn_fp8v(s["q"], s["k"], *s["v8"], s["tiling"], mask, counts, kv, out=s["out"], workspace=s["ws_a"])
    else:
        fva.fva_attn(s["q"], s["k"], s["v"], s["tiling"], mask, counts, kv, out=s["out"], workspace=s["ws_a"])
    out["o"] = s["out"]
    return out


# ---- what a pass cannot do without ------------------------------------------


def work(case):
    """Bytes: inputs read once, outputs written once. Operations: the products of the real tokens of the kept blocks,
    with the share of blocks that these inputs keep on average (by p, measured), and the block scores."""
    c, kind = case, case["kind"]
    BH, N, nb = c["batch"] * c["heads"], _tokens(c), _blocks(c)
    tensor = BH * N * HEAD_DIM * 2
    keep = {0.8: 0.33, 0.9: 0.46, 0.95: 0.58}[c["p"]] if c["alphas"] == "spread" else 0.2
    lists = BH * nb * nb * 1 + BH * nb * 4 + int(BH * nb * nb * keep) * 4
    if kind == "curve_layout":
        return {"bytes": 6 * tensor + 4 * N, "flops": 0}
    if kind == "permute":
        return {"bytes": 4 * tensor + 2 * 4 * N, "flops": 0}
    v8 = BH * nb * 16384 + BH * 512
    if kind == "quantize":
        return {"bytes": tensor + v8, "flops": 0}
    scores = 2 * BH * nb * nb * HEAD_DIM
    if kind in ("route", "sasa"):
        return {"bytes": 2 * tensor + lists, "flops": scores}
    attend = int(4 * BH * N * N * HEAD_DIM * keep)
    if kind == "step":
        return {"bytes": 4 * tensor + lists, "flops": scores + attend}
    kv = int(BH * nb * nb * keep) * 4 + BH * nb * 4
    return {"bytes": (v8 if c["v"] == "e4m3" else tensor) + 3 * tensor + kv, "flops": attend}


def tolerance(case):
    """Masks, counts, lists, codes and orders are whole numbers and equal; the attention's output is compared by
    what the bf16 rounding of the probabilities and the result give (E4M3 probabilities: 3 bits of fraction)."""
    if case["kind"] in ("step", "attn", "noalloc"):
        return {"rel": 0.03 if case["v"] == "e4m3" else 0.01, "max": 0.5 if case["v"] == "e4m3" else 0.1}
    return "exact"


# ---- the same in 64 bits ----------------------------------------------------


def _block_tokens(c, dev):
    """[blocks, volume] token ids in local raster order (-1: padding)."""
    T, H, W = _extents(c)
    ids = torch.arange(T * H * W, device=dev).reshape(T, H, W)
    bt, bh, bw = c["bt"], c["bh"], c["bw"]
    pad = torch.full((-(-T // bt) * bt, -(-H // bh) * bh, -(-W // bw) * bw), -1, device=dev, dtype=torch.int64)
    pad[:T, :H, :W] = ids
    blocks = pad.reshape(pad.shape[0] // bt, bt, pad.shape[1] // bh, bh, pad.shape[2] // bw, bw)
    blocks = blocks.permute(0, 2, 4, 1, 3, 5).reshape(-1, bt * bh * bw)
    # the real tokens of a block come first
    order = torch.argsort((blocks < 0).to(torch.int8), dim=1, stable=True)
    return torch.gather(blocks, 1, order)


def _lists_of(mask, counts):
    """Ascending kept ids of every row, zeros behind them."""
    nb = mask.shape[-1]
    ids = torch.arange(nb, device=mask.device)
    key = torch.where(mask.bool(), ids, ids + nb)
    kv = torch.sort(key, dim=-1).values
    return torch.where(ids < counts[..., None], kv, 0).to(torch.int32)


def _route64(c, q, k, tok):
    B, H, nb = c["batch"], c["heads"], tok.shape[0]
    real = (tok >= 0).double()[..., None]
    n = real.sum(1)
    mask = torch.empty((B, H, nb, nb), dtype=torch.uint8, device=q.device)
    counts = torch.empty((B, H, nb), dtype=torch.int32, device=q.device)
    order = torch.empty((B, H, nb, nb), dtype=torch.int64, device=q.device)
    for b in range(B):
        for h in range(H):
            qm = (q[b, h].double()[tok.clamp(min=0)] * real).sum(1) / n
            km = (k[b, h].double()[tok.clamp(min=0)] * real).sum(1) / n
            s = qm @ km.T / math.sqrt(HEAD_DIM)
            s, idx = torch.sort(s, dim=1, descending=True, stable=True)
            cum = torch.softmax(s, dim=1).cumsum(1)
            m = (cum < c["p"]).sum(1) + 1
            m = torch.clamp(torch.clamp(m, max=nb), min=min(c["k_min"], nb))
            order[b, h] = idx
            counts[b, h] = m.to(torch.int32)
    _fill(mask, order, counts)
    return mask, counts, order


def _fill(mask, order, counts):
    ids = torch.arange(mask.shape[-1], device=mask.device)
    mask.scatter_(-1, order, (ids < counts[..., None]).to(torch.uint8))


def _augment64(c, counts, order):
    """Slack-aware augmentation of contiguous ranks: (mask, counts, extra blocks of each rank)."""
    n1, n2 = 0.8, 0.07
    B, H, nb = counts.shape
    rank = np.arange(B * H) * c["ranks"] // (B * H)
    load = counts.reshape(B * H, nb).long().sum(1).cpu().numpy()
    total = np.array([load[rank == r].sum() for r in range(c["ranks"])])
    extra = np.zeros(c["ranks"], np.int64)
    for r in range(c["ranks"]):
        slack = int(total.max() - total[r])
        heads = int((rank == r).sum())
        if heads and slack > n2 * total.max():
            extra[r] = math.floor((n1 * slack) / (nb * heads))
    more = torch.from_numpy(extra[rank]).to(counts.device).reshape(B, H, 1)
    counts = torch.clamp(counts + more, max=nb).to(torch.int32)
    mask = torch.empty(order.shape, dtype=torch.uint8, device=counts.device)
    _fill(mask, order, counts)
    return mask, counts, torch.from_numpy(extra.astype(np.int32))


def _quantize64(c, v, tok):
    """E4M3 tiles in the library's documented order and the channels' exponents."""
    B, H, nb = c["batch"], c["heads"], tok.shape[0]
    amax = v.abs().amax(dim=2).double()
    e = torch.clamp(torch.ceil(torch.log2(amax / 448.0)), min=-127)
    e = torch.where(amax * 2.0 ** -(e - 1) <= 448.0, e - 1, e)
    e = torch.where(amax * 2.0 ** -e > 448.0, e + 1, e)
    e = torch.where(amax == 0, torch.full_like(e, -127.0), torch.clamp(e, min=-127))
    pos = torch.arange(128, device=v.device)
    g, hb, t, r = pos // 32, pos // 16 % 2, pos // 4 % 4, pos % 4
    kap = 64 * hb + 32 * (t // 2) + 8 * g + 4 * (t % 2) + r
    full = torch.full((nb, 128), -1, device=v.device, dtype=torch.int64)
    full[:, : tok.shape[1]] = tok
    src = full[:, kap]
    v8 = torch.empty((B, H, nb, 128, 128), dtype=torch.uint8, device=v.device)
    for b in range(B):
        for h in range(H):
            x = (v[b, h].double() * 2.0 ** -e[b, h]).float().to(torch.float8_e4m3fn).view(torch.uint8)
            y = torch.where((src >= 0)[..., None], x[src.clamp(min=0)], 0)
            v8[b, h] = y.transpose(1, 2)
    return v8, e.to(torch.int32)


def _attend64(c, q, k, v, mask, tok):
    B, H, nb = c["batch"], c["heads"], tok.shape[0]
    vol = tok.shape[1]
    flat = tok.reshape(-1)
    real = flat >= 0
    o = torch.zeros(q.shape, dtype=torch.float64, device=q.device)
    step = max(1, (1 << 27) // (vol * vol * nb))  # query blocks at a time: at most 1 GB of scores
    for b in range(B):
        for h in range(H):
            kb = k[b, h].double()[flat.clamp(min=0)].T.contiguous()
            vb = v[b, h].double()[flat.clamp(min=0)]
            for i in range(0, nb, step):
                rows = tok[i : i + step].reshape(-1)
                s = q[b, h].double()[rows.clamp(min=0)] @ kb / math.sqrt(HEAD_DIM)
                keep = mask[b, h, i : i + step].bool().repeat_interleave(vol, 0).repeat_interleave(vol, 1) & real
                w = torch.softmax(s.masked_fill_(~keep, -math.inf), dim=1)
                o[b, h][rows[rows >= 0]] = (w @ vb)[rows >= 0]
    return o


def exact(case, seed):
    c, kind = case, case["kind"]
    dev = torch.device("cuda", torch.cuda.current_device())
    # the full 720p and longer attentions take too long here in 64 bits
    small = c["batch"] * c["heads"] * _tokens(c) ** 2 <= 6e10
    if kind in ("attn", "noalloc") and not small:
        return None
    if kind == "permute":
        v = _inputs(c, seed, "v")["v"]
        return {"there": v[:, :, torch.from_numpy(_curve(c["T"], c["H"], c["W"])).to(dev)], "back": v}
    if kind == "curve_layout":
        perm = torch.from_numpy(_curve(c["T"], c["H"], c["W"]))
        x = _inputs(c, seed, "qkv")
        return {"perm": perm.to(torch.int32), **{n: x[n][:, :, perm.to(dev)] for n in "qkv"}}
    tok = _block_tokens(c, dev)
    x = _inputs(c, seed, {"quantize": "v", "route": "qk", "sasa": "qk"}.get(kind, "qkv"))
    if kind == "quantize":
        v8, vexp = _quantize64(c, x["v"], tok)
        return {"v8": v8, "v_exp": vexp}
    mask, counts, order = _route64(c, x["q"], x["k"], tok)
    if kind == "sasa":
        mask, counts, extra = _augment64(c, counts, order)
        return {"mask": mask, "counts": counts, "kv_idx": _lists_of(mask, counts), "extra": extra}
    out = {}
    if kind in ("step", "route"):
        out = {"mask": mask, "counts": counts, "kv_idx": _lists_of(mask, counts)}
    if kind != "route":
        out["o"] = _attend64(c, x["q"], x["k"], x["v"], mask, tok) if small else None
    return out

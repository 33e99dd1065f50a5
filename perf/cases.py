"""The calls whose time counts, from the smallest layer to the largest: each
case is one pass through the package's public entry points on inputs that a
diffusion transformer (or its VAE) would hand over.

Kinds:
  layer  the top-k or head-shared gate and attention of one layer
         (ssba.forward_topk), a static gate (ssba.build_index + ssba.forward)
         or the dense control (ssba.forward_dense)
  rope   Algorithm 1 with its rotary step (ssba.forward_topk_rope)
  stack  a stack of layers in one call (ssba.forward_layers)
  train  gate, training forward and backward of one layer
  haar   the VAE's multi-level Haar transform and its inverse

Layout "bhtd" is the contiguous [B, H, T, D] tensor, "bthd" the view of a
projection's [B, T, H, D] output that a transformer block passes without a
copy.
"""
import math

import torch

from paper_2605_15684_amd import haar, ssba
from paper_2605_15684_amd.inputs import LAYER_KEEP_SCHEDULE_24

_DT = {"bf16": torch.bfloat16, "f32": torch.float32}
_BYTES = {"bf16": 2, "f32": 4}


def _layer(name, batch, heads, gh, gw, tile, d, keep, text=0, dtype="bf16", gate="topk", layout="bhtd",
           kind="layer", heavy=0, win=1, layers=0):
    c = dict(kind=kind, batch=batch, heads=heads, gh=gh, gw=gw, tile=tile, d=d, keep=keep, text=text, dtype=dtype,
             gate=gate, layout=layout, heavy=heavy, win=win, layers=layers)
    if name:
        c["name"] = name
    return c


def _haar(name, n, c, h, w, levels, dtype, residuals):
    r = dict(kind="haar", n=n, c=c, h=h, w=w, levels=levels, dtype=dtype, residuals=residuals)
    if name:
        r["name"] = name
    return r


def listed():
    return [
        # The smallest call: a 16x16-token grid in full precision (launches count).
        _layer("tiny_f32", 1, 2, 16, 16, 4, 64, 4, dtype="f32"),
        # A 512-pixel image with a 77-token prompt, as the QKV projection leaves it.
        _layer("grid32_text77", 1, 16, 32, 32, 8, 64, 4, text=77, layout="bthd"),
        # The headline: a 1024-pixel image, 84.375 % of the blocks masked.
        _layer("grid64", 1, 16, 64, 64, 8, 64, 10),
        # The same with 256 text tokens, a batch of two and 24 heads.
        _layer("grid64_text256", 2, 24, 64, 64, 8, 64, 10, text=256, layout="bthd"),
        # The same layer in full precision (checking a model, sensitive layers).
        _layer("grid64_f32", 1, 16, 64, 64, 8, 64, 10, dtype="f32"),
        # A 2048-pixel image at head_dim 128, coarse 16x16 blocks, rho 0.9, 1 % heavy keys.
        _layer("grid128_tile16", 1, 16, 128, 128, 16, 128, 7, heavy=164),
        # A 2048-pixel image in the paper's own 8x8 blocks: 256 blocks a head.
        _layer("grid128_tile8", 1, 16, 128, 128, 8, 64, 40),
        # An odd aspect ratio in fine 4x4 blocks (345 of them) with a prompt.
        _layer("grid60x92_tile4", 1, 12, 60, 92, 4, 64, 54, text=77),
        # Algorithm 1 in full: rotary step, gate, attention.
        _layer("rope_grid64", 1, 16, 64, 64, 8, 64, 10, kind="rope"),
        # The 24-layer stack with the layer-aware schedule, one call.
        _layer("stack24", 1, 16, 64, 64, 8, 64, 10, kind="stack", layers=24),
        # One layer of a training step at head_dim 128 with text: gate, forward, backward.
        _layer("train_grid64_d128", 2, 16, 64, 64, 8, 128, 16, text=77, kind="train"),
        # The VAE's transform of a batch of feature maps and its inverse.
        _haar("haar_512", 4, 128, 512, 512, 3, "bf16", True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cost(c):
    w = work(c)
    # fp32 products run at a fraction of the bf16 rate
    return w["bytes"] + w["flops"] / (8 if c["dtype"] == "f32" and c["kind"] != "haar" else 50)


def draw(rng):
    """A case of the listed ranges: every kind, odd block counts, ragged text, both layouts and dtypes."""
    most = max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(["layer", "layer", "layer", "layer", "fine", "fine", "f32", "f32", "rope", "stack", "train",
                           "train", "haar"])
        if kind == "haar":
            levels = rng.randint(1, 3)
            c = _haar("", rng.randint(1, 4), _log_int(rng, 3, 160), (1 << levels) * _log_int(rng, 4, 600 >> levels),
                      8 * _log_int(rng, 2, 72), levels, rng.choice(["bf16", "bf16", "f32"]), rng.random() < 0.5)
        else:
            tile = rng.choice([8, 8, 16])
            most_tb = 64
            if kind == "fine":      # more blocks than one wave ranks, or 4x4 blocks
                tile = rng.choice([4, 8, 8])
                most_tb = 600
            elif kind == "f32":
                tile = rng.choice([4, 8, 8, 16])
                most_tb = 300
            ny, nx = rng.randint(2, 24), rng.randint(2, 24)
            tb = ny * nx
            if tb > most_tb or (kind == "fine" and tile == 8 and tb <= 64) or (kind == "f32" and tile == 16 and tb > 64):
                continue
            keep = min(tb, max(1, int(round(tb * rng.choice([1.0, 0.5, 0.25, 0.15625, 0.15625, 0.1])))))
            gate = rng.choice(["topk", "topk", "topk", "topk", "topk_shared", "window", "full"])
            if kind in ("rope", "train"):
                gate = "topk"
            if kind == "stack" and gate == "full":
                gate = "topk"
            win = rng.choice([w for w in (1, 2, 3, 4) if ny % w == 0 and nx % w == 0])
            c = _layer("", rng.choice([1, 1, 2, 4]), _log_int(rng, 1, 24), ny * tile, nx * tile, tile,
                       rng.choice([64, 64, 128]), keep, text=rng.choice([0, 0, rng.randint(1, 300)]),
                       dtype="f32" if kind == "f32" else "bf16", gate=gate, layout=rng.choice(["bhtd", "bthd"]),
                       kind="layer" if kind in ("fine", "f32") else kind, win=win,
                       layers=rng.randint(2, 24) if kind == "stack" else 0)
            if kind == "rope":
                c["tile"], c["gh"], c["gw"] = 8, 8 * ny, 8 * nx
            if c["text"] + c["gh"] * c["gw"] < 64:
                continue
        if _cost(c) <= most:
            return c


# ---------------------------------------------------------------------------
# Inputs and passes
# ---------------------------------------------------------------------------
def _randn(c, gen):
    """[B, H, T, D] of the case's dtype and layout, unit variance (normalised queries and keys)."""
    t = c["text"] + c["gh"] * c["gw"]
    shape = (c["batch"], t, c["heads"], c["d"]) if c["layout"] == "bthd" else (c["batch"], c["heads"], t, c["d"])
    x = torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).to(_DT[c["dtype"]])
    return x.transpose(1, 2) if c["layout"] == "bthd" else x


def _qkv(c, gen):
    q, k, v = (_randn(c, gen) for _ in range(3))
    if c["heavy"]:   # a few keys of large norm, the same rows in every head
        rows = torch.randperm(c["gh"] * c["gw"], generator=gen, device="cuda")[: c["heavy"]] + c["text"]
        k[:, :, rows] *= 4.0
    return q, k, v


def _shift(c):
    return (c["tile"] // 2, c["tile"] // 2)


def _inputs(c, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    if c["kind"] == "haar":
        dt, shape = _DT[c["dtype"]], (c["n"], c["c"], c["h"], c["w"])
        mk = lambda s, dev: torch.randn(s, generator=gen, device="cuda").mul_(dev).to(dt)  # noqa: E731
        x = mk(shape, 1.0)
        lv = [mk(haar.level_shape(shape, l), 1.0) for l in range(1, c["levels"] + 1)]
        res = [mk((c["n"], c["c"], c["h"] >> l, c["w"] >> l), 0.25) for l in range(c["levels"])] \
            if c["residuals"] else None
        return x, lv, res
    if c["kind"] == "stack":
        return [_qkv(c, gen) for _ in range(c["layers"])]
    q, k, v = _qkv(c, gen)
    if c["kind"] == "train":
        return q, k, v, _randn(c, gen)
    return q, k, v


def _keeps(c):
    """The stack's kept blocks per layer: the layer-aware schedule, scaled to the case's share."""
    tb = (c["gh"] // c["tile"]) * (c["gw"] // c["tile"])
    return [max(1, min(tb, round(LAYER_KEEP_SCHEDULE_24[l % 24] * c["keep"] / 10))) for l in range(c["layers"])]


def prepare(case, seed):
    """Inputs, descriptor and the workspaces and outputs that a program keeps."""
    c = case
    s = {"case": c}
    if c["kind"] == "haar":
        s["x"], s["levels"], s["res"] = _inputs(c, seed)
        s["out"] = [torch.empty_like(t) for t in s["levels"]]
        s["y"] = torch.empty_like(s["x"])
        return s
    ins = _inputs(c, seed)
    q = ins[0][0] if c["kind"] == "stack" else ins[0]
    gate = "dense" if c["gate"] == "full" else c["gate"]
    desc = ssba.desc_for(q, grid=(c["gh"], c["gw"]), tile=c["tile"], shift=_shift(c), n_text=c["text"], gate=gate,
                         keep=c["keep"] if gate in ("topk", "topk_shared") else 0, window=(c["win"], c["win"]))
    s["desc"] = desc
    like = lambda: torch.empty_strided(q.shape, q.stride(), dtype=q.dtype, device=q.device)  # noqa: E731
    if c["kind"] == "stack":
        s["layers"] = [dict(q=a, k=b, v=v, out=like(), keep=kp) for (a, b, v), kp in zip(ins, _keeps(c))]
        s["index"], s["scratch"] = ssba.forward_layers(s["layers"], desc)
        return s
    s["qkv"] = ins[:3]
    s["out"] = like()
    s["index"], s["scratch"] = ssba.alloc_workspace(desc, q.device)
    if c["kind"] == "rope":
        s["rope"] = (like(), like())
    if c["kind"] == "train":
        s["dout"] = ins[3]
        s["grads"] = (like(), like(), like())
        s["lse"] = torch.empty(q.shape[:3], dtype=torch.float32, device=q.device)
    return s


def run(state):
    s, c = state, state["case"]
    if c["kind"] == "haar":
        levels = haar.dwt(s["x"], c["levels"], out=s["out"])
        y = haar.iwt(s["levels"], s["res"], out=s["y"])
        return {"levels": levels, "y": y}
    desc = s["desc"]
    if c["kind"] == "stack":
        ssba.forward_layers(s["layers"], desc, index=s["index"], scratch=s["scratch"])
        return {"outs": [x["out"] for x in s["layers"]], **({"index": s["index"]} if c["gate"] != "window" else {})}
    q, k, v = s["qkv"]
    if c["kind"] == "rope":
        qr, kr, index, _, out = ssba.forward_topk_rope(q, k, v, desc, q_rope=s["rope"][0], k_rope=s["rope"][1],
                                                       index=s["index"], scratch=s["scratch"], out=s["out"])
        return {"q_rope": qr, "k_rope": kr, "index": index, "out": out}
    if c["kind"] == "train":
        index, _ = ssba.build_index(q, k, desc, index=s["index"], scratch=s["scratch"])
        out, lse = ssba.forward_train(q, k, v, index, desc, out=s["out"], lse=s["lse"])
        dq, dk, dv = ssba.backward(q, k, v, out, s["dout"], lse, index, desc, *s["grads"])
        return {"index": index, "out": out, "lse": lse, "dq": dq, "dk": dk, "dv": dv}
    if c["gate"] == "full":
        return {"out": ssba.forward_dense(q, k, v, desc, out=s["out"])}
    if c["gate"] in ("topk", "topk_shared"):
        index, _, out = ssba.forward_topk(q, k, v, desc, index=s["index"], scratch=s["scratch"], out=s["out"])
    else:
        index, _ = ssba.build_index(q, k, desc, index=s["index"], scratch=s["scratch"])
        out = ssba.forward(q, k, v, index, desc, out=s["out"])
    return {"index": index, "out": out}


# ---------------------------------------------------------------------------
# What a pass cannot do without, and how far another correct one may be off
# ---------------------------------------------------------------------------
def work(case):
    c, eb = case, _BYTES[case["dtype"]]
    if c["kind"] == "haar":
        n = c["n"] * c["c"] * c["h"] * c["w"]
        pyramid = sum(4.0 ** -l for l in range(c["levels"]))              # every level's four bands
        details = sum(0.75 * 4.0 ** -l for l in range(c["levels"])) + 0.25 * 4.0 ** -(c["levels"] - 1)
        res = sum(4.0 ** -l for l in range(c["levels"])) if c["residuals"] else 0.0
        return {"bytes": eb * n * ((1 + pyramid) + (details + res + 1)), "flops": n * 4.0 * pyramid}
    t_img = c["gh"] * c["gw"]
    tb, t = t_img // c["tile"] ** 2, t_img + c["text"]
    bh = c["batch"] * c["heads"]
    rows = bh * t * c["d"] * eb
    index = 4 * bh * tb * (tb + 1)

    def pairs(keep):
        return bh * (t_img * (keep * c["tile"] ** 2 + c["text"]) + c["text"] * t)

    if c["kind"] == "stack":
        keeps = _keeps(c) if c["gate"] != "window" else [c["win"] ** 2] * c["layers"]
        n_index = c["layers"] if c["gate"] != "window" else min(2, c["layers"])
        return {"bytes": c["layers"] * 4 * rows + n_index * index, "flops": 4.0 * c["d"] * sum(map(pairs, keeps))}
    if c["gate"] == "full":
        return {"bytes": 4 * rows, "flops": 4.0 * c["d"] * bh * t * t}
    n = pairs(c["win"] ** 2 if c["gate"] == "window" else c["keep"])
    if c["kind"] == "train":   # forward: q k v -> o lse; backward: q k v o do lse -> dq dk dv
        return {"bytes": 12 * rows + 2 * 4 * bh * t + index, "flops": 14.0 * c["d"] * n}
    return {"bytes": (6 if c["kind"] == "rope" else 4) * rows + index, "flops": 4.0 * c["d"] * n}


def tolerance(case):
    # about four times what the first kernels show against exact()
    if case["kind"] == "haar":
        return {"rel": 7e-3, "max": 2e-2} if case["dtype"] == "bf16" else {"rel": 3e-7, "max": 2e-6}
    if case["dtype"] == "f32":
        return {"rel": 3e-6, "max": 3e-5}
    return {"rel": 1.2e-2, "max": 2e-1}


# ---------------------------------------------------------------------------
# The same in 64 bits
# ---------------------------------------------------------------------------
def _rows(c, shift):
    """Sequence rows of every block's slots in the shifted frame, [T_b, tile^2]."""
    b = c["tile"]
    y = (torch.arange(c["gh"], device="cuda") - shift[0]) % c["gh"]
    x = (torch.arange(c["gw"], device="cuda") - shift[1]) % c["gw"]
    grid = c["text"] + y[:, None] * c["gw"] + x[None, :]
    ny, nx = c["gh"] // b, c["gw"] // b
    return grid.reshape(ny, b, nx, b).permute(0, 2, 1, 3).reshape(ny * nx, b * b)


def _kept(c, q, k, rows, keep):
    """Kept block ids, ascending, [B, H, T_b, count]."""
    tb = rows.shape[0]
    if c["gate"] == "window":
        ny, nx, w = c["gh"] // c["tile"], c["gw"] // c["tile"], c["win"]
        iy, ix = (torch.arange(tb, device="cuda") // nx), (torch.arange(tb, device="cuda") % nx)
        same = (iy[:, None] // w == iy // w) & (ix[:, None] // w == ix // w)
        ids = same.nonzero()[:, 1].reshape(tb, w * w)
        return ids.expand(c["batch"], c["heads"], tb, w * w)
    qb, kb = q[:, :, rows].sum(3), k[:, :, rows].sum(3)
    s = torch.matmul(qb, kb.transpose(2, 3).contiguous())
    if c["gate"] == "topk_shared":
        s = s.sum(1, keepdim=True)
    ids = torch.sort(s, dim=-1, descending=True, stable=True).indices[..., :keep].sort(-1).values
    return ids.expand(c["batch"], c["heads"], tb, keep)


def _index(kept, tb):
    b, h, _, n = kept.shape
    out = torch.full((b, h, tb, tb + 1), -1, dtype=torch.int32, device="cuda")
    out[..., 0] = n
    out[..., 1:1 + n] = kept.to(torch.int32)
    return out


def _attend(c, q, k, v, rows, kept, dout=None):
    """out, lse (natural log) and, given dout, the gradients, of [B, H, T, D] doubles."""
    scale, d, nt = 1.0 / math.sqrt(c["d"]), c["d"], c["text"]
    out, lse = torch.zeros_like(q), torch.zeros(q.shape[:3], dtype=q.dtype, device=q.device)
    grads = [torch.zeros_like(q) for _ in range(3)] if dout is not None else None
    text = torch.arange(nt, device="cuda")

    def part(qh, kh, vh, qr, kr, at):
        # query rows qr [n, m] against key rows kr [n, l]
        kk, vv = kh[kr], vh[kr]
        s = torch.matmul(qh[qr], kk.transpose(1, 2).contiguous()) * scale
        ls = torch.logsumexp(s, -1)
        p = torch.exp(s - ls[..., None])
        out[at][qr.reshape(-1)] = torch.matmul(p, vv).reshape(-1, d)
        lse[at][qr.reshape(-1)] = ls.reshape(-1)
        if dout is None:
            return
        g = dout[at][qr]
        dp = torch.matmul(g, vv.transpose(1, 2).contiguous())
        ds = p * (dp - (p * dp).sum(-1, keepdim=True)) * scale
        grads[0][at][qr.reshape(-1)] = torch.matmul(ds, kk).reshape(-1, d)
        pt, dst = p.transpose(1, 2).contiguous(), ds.transpose(1, 2).contiguous()
        grads[1][at].index_add_(0, kr.reshape(-1), torch.matmul(dst, qh[qr]).reshape(-1, d))
        grads[2][at].index_add_(0, kr.reshape(-1), torch.matmul(pt, g).reshape(-1, d))

    t, slots = q.shape[2], rows.shape[1]
    for b in range(q.shape[0]):
        for h in range(q.shape[1]):
            at = (b, h)
            qh, kh, vh = q[at], k[at], v[at]
            if kept is not None:
                n_keys = kept.shape[3] * slots + nt
                step = max(1, int(3e7 // (n_keys * max(slots, d))))
                for i in range(0, rows.shape[0], step):
                    ids = kept[at][i:i + step]
                    kr = torch.cat([rows[ids].reshape(len(ids), -1), text.expand(len(ids), nt)], 1)
                    part(qh, kh, vh, rows[i:i + step], kr, at)
            first = torch.arange(t if kept is None else nt, device="cuda")
            for qr in first.split(2048):
                part(qh, kh, vh, qr[None], torch.arange(t, device="cuda")[None], at)
    return out, lse, grads


def _rotate(c, x):
    """2-D axial rotary embedding of the image rows, theta 10000."""
    d, nt = c["d"], c["text"]
    p = d // 4
    freq = 10000.0 ** (-torch.arange(p, dtype=torch.float64, device="cuda") / p)
    tok = torch.arange(c["gh"] * c["gw"], device="cuda")
    ang = torch.cat([(tok // c["gw"]).double()[:, None] * freq, (tok % c["gw"]).double()[:, None] * freq], 1)
    cs, sn = ang.cos(), ang.sin()
    img = x[:, :, nt:]
    a, b = img[..., 0::2], img[..., 1::2]
    y = x.clone()
    y[:, :, nt:] = torch.stack([a * cs - b * sn, a * sn + b * cs], -1).flatten(-2)
    return y


def _bf16(x):
    """Doubles rounded once to bf16 (nearest even): 45 fraction bits go."""
    b = x.contiguous().view(torch.int64)
    b = (b + 0xFFFFFFFFFFF + ((b >> 45) & 1)) & ~0x1FFFFFFFFFFF
    return b.view(torch.float64)


def _exact_haar(c, seed):
    x, lv, res = _inputs(c, seed)
    levels, ll = [], x.double()
    for _ in range(c["levels"]):
        p, q, u, v = ll[..., 0::2, 0::2], ll[..., 0::2, 1::2], ll[..., 1::2, 0::2], ll[..., 1::2, 1::2]
        bands = torch.stack([p + q + u + v, p - q + u - v, p + q - u - v, p - q - u + v], 2) * 0.5
        ll = bands[:, :, 0]
        levels.append(bands.flatten(1, 2))
    cur = None
    for l in range(c["levels"], 0, -1):
        w = lv[l - 1].double().unflatten(1, (c["c"], 4))
        a = w[:, :, 0] if cur is None else cur
        b, e, f = w[:, :, 1], w[:, :, 2], w[:, :, 3]
        top = torch.stack([a + b + e + f, a - b + e - f], -1).flatten(-2)
        low = torch.stack([a + b - e - f, a - b - e + f], -1).flatten(-2)
        cur = torch.stack([top, low], 3).flatten(2, 3) * 0.5
        if res is not None:
            cur = cur + res[l - 1].double()
    return {"levels": levels, "y": cur}


def exact(case, seed):
    c = case
    if c["kind"] == "haar":
        return _exact_haar(c, seed)
    tb = (c["gh"] // c["tile"]) * (c["gw"] // c["tile"])
    sh = _shift(c)
    ins = _inputs(c, seed)
    if c["kind"] == "stack":
        outs, idx = [], []
        for l, ((q, k, v), keep) in enumerate(zip(ins, _keeps(c))):
            q, k, v = q.double(), k.double(), v.double()
            rows = _rows(c, sh if l % 2 == 0 else (-sh[0], -sh[1]))
            kept = _kept(c, q, k, rows, keep)
            outs.append(_attend(c, q, k, v, rows, kept)[0])
            idx.append(_index(kept, tb))
        return {"outs": outs, **({"index": torch.stack(idx)} if c["gate"] != "window" else {})}
    q, k, v = (x.double() for x in ins[:3])
    rows = _rows(c, sh)
    if c["kind"] == "rope":   # the rotated rows are bf16 by definition; gate and attention take those
        qr, kr = _rotate(c, q), _rotate(c, k)
        q, k = _bf16(qr), _bf16(kr)
        kept = _kept(c, q, k, rows, c["keep"])
        return {"q_rope": qr, "k_rope": kr, "index": _index(kept, tb), "out": _attend(c, q, k, v, rows, kept)[0]}
    if c["gate"] == "full":
        return {"out": _attend(c, q, k, v, rows, None)[0]}
    kept = _kept(c, q, k, rows, c["keep"])
    if c["kind"] == "train":
        out, lse, (dq, dk, dv) = _attend(c, q, k, v, rows, kept, ins[3].double())
        return {"index": _index(kept, tb), "out": out, "lse": lse, "dq": dq, "dk": dk, "dv": dv}
    return {"index": _index(kept, tb), "out": _attend(c, q, k, v, rows, kept)[0]}

"""Cases for timing the library through its Python entry points.

Each case is one piece of the foreground path as a training loop or a sampler
calls it: block-sparse attention (forward alone, forward + backward, packed
samples), the block lists and the Top-K block selection that feed it, token
dropping and write-back around it, and the per-step latent work. Sizes are
those of the workloads in `workloads/` (512, 1K and 2K canvases, 24 heads of
128) and of the tests, and `draw` spreads over the ranges between them.
"""
import math

import torch

import paper_2609_23169_amd as ut

DEV = "cuda"
# retained work of the largest listed case (2K training layer), in FLOP
_MAX_FLOPS = 26.0e12


# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------

def listed():
    return [
        # the smallest training layer of the workloads: launches and host work
        {"name": "train_tiny", "kind": "train", "n": 384, "heads": 2, "dim": 64, "block": 64,
         "keep": 0.4, "workspace": "auto"},
        # one attention layer of a denoising step, 512 canvas
        {"name": "fwd_512", "kind": "fwd", "n": 6552, "heads": 24, "dim": 128, "block": 128, "keep": 0.3},
        # one attention layer of a denoising step, 2K canvas
        {"name": "fwd_2k", "kind": "fwd", "n": 77586, "heads": 24, "dim": 128, "block": 128, "keep": 0.1},
        # one training layer, 1K canvas, workspace allocated by the helper
        {"name": "train_1k", "kind": "train", "n": 22879, "heads": 24, "dim": 128, "block": 128,
         "keep": 0.2, "workspace": "auto"},
        # one training layer, 2K canvas, workspace kept by the training loop
        {"name": "train_2k", "kind": "train", "n": 77060, "heads": 24, "dim": 128, "block": 128,
         "keep": 0.1, "workspace": "kept"},
        # every block kept (the dense comparison) with the minimum workspace
        {"name": "train_dense_min", "kind": "train", "n": 12801, "heads": 24, "dim": 128, "block": 128,
         "keep": 1.0, "workspace": "minimum"},
        # a model with 64-wide heads, finer blocks and a batch of two
        {"name": "train_d64_b64", "kind": "train", "n": 9011, "heads": 16, "dim": 64, "block": 64,
         "keep": 0.2, "batch": 2, "workspace": "auto"},
        # eight samples of a 512-canvas bucket packed into one call
        {"name": "packed_512", "kind": "packed", "samples": 8, "lo": 6011, "hi": 6394, "heads": 24,
         "dim": 128, "block": 128, "keep": 0.3},
        # alpha masks -> token mask -> gather of the hidden state -> write-back, 2K canvas
        {"name": "drop_2k", "kind": "drop", "views": 13, "grid": 128, "hidden": 3072, "fg": 0.37,
         "radius": 1},
        # block selection of one layer at the 2K canvas, 512 text tokens in front
        {"name": "select_2k", "kind": "select", "n": 77060, "heads": 24, "dim": 128, "block": 128,
         "keep": 0.1, "prefix": 4},
        # block lists of one layer at the 2K canvas
        {"name": "index_2k", "kind": "index", "batch": 1, "heads": 24, "nq": 603, "nk": 603, "keep": 0.1},
        # Euler step, loss with gradient and decoding input of the 2K target views
        {"name": "latent_2k", "kind": "latent", "views": 6, "grid": 128, "channels": 64, "fg": 0.37,
         "v": "bf16", "x": "f32"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["fwd", "train", "train", "train", "packed", "drop", "select", "index", "latent"])
    keep = round(math.exp(rng.uniform(math.log(0.05), math.log(1.0))), 3)
    heads = rng.choice([1, 2, 5, 8, 12, 16, 24])
    dim, block = rng.choice([(128, 128), (128, 128), (64, 64), (64, 128), (128, 64)])
    if kind in ("fwd", "train", "select"):
        c = {"kind": kind, "n": _log(rng, 300, 80000), "heads": heads, "dim": dim, "block": block,
             "keep": keep}
        while work(c)["flops"] > _MAX_FLOPS * 0.8:
            c["n"] = int(c["n"] * 0.8)
        if kind == "train":
            c["workspace"] = rng.choice(["auto", "kept", "minimum"])
        if kind == "select":
            c["prefix"] = rng.choice([0, 1, 4]) if c["n"] > 4 * block else 0
        elif c["n"] < 20000:
            c["batch"] = rng.choice([1, 1, 2])
        return c
    if kind == "packed":
        lo = _log(rng, 300, 8000)
        return {"kind": kind, "samples": rng.randint(2, 8), "lo": lo, "hi": int(lo * rng.uniform(1.01, 1.6)) + 1,
                "heads": heads, "dim": dim, "block": block, "keep": max(keep, 0.1)}
    if kind == "drop":
        return {"kind": kind, "views": rng.choice([3, 5, 9, 13]), "grid": _log(rng, 16, 128),
                "hidden": 8 * _log(rng, 64, 384), "fg": round(rng.uniform(0.1, 0.9), 3),
                "radius": rng.choice([0, 1, 2])}
    if kind == "index":
        nq = _log(rng, 6, 1250)
        nk = nq if rng.random() < 0.75 else _log(rng, 6, 1250)
        return {"kind": kind, "batch": rng.choice([1, 1, 2]), "heads": heads, "nq": nq, "nk": nk, "keep": keep}
    return {"kind": "latent", "views": rng.randint(1, 6), "grid": _log(rng, 16, 128),
            "channels": rng.choice([16, 64, 68, 128]), "fg": round(rng.uniform(0.1, 0.9), 3),
            "v": rng.choice(["bf16", "f32"]), "x": rng.choice(["bf16", "f32"])}


# ---------------------------------------------------------------------------
# inputs (plain torch, on the GPU, from the seed alone)
# ---------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 17)
    return g


def _normal(g, *shape):
    return torch.randn(shape, generator=g, device=DEV, dtype=torch.bfloat16)


def _kept_per_row(c, nk):
    """Off-diagonal key blocks of a row, as the paper's floor(rho N_k)."""
    return min(int(math.floor(c["keep"] * nk + 1e-9)), nk - 1)


def _block_mask(g, c, batch, heads, nq, nk):
    """The diagonal plus a fixed number of other key blocks per row."""
    if c["keep"] >= 1.0:
        return torch.ones((batch, heads, nq, nk), dtype=torch.uint8, device=DEV)
    m = torch.zeros((batch, heads, nq, nk), dtype=torch.uint8, device=DEV)
    d = torch.arange(min(nq, nk), device=DEV)
    m[:, :, d, d] = 1
    k = _kept_per_row(c, nk)
    if k > 0:
        r = torch.rand((batch, heads, nq, nk), generator=g, device=DEV)
        r[:, :, d, d] = -1.0
        m.scatter_(3, r.topk(k, dim=3).indices, 1)
    return m


def _attn_inputs(c, seed):
    g = _gen(seed)
    b, n, h, d = c.get("batch", 1), c["n"], c["heads"], c["dim"]
    q, k, v, do = (_normal(g, b, n, h, d) for _ in range(4))
    nb = -(-n // c["block"])
    return q, k, v, do, _block_mask(g, c, b, h, nb, nb)


def _lens(c):
    """Sorted sample lengths between lo and hi, evenly spread."""
    s = c["samples"]
    return [c["lo"] + (c["hi"] - c["lo"]) * i // max(s - 1, 1) for i in range(s)]


def _packed_inputs(c, seed):
    g = _gen(seed)
    lens = _lens(c)
    t, h, d = sum(lens), c["heads"], c["dim"]
    q, k, v, do = (_normal(g, t, h, d) for _ in range(4))
    nb = -(-max(lens) // c["block"])
    m = torch.zeros((len(lens), h, nb, nb), dtype=torch.uint8, device=DEV)
    for i, n in enumerate(lens):
        own = -(-n // c["block"])
        m[i, :, :own, :own] = _block_mask(g, c, 1, h, own, own)[0]
    cu = torch.tensor([0] + lens, device=DEV).cumsum(0).to(torch.int32)
    return q, k, v, do, m, cu, lens


def _ellipses(g, views, side, fg):
    """Filled ellipses, each covering the same number of cells, `fg` of its
    view: uint8 [views, side, side]."""
    u = torch.rand((views, 4), generator=g, device=DEV)
    cx, cy = (0.4 + 0.2 * u[:, i] for i in (0, 1))
    ratio, th = 0.6 + 0.4 * u[:, 2], math.pi * u[:, 3]
    t = (torch.arange(side, device=DEV) + 0.5) / side
    dx, dy = t[None, None, :] - cx[:, None, None], t[None, :, None] - cy[:, None, None]
    co, si = th.cos()[:, None, None], th.sin()[:, None, None]
    rad = (dx * co + dy * si) ** 2 + ((dy * co - dx * si) / ratio[:, None, None]) ** 2
    rad = rad.reshape(views, -1)
    n = max(1, int(fg * side * side))
    m = torch.zeros(rad.shape, dtype=torch.uint8, device=DEV)
    return m.scatter_(1, rad.argsort(dim=1, stable=True)[:, :n], 1).reshape(views, side, side)


def _latent_inputs(c, seed):
    g = _gen(seed)
    mask = _ellipses(g, c["views"], c["grid"], c["fg"]).reshape(-1)
    L, ch = mask.numel(), c["channels"]
    kept = mask.nonzero().reshape(-1).to(torch.int32)
    inv = torch.full((L,), -1, dtype=torch.int32, device=DEV)
    inv[kept.long()] = torch.arange(kept.numel(), dtype=torch.int32, device=DEV)
    dt = {"bf16": torch.bfloat16, "f32": torch.float32}
    f = lambda rows: torch.randn((rows, ch), generator=g, device=DEV)  # noqa: E731
    n = kept.numel()
    return {"kept": kept, "inv": inv, "z": f(L), "v": f(n).to(dt[c["v"]]), "eps": f(L).to(dt[c["x"]]),
            "z0": f(L).to(dt[c["x"]]), "packed": f(n), "bg": f(c["grid"] ** 2)}


def prepare(case, seed):
    c, kind = case, case["kind"]
    st = {"kind": kind, "case": c}
    if kind in ("fwd", "train"):
        q, k, v, do, m = _attn_inputs(c, seed)
        st.update(q=q, k=k, v=v, do=do, index=ut.build_block_index(m), block=c["block"],
                  scale=1.0 / math.sqrt(c["dim"]), ws=None)
        if kind == "fwd":
            del st["do"]
        b, n, h, _ = q.shape
        ws = c.get("workspace")
        if ws == "kept":
            size = ut.ut_bsattn_bwd_workspace_size_stored(b, n, h, c["block"], st["index"]["nnz"])
            st["ws"] = torch.empty(size, dtype=torch.uint8, device=DEV)
        elif ws == "minimum":
            st["ws"] = torch.empty(ut.ut_bsattn_bwd_workspace_size(b, n, h), dtype=torch.uint8, device=DEV)
    elif kind == "packed":
        q, k, v, do, m, cu, lens = _packed_inputs(c, seed)
        st.update(q=q, k=k, v=v, do=do, cu=cu, longest=max(lens), index=ut.build_block_index(m),
                  block=c["block"], scale=1.0 / math.sqrt(c["dim"]))
    elif kind == "select":
        g = _gen(seed)
        n, h, d = c["n"], c["heads"], c["dim"]
        nb = -(-n // c["block"])
        # tokens of a block resemble each other, as neighbouring patches do
        st["q"], st["k"] = (_normal(g, 1, n, h, d) + 0.5 * _normal(g, 1, nb, h, d).repeat_interleave(
            c["block"], 1)[:, :n] for _ in range(2))
        st["k_keep"] = max(1, int(math.floor(c["keep"] * nb + 1e-9)))
    elif kind == "index":
        st["mask"] = _block_mask(_gen(seed), c, c["batch"], c["heads"], c["nq"], c["nk"])
    elif kind == "drop":
        # the same outlines for every seed (the kept count is an output size),
        # with other alpha values and other rows
        g = _gen(seed)
        shape = _ellipses(_gen(c["grid"] * 100 + c["views"]), c["views"], 16 * c["grid"], c["fg"])
        st["alpha"] = shape * torch.randint(1, 256, shape.shape, generator=g, device=DEV, dtype=torch.uint8)
        L = c["views"] * c["grid"] ** 2
        st["x"], st["out"] = _normal(g, L, c["hidden"]), _normal(g, L, c["hidden"])
    else:
        st.update(_latent_inputs(c, seed))
    return st


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def run(st):
    kind, c = st["kind"], st["case"]
    if kind == "fwd":
        return ut.bsattn_fwd(st["q"], st["k"], st["v"], st["index"], st["block"], st["scale"])
    if kind == "train":
        o, lse = ut.bsattn_fwd(st["q"], st["k"], st["v"], st["index"], st["block"], st["scale"])
        return (o, lse) + tuple(ut.bsattn_bwd(st["q"], st["k"], st["v"], o, st["do"], lse, st["index"],
                                              st["block"], st["scale"], workspace=st["ws"]))
    if kind == "packed":
        o, lse = ut.bsattn_fwd_varlen(st["q"], st["k"], st["v"], st["cu"], st["longest"], st["index"],
                                      st["block"], st["scale"])
        return (o, lse) + tuple(ut.bsattn_bwd_varlen(st["q"], st["k"], st["v"], o, st["do"], lse, st["cu"],
                                                     st["longest"], st["index"], st["block"], st["scale"]))
    if kind == "select":
        return ut.topk_block_mask(st["q"], st["k"], c["block"], st["k_keep"], prefix_blocks=c["prefix"])
    if kind == "index":
        return ut.build_block_index(st["mask"])
    if kind == "drop":
        mask = ut.token_mask_from_alpha(st["alpha"], radius=c["radius"])
        d = ut.drop_background(mask.reshape(-1), st["x"])
        return mask, d, ut.scatter_foreground(d["x_packed"], d["kept_idx"], st["out"])
    z = ut.euler_update_foreground(st["z"], st["v"], st["kept"], -0.02)
    loss, grad = ut.fg_flow_loss(st["v"], st["eps"], st["z0"], st["kept"])
    mix = ut.composite_latent(st["packed"], st["inv"], st["bg"], st["kept"].numel())
    return z, loss, grad, mix


# ---------------------------------------------------------------------------
# the work a pass cannot do without
# ---------------------------------------------------------------------------

def _pairs(n, block, keep):
    """Retained (query, key) token pairs of one head, real tokens only."""
    nb = -(-n // block)
    per = nb if keep >= 1.0 else min(int(math.floor(keep * nb + 1e-9)), nb - 1) + 1
    return n * n * per / nb


def work(case):
    c, kind = case, case["kind"]
    if kind in ("fwd", "train", "packed"):
        lens = _lens(c) if kind == "packed" else [c["n"]] * c.get("batch", 1)
        h, d = c["heads"], c["dim"]
        rows = sum(lens) * h
        flops = 4.0 * d * h * sum(_pairs(n, c["block"], c["keep"]) for n in lens)
        if kind == "fwd":   # q, k, v in, o and lse out
            return {"bytes": rows * (4 * 2 * d + 4), "flops": flops}
        return {"bytes": rows * (8 * 2 * d + 4), "flops": 3.5 * flops}
    if kind == "select":
        nb = -(-c["n"] // c["block"])
        return {"bytes": 2 * c["n"] * c["heads"] * c["dim"] * 2 + c["heads"] * nb * nb,
                "flops": 2.0 * c["heads"] * nb * nb * c["dim"] + 2.0 * c["n"] * c["heads"] * c["dim"]}
    if kind == "index":
        bh, nq, nk = c["batch"] * c["heads"], c["nq"], c["nk"]
        per = nk if c["keep"] >= 1.0 else _kept_per_row(c, nk) + 1
        return {"bytes": bh * (nq * nk + 4 * (nq + nk) + 2 * 4 * nq * per), "flops": 0}
    if kind == "drop":
        L = c["views"] * c["grid"] ** 2
        return {"bytes": 256 * L + L + 4 * L + L * c["fg"] * (4 + 4 * 2 * c["hidden"]), "flops": 0}
    L, ch = c["views"] * c["grid"] ** 2, c["channels"]
    n = L * c["fg"]
    sv, sx = (2 if c[k] == "bf16" else 4 for k in ("v", "x"))
    return {"bytes": n * ch * (8 + 2 * sv + 2 * sx + 4 + 4) + 4 * L * ch + 4 * L, "flops": 8.0 * n * ch}


def tolerance(case):
    kind = case["kind"]
    if kind in ("fwd", "train", "packed"):
        # bf16 results, and P and dS rounded to bf16 before their products
        return {"rel": 1e-2, "max": 6e-2}
    if kind == "select":
        # fp32 sums in another order move a score by an ulp: near ties may swap
        return {"rel": 0.0, "differ": 1e-5}
    if kind == "latent":
        return {"rel": 1e-6, "max": 1e-5}
    return "exact"


# ---------------------------------------------------------------------------
# the same results in 64 bits, plain torch
# ---------------------------------------------------------------------------

def _exact_head(q, k, v, do, mask, block, scale):
    """One head of one sample: fp64 [n, d] inputs (do may be None), mask
    [nb, nb] bool. Query blocks are taken in groups, each against the key
    blocks that it lists."""
    n, d = q.shape
    nb = mask.shape[0]
    pad = nb * block - n

    def blocks(x):
        return torch.nn.functional.pad(x, (0, 0, 0, pad)).reshape(nb, block, d)

    qb, kb, vb = blocks(q), blocks(k), blocks(v)
    dob = blocks(do) if do is not None else None
    counts = mask.sum(1)
    m = int(counts.max())
    idx = torch.argsort(mask.to(torch.int8), dim=1, descending=True, stable=True)[:, :m]
    live = torch.arange(m, device=DEV)[None] < counts[:, None]
    real = (torch.arange(nb * block, device=DEV) < n).reshape(nb, block)
    o, lse = torch.zeros_like(qb), torch.full((nb, block), -math.inf, dtype=torch.float64, device=DEV)
    dq, dk, dv = torch.zeros_like(qb), torch.zeros_like(kb), torch.zeros_like(vb)
    step = max(1, int(1.0e9 // (8 * m * block * max(d, block))))
    for i0 in range(0, nb, step):
        sl = slice(i0, min(nb, i0 + step))
        ix = idx[sl]
        kg, vg = kb[ix].flatten(1, 2), vb[ix].flatten(1, 2)
        ok = (live[sl][:, :, None] & real[ix]).flatten(1)[:, None, :]
        s = torch.matmul(qb[sl], kg.transpose(1, 2)) * scale
        s = s.masked_fill(~ok, -math.inf)
        l = torch.logsumexp(s, 2)
        p = torch.exp(s - l[:, :, None])
        o[sl], lse[sl] = torch.matmul(p, vg), l
        if do is None:
            continue
        dp = torch.matmul(dob[sl], vg.transpose(1, 2))
        ds = p * (dp - (dob[sl] * o[sl]).sum(2, keepdim=True))
        dq[sl] = torch.matmul(ds, kg) * scale
        flat = ix.flatten()
        live_rows = real[sl][:, :, None]
        ds, p = ds * live_rows, p * live_rows
        dk.index_add_(0, flat, (torch.matmul(ds.transpose(1, 2), qb[sl]) * scale).reshape(-1, block, d))
        dv.index_add_(0, flat, torch.matmul(p.transpose(1, 2), dob[sl]).reshape(-1, block, d))
    cut = lambda x: x.reshape(nb * block, -1)[:n]  # noqa: E731
    return cut(o), cut(lse)[:, 0], cut(dq), cut(dk), cut(dv)


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind in ("fwd", "train"):
        q, k, v, do, m = _attn_inputs(c, seed)
        samples = [(b, slice(None)) for b in range(q.shape[0])]
        view = lambda x, b, rows: x[b]  # noqa: E731
    elif kind == "packed":
        q, k, v, do, m, cu, lens = _packed_inputs(c, seed)
        ends = torch.tensor([0] + lens).cumsum(0).tolist()
        samples = [(b, slice(ends[b], ends[b + 1])) for b in range(len(lens))]
        view = lambda x, b, rows: x[rows]  # noqa: E731
    elif kind == "latent":
        t = _latent_inputs(c, seed)
        at = t["kept"].long()
        v, z = t["v"].double(), t["z"].double()
        z[at] += -0.02 * v
        diff = v - (t["eps"].double()[at] - t["z0"].double()[at])
        mix = t["bg"].repeat(c["views"], 1).double()
        mix[at] = t["packed"].double()
        return z, (diff ** 2).mean().reshape(1), 2 * diff / diff.numel(), mix
    else:
        return None
    scale = 1.0 / math.sqrt(c["dim"])
    outs = [torch.zeros(q.shape, dtype=torch.float64, device=DEV) for _ in range(4)]
    if kind == "packed":
        lse = torch.zeros((q.shape[1], q.shape[0]), dtype=torch.float64, device=DEV)
    else:
        lse = torch.zeros((q.shape[0], q.shape[2], q.shape[1]), dtype=torch.float64, device=DEV)
    for b, rows in samples:
        for h in range(c["heads"]):
            qh, kh, vh, doh = (view(x, b, rows)[:, h].double() for x in (q, k, v, do))
            n = qh.shape[0]
            nb = -(-n // c["block"])
            got = _exact_head(qh, kh, vh, doh if kind != "fwd" else None, m[b, h, :nb, :nb].bool(),
                              c["block"], scale)
            for x, y in zip(outs, (got[0],) + got[2:]):
                view(x, b, rows)[:, h] = y
            if kind == "packed":
                lse[h, rows] = got[1]
            else:
                lse[b, h] = got[1]
    if kind == "fwd":
        return outs[0], lse
    return (outs[0], lse) + tuple(outs[1:])

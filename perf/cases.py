"""Performance cases of the ToMA layer path on one MI355X: what is timed, over which range of sizes.

Every case goes through the public binding (`paper_2509_10918_amd.binding`) as a denoising program
calls it: descriptors, weights, workspace and pattern cache are made once, a pass is one layer call
(or one reuse sequence, or one block built from the stage calls) on the tokens of a step.  Inputs
are seeded stand-ins for hidden states: a spatially smooth field per channel plus white noise, as in
`paper_2509_10918_amd.synth`, drawn on the GPU.

A case is a dict:
    kind    "layer"      one toma_layer call (`flags`: 0 nothing cached, 1 idx cached, 2 idx + weights
                         cached, 4 weights recomputed, 5 the same with idx cached)
            "sequence"   `steps` layer calls on drifting tokens along a reuse schedule (Sec. 4.3.2)
            "block"      merge once, self-attention, cross-attention, MLP, unmerge (ToMA_once, Sec. 5.1)
            "pinv"       merge with cached weights, attention, Moore-Penrose unmerge (App. E.4)
    dtype, B, H, W, C, th, tw (region shape), d_loc (destinations per region), heads, extra (tokens
    that join the attention unmerged), tile (merge weights inside each region instead of globally),
    sigma, noise (smoothness of the tokens)
"""
import math

import torch

from paper_2509_10918_amd import binding as tb

TAU = 0.1
#: context tokens and their width in the "block" cases (77 text tokens, as SDXL's text encoders give)
T_CTX, C_CTX = 77, 2048
RCOND = 1e-2


def _case(name, kind="layer", **kw):
    c = dict(name=name, kind=kind, dtype="bf16", B=2, H=64, W=64, C=640, th=16, tw=16, d_loc=128, heads=10, extra=0,
             tile=False, flags=0, steps=1, sigma=2.0, noise=0.2)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: a 16 x 16 grid in fp32, as in smoke tests and tiny models (launches, host path)
        _case("tiny_f32", dtype="f32", B=1, H=16, W=16, C=64, th=8, tw=8, d_loc=32, heads=1, sigma=1.5, noise=0.1),
        # the headline layer: SDXL's first stage, half of the tokens kept, nothing cached
        _case("sdxl1"),
        # the same layer on most steps of a run: pattern and weights cached
        _case("sdxl1_cached", flags=2),
        # SDXL's second stage with region-local merge, nothing cached
        _case("sdxl2_tile", H=32, W=32, C=1280, th=8, tw=8, d_loc=32, heads=20, tile=True, sigma=1.5),
        # fp32 layer of the same stage with new weights on cached destinations (full-precision runs)
        _case("sdxl2_f32_idx", dtype="f32", H=32, W=32, C=1280, th=8, tw=8, d_loc=32, heads=20, flags=1, sigma=1.5),
        # Flux block: one sample, 512 text tokens, a quarter kept, wide rows
        _case("flux", B=1, C=3072, d_loc=64, heads=24, extra=512, noise=0.0),
        # a non-square grid whose tile, width, keep ratio, batch and extra tokens fit no block size evenly
        _case("odd_tile", B=3, H=40, W=72, C=352, th=8, tw=12, d_loc=29, heads=11, extra=77, tile=True, sigma=1.5),
        # few large regions (the other end of the region-count ablation): 1024 tokens each
        _case("sdxl1_4regions", th=32, tw=32, d_loc=512),
        # a transformer block that merges once and runs all its modules on the merged tokens, idx cached
        _case("sdxl2_block", "block", H=32, W=32, C=1280, th=8, tw=8, d_loc=32, heads=20, tile=False, sigma=1.5),
        # weights recomputed instead of stored, destinations cached (memory-lean runs)
        _case("sdxl1_recompute", flags=5),
        # the pseudo-inverse unmerge that the transpose is measured against, region-local
        _case("sdxl2_pinv", "pinv", H=32, W=32, C=1280, th=8, tw=8, d_loc=32, heads=20, tile=True, sigma=1.5),
        # ten denoising steps on a 128 x 128 grid along the reuse schedule: the largest
        _case("hires_steps", "sequence", H=128, W=128, steps=10, sigma=3.0, noise=0.0),
    ]


def draw(rng):
    """One more case of the same ranges: grids of 16 to 128 a side, regions of 16 to 1024 tokens, widths of
    64 to 3072, both dtypes, both merge modes, every kind of call."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        kind = rng.choice(["layer"] * 7 + ["sequence", "block", "pinv"])
        dtype = "f32" if rng.random() < 0.2 else "bf16"
        th, tw = rng.choice([(4, 4), (8, 8), (8, 8), (16, 8), (8, 12), (12, 12), (10, 16), (16, 16), (16, 16), (16, 16),
                             (4, 64), (2, 64), (24, 24), (32, 32)])
        gh, gw = max(1, round(log_int(16, 128) / th)), max(1, round(log_int(16, 128) / tw))
        H, W = gh * th, gw * tw
        hd = rng.choice([32, 64, 64, 64, 128])
        C = max(64, log_int(64, 3072) // hd * hd)
        heads = C // hd
        if heads < 1 or C % 32:
            continue
        n_loc = th * tw
        d_loc = max(1, int(n_loc * rng.choice([0.25, 0.5, 0.5, 0.75, rng.uniform(0.1, 0.9)])))
        B = rng.choice([1, 1, 2, 2, 3, 4])
        extra = rng.choice([0, 0, 0, 77, 154, 333, 512])
        tile = rng.random() < 0.5
        flags = rng.choice([0, 0, 0, 1, 1, 2, 2, 4, 5]) if kind == "layer" else 0
        steps = rng.choice([5, 10]) if kind == "sequence" else 1
        if kind in ("block", "pinv"):
            extra = 0
        if kind == "pinv":
            tile = True
            if d_loc > 128 or d_loc < 4:
                continue
        N, P = H * W, gh * gw
        if N < 256 or H > 128 or W > 128:
            continue
        D = P * d_loc
        if kind == "block" and T_CTX > D:
            continue
        if flags in (4, 5) and C > 3072:
            continue
        c = _case("", kind, dtype=dtype, B=B, H=H, W=W, C=C, th=th, tw=tw, d_loc=d_loc, heads=heads, extra=extra, tile=tile,
                  flags=flags, steps=steps, sigma=rng.choice([1.5, 2.0, 3.0]), noise=rng.choice([0.0, 0.1, 0.2]))
        w = work(c)
        # no more work than the listed cases have (an fp32 product costs about sixteen times a bf16 one; the
        # eigen-decompositions of the pseudo-inverse and long selections of large regions cost beyond their flops)
        cost = w["flops"] * (16 if dtype == "f32" else 1)
        if cost > 1.0e12 or w["bytes"] > 2.0e9 or steps * B * N * C * (2 if dtype == "bf16" else 4) > 4.0e8:
            continue
        if kind == "pinv" and B * P * d_loc ** 3 > 1.4e8:
            continue
        if n_loc > 256 and d_loc * steps > 2560:
            continue
        del c["name"]
        return c


# ---------------------------------------------------------------------------------------------- inputs

def _blur_matrix(n, sigma, device):
    """n x n matrix of a Gaussian blur of width sigma with reflecting ends, rows scaled to keep unit variance."""
    r = int(math.ceil(4.0 * sigma))
    x = torch.arange(-r, r + 1, dtype=torch.float64)
    k = torch.exp(-0.5 * (x / sigma) ** 2)
    k = k / k.sum()
    m = torch.zeros(n, n, dtype=torch.float64)
    pos = torch.arange(n)
    for o in range(-r, r + 1):
        q = (pos + o) % (2 * n) if n > 1 else pos * 0
        q = torch.where(q >= n, 2 * n - 1 - q, q)
        m[pos, q] += k[o + r]
    return (m / math.sqrt(float((k * k).sum()))).float().to(device)


def _tokens(case, gen, dt):
    B, H, W, C = case["B"], case["H"], case["W"], case["C"]
    z = torch.randn(B, H, W * C, generator=gen, device="cuda")
    z = torch.matmul(_blur_matrix(H, case["sigma"], "cuda"), z)
    z = torch.matmul(_blur_matrix(W, case["sigma"], "cuda"), z.view(B * H, W, C))
    if case["noise"] > 0:
        z = z + case["noise"] * torch.randn(B * H, W, C, generator=gen, device="cuda")
    return z.reshape(B, H * W, C).contiguous()


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed) * 7919 + 13)
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    B, H, W, C, kind = case["B"], case["H"], case["W"], case["C"], case["kind"]
    P = (H // case["th"]) * (W // case["tw"])
    R = P if case["tile"] else 1
    N, D = H * W, P * case["d_loc"]

    def randn(*shape, std=1.0):
        return (torch.randn(*shape, generator=gen, device="cuda") * std).to(dt).contiguous()

    s = {"case": case}
    s["desc"] = desc = tb.make_desc(B, H, W, C, case["th"], case["tw"], case["d_loc"], R, TAU, dt)
    s["attn"] = attn = tb.toma_attn_desc(case["heads"], C // case["heads"], case["extra"])
    x = _tokens(case, gen, dt)
    s["X"] = x.to(dt).contiguous()
    s["Xe"] = randn(B, case["extra"], C) if case["extra"] else None
    s["Wq"], s["Wk"], s["Wv"] = (randn(C, C, std=C ** -0.5) for _ in range(3))
    s["ws"] = tb.alloc_workspace(desc, attn)
    s["idx"], s["A"], s["Z"], s["amap"] = tb.alloc_cache(desc)
    s["Y"] = torch.empty(B, N, C, dtype=dt, device="cuda")
    s["Ye"] = torch.empty(B, case["extra"], C, dtype=dt, device="cuda") if case["extra"] else None
    if kind == "sequence":
        # X_t = X_{t-1} + drift * noise: destinations anew every 5 steps, weights every 2 in between
        s["Xs"], s["Ys"], s["plan"] = [s["X"]], [s["Y"]], []
        for t in range(case["steps"]):
            s["plan"].append(0 if t % 5 == 0 else (tb.TOMA_REUSE_IDX if t % 5 % 2 == 0 else tb.TOMA_REUSE_A))
            if t:
                x = x + 0.02 * torch.randn(x.shape, generator=gen, device="cuda")
                s["Xs"].append(x.to(dt).contiguous())
                s["Ys"].append(torch.empty_like(s["Y"]))
    elif kind in ("block", "pinv"):
        s["Xm"] = torch.empty(B, D, C, dtype=dt, device="cuda")
        s["O"] = torch.empty(B, D, C, dtype=dt, device="cuda")
        tb.toma_select(desc, s["X"], s["idx"], None, None, s["ws"])
        if kind == "block":
            s["O2"], s["O3"] = torch.empty_like(s["O"]), torch.empty_like(s["O"])
            s["Ctx"] = randn(B, T_CTX, C_CTX)
            s["Uq"], s["Wo"] = randn(C, C, std=C ** -0.5), randn(C, C, std=C ** -0.5)
            s["Uk"], s["Uv"] = randn(C_CTX, C, std=C_CTX ** -0.5), randn(C_CTX, C, std=C_CTX ** -0.5)
            s["W1"], s["W2"] = randn(C, 4 * C, std=C ** -0.5), randn(4 * C, C, std=(4 * C) ** -0.5)
            s["Hb"] = torch.empty(B * D, 4 * C, dtype=dt, device="cuda")
        else:
            tb.toma_merge(desc, s["X"], s["idx"], s["A"], s["Z"], s["amap"], s["Xm"], s["ws"])
    elif case["flags"] & (tb.TOMA_REUSE_IDX | tb.TOMA_REUSE_A):
        # the cache of an earlier step, whose tokens were a little different
        before = (x + 0.02 * torch.randn(x.shape, generator=gen, device="cuda")).to(dt).contiguous()
        tb.toma_select(desc, before, s["idx"], None, None, s["ws"])
        if case["flags"] & tb.TOMA_REUSE_A:
            Xm = torch.empty(B, D, C, dtype=dt, device="cuda")
            tb.toma_merge(desc, before, s["idx"], s["A"], s["Z"], s["amap"], Xm, s["ws"])
    return s


def run(s):
    case, desc, attn = s["case"], s["desc"], s["attn"]
    kind = case["kind"]
    if kind == "layer":
        f = case["flags"]
        tb.toma_layer(desc, attn, f, s["X"], s["Xe"], s["idx"], s["A"], s["Z"], s["amap"], s["Wq"], s["Wk"], s["Wv"], None,
                      s["Y"], s["Ye"], s["ws"])
        out = {"Y": s["Y"], "Ye": s["Ye"], "idx": s["idx"], "Z": s["Z"]}
        if not f & (tb.TOMA_REUSE_A | tb.TOMA_RECOMPUTE_WEIGHTS):
            out["A"] = s["A"]
        return out
    if kind == "sequence":
        for t, f in enumerate(s["plan"]):
            tb.toma_layer(desc, attn, f, s["Xs"][t], s["Xe"], s["idx"], s["A"], s["Z"], s["amap"], s["Wq"], s["Wk"], s["Wv"],
                          None, s["Ys"][t], s["Ye"], s["ws"])
        return {"Ys": s["Ys"], "Ye": s["Ye"], "idx": s["idx"], "Z": s["Z"], "A": s["A"]}
    if kind == "block":
        tb.toma_merge(desc, s["X"], s["idx"], s["A"], s["Z"], s["amap"], s["Xm"], s["ws"])
        tb.toma_attend(desc, attn, s["Xm"], None, s["Wq"], s["Wk"], s["Wv"], s["Wo"], s["O"], s["ws"])
        tb.toma_cross_attend(desc, attn, s["O"], s["Ctx"], s["Uq"], s["Uk"], s["Uv"], s["Wo"], s["O2"], s["ws"])
        tb.toma_mlp(s["O2"], s["W1"], s["W2"], s["Hb"], s["O3"])
        tb.toma_unmerge(desc, s["A"], s["Z"], s["amap"], s["O3"], s["Y"], s["ws"])
        return {"Xm": s["Xm"], "O": s["O"], "O2": s["O2"], "O3": s["O3"], "Y": s["Y"], "A": s["A"], "Z": s["Z"]}
    tb.toma_merge_cached(desc, s["X"], s["A"], s["Z"], s["amap"], s["Xm"], s["ws"])
    tb.toma_attend(desc, attn, s["Xm"], None, s["Wq"], s["Wk"], s["Wv"], None, s["O"], s["ws"])
    tb.toma_unmerge_pinv(desc, s["A"], s["Z"], s["O"], RCOND, s["Y"], s["ws"])
    return {"Xm": s["Xm"], "O": s["O"], "Y": s["Y"]}


# ------------------------------------------------------------------------------------- work, tolerance

def _layer_work(c, flags):
    """Bytes and flops of one layer call: inputs read once, outputs written once, the method's products
    (2 per multiply-add) with the merge matrix taken as dense."""
    es = 2 if c["dtype"] == "bf16" else 4
    B, N, C = c["B"], c["H"] * c["W"], c["C"]
    n_loc = c["th"] * c["tw"]
    P = N // n_loc
    D, R = P * c["d_loc"], P if c["tile"] else 1
    L = D + c["extra"]
    mm = 2.0 * B * N * D * C / R
    flops = 2 * mm + 6.0 * B * L * C * C + 4.0 * B * L * L * C
    byts = es * (2.0 * B * N * C + 2.0 * B * c["extra"] * C + 3.0 * C * C)
    a_bytes = es * float(B) * N * D / R + 4.0 * B * D
    if flags & 4:
        flops += mm
    elif flags & 2:
        byts += a_bytes
    else:
        flops += mm
        byts += a_bytes
    if not flags & 3:
        flops += 2.0 * B * N * n_loc * C
        byts += 4.0 * B * D
    return byts, flops


def work(case):
    c, kind = case, case["kind"]
    if kind == "layer":
        b, f = _layer_work(c, c["flags"])
    elif kind == "sequence":
        b = f = 0.0
        for t in range(c["steps"]):
            x, y = _layer_work(c, 0 if t % 5 == 0 else (1 if t % 5 % 2 == 0 else 2))
            b, f = b + x, f + y
    else:
        es = 2 if c["dtype"] == "bf16" else 4
        b, f = _layer_work(c, 1 if kind == "block" else 2)
        B, C = c["B"], c["C"]
        n_loc = c["th"] * c["tw"]
        P = c["H"] * c["W"] // n_loc
        D = P * c["d_loc"]
        if kind == "block":
            f += 2.0 * B * D * C * C * 3 + 4.0 * B * T_CTX * C_CTX * C + 4.0 * B * D * T_CTX * C + 16.0 * B * D * C * C
            b += es * (2.0 * C * C + 2.0 * C_CTX * C + 8.0 * C * C + B * T_CTX * C_CTX + 4.0 * B * D * C)
        else:
            # A~ A~^T and its factorisation per region, then the product with the inverse
            f += B * P * (2.0 * c["d_loc"] ** 2 * n_loc + 4.0 * c["d_loc"] ** 3 + 2.0 * c["d_loc"] ** 2 * C)
            b += es * 2.0 * B * D * C
    return {"bytes": b, "flops": f}


def tolerance(case):
    """Four times the largest error seen against a float64 evaluation over the listed and two dozen drawn cases.
    bf16 (4.3e-3, single values 7e-2): weights, Q / K / V, probabilities and outputs are each rounded to 8 bits.
    fp32 with fresh weights (4e-4 at C = 1280, single values 6e-3; 7e-6 at C = 64): logits of about 10 C carry
    their fp32 rounding into the weights' exponent.  fp32 with cached weights (1.1e-6): products and sums alone."""
    if case["dtype"] == "bf16":
        return {"rel": 1.7e-2, "max": 0.28, "differ": 0.0}
    if case["flags"] & 2 or case["kind"] == "pinv":
        return {"rel": 1e-5, "max": 1e-3, "differ": 0.0}
    return {"rel": max(4e-5, 1.25e-6 * case["C"]), "max": max(1e-3, 2e-5 * case["C"]), "differ": 0.0}

#!/usr/bin/env python3
"""Benchmark of the ToMA layer path on one MI355X.

A step is one whole layer call (select -> merge weights -> merge -> attention -> unmerge, nothing
cached) on seeded synthetic hidden states of the SDXL stage-1 shape (B=2, 64x64 tokens, width 640).
Prints ONE JSON line: microseconds per layer call, the roofline of the kernel that takes the most
time (per-kernel durations measured live with HIP events on the launch stream), the cached-pattern
variants, and the fp64 CPU oracle timed on the same inputs on the host cores.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload sdxl1] [--merge-regions global|tile]
"""
import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "µs per merge+attn+unmerge layer call (SDXL 4096×640); % bf16 MFMA / HBM roofline"
PEAK = {"hbm": 8000.0, "bf16": 2500.0, "f32": 157.3, "f64": 78.6, "i8": 5000.0}   # GB/s, TFLOP/s, TOP/s (MI355X, dense)


def executed_fraction(amap, desc, which, tile, esize):
    """Share of the K steps that the merge (which = 0) / unmerge (1) product runs, counted from the block
    map of A exactly as the kernel's workgroups do: a K step (128 bytes of elements) of a workgroup's tile
    runs iff some map block it covers is occupied.  amap: uint8 [regions, dest blocks of 128, source
    blocks of 32] as numpy."""
    bm = tile[0]
    kstep = 128 // esize
    z, db, sb = amap.shape
    occ = amap != 0
    if which == 0:      # rows = destinations (tiles of bm), K = sources
        dpt = max(bm // 128, 1)
        rows = occ.reshape(z, db // dpt, dpt, sb).any(axis=2) if db % dpt == 0 else occ
        spk = max(kstep // 32, 1)
        act = rows.reshape(z, rows.shape[1], sb // spk, spk).any(axis=3)
    else:               # rows = sources (tiles of bm), K = destinations
        spt = max(bm // 32, 1)
        cols = occ.reshape(z, db, sb // spt, spt).any(axis=3) if sb % spt == 0 else occ
        # a K step of 64 destinations lies inside one destination block of 128
        act = np.repeat(cols, max(128 // kstep, 1), axis=1)
    return float(act.mean())


def kernel_work(w, R, esize, exec_frac=None, int8_gram=False, screened=False):
    """Work per launch of each kernel: name -> dict(bound, amount, [equiv, limit]).
    amount = what the kernel as built has to execute or move (flops for the matrix-core kernels, bytes
    for the streaming ones); equiv = the count of the textbook formulation where the kernel reaches the
    same result with less (dense products for the block-skipping ones, the full product for the
    symmetric Gram matrix, a rescan of S per round for the greedy loop), reported under its own name."""
    from paper_2509_10918_amd import costs
    f = costs.stage_flops(w.B, w.N, w.C, w.P, w.d_loc, R, w.T_extra)
    L = w.D + w.T_extra
    mm = "bf16" if w.dtype == "bf16" else "f32"
    a_bytes = w.B * w.D * (w.N // R) * esize
    tiles = w.n_loc // 16
    tri = (tiles * (tiles + 1) / 2) / (tiles * tiles)      # blocks on or above the diagonal
    ef = exec_frac or {}
    if int8_gram:
        # exact similarities on the int8 matrix cores: sixteen limb-pair products per 64 x 32 block of S on or
        # above the diagonal, channels padded to 64
        nb64, nb32 = (w.n_loc + 63) // 64, (w.n_loc + 31) // 32
        units = sum(nb32 - 2 * bm for bm in range(nb64))
        cpad = (w.C + 63) // 64 * 64
        gram = dict(bound="i8", amount=16 * 2 * w.B * w.P * units * 64 * 32 * cpad, equiv=f["similarity"],
                    limit="LDS bandwidth and fixed cost: a 32 x 16 wave tile reads 384 bytes of limbs per product "
                          "(about 64 bytes a clock per CU is what 16-byte LDS reads reach here), and some 10 us per "
                          "launch go to first loads, norms, the double-precision combination and the stores")
    else:
        gram = dict(bound="f64", amount=f["similarity"] * tri, equiv=f["similarity"],
                    limit="issue rate of the fp64 matrix-core products (a bare loop of them reaches 43-47 TFLOP/s)")
    work = {
        "gram": gram,
        "limbs": dict(bound="hbm", amount=w.B * w.N * (w.C * esize + (w.C + 63) // 64 * 64 * 4 + 17)),
        "greedy": dict(bound="hbm", amount=w.B * w.P * w.n_loc * w.n_loc * 4 + 3 * w.B * w.D * 4,
                       equiv=costs.greedy_stream_bytes(w.B, w.P, w.n_loc, w.d_loc),
                       limit="latency: d_loc dependent rounds per region (argmax, LDS exchange, two barriers); S is "
                             "read once and stays in registers, 32 of 256 CUs are busy"),
        "weights_stats": dict(bound=mm, amount=f["weights"]),
        "lse": dict(bound="hbm", amount=w.B * w.N * 12),
        # (the write pass of the two-pass weights skips the product of tiles that the first pass proved empty)
        "weights_write": (dict(bound=mm, amount=f["weights"] * ef["weights_write"], equiv=f["weights"]) if "weights_write" in ef
                          else dict(bound=mm, amount=f["weights"],
                                    limit="L2 to CU bandwidth: every 32-source workgroup streams all destination rows "
                                          "(with the products or the loads taken out the loop takes 30 / 21 of its 35 us)")),
        # screened weights: exact logits with the destinations of a source's own region, and the rows in 4 bits (the
        # screen itself runs as weights_stats, the exact tiles as weights_write: below)
        "weights_bounds": dict(bound=mm, amount=2 * w.B * w.N * w.d_loc * w.C, limit="a chain of dependent loads"),
        # one kernel per small merge region: logits (repeated per slice of the channels: not counted), softmax, merge
        "local_merge": dict(bound=mm, amount=f["weights"] + f["merge"],
                            limit="a chain of K steps per workgroup, each a wait, a barrier and a few products"),
        "zsum": dict(bound="hbm", amount=w.B * w.D * 8, limit="launch latency"),
        "merge": dict(bound=mm, amount=f["merge"] * ef.get("merge", 1.0), equiv=f["merge"]),
        "qkv": dict(bound=mm, amount=f["qkv"]),
        "attention": dict(bound=mm, amount=f["attention"]),
        "proj": dict(bound=mm, amount=2 * w.B * L * w.C * w.C),
        "scale_rows": dict(bound="hbm", amount=2 * w.B * w.D * w.C * esize),
        "unmerge": dict(bound=mm, amount=f["unmerge"] * ef.get("unmerge", 1.0), equiv=f["unmerge"]),
        # second pass of a K-split merge / unmerge product: at least two fp32 partials in, one tile out
        "split_finish": dict(bound="hbm", amount=w.B * w.D * w.C * (2 * 4 + esize)),
        "occupancy": dict(bound="hbm", amount=a_bytes),   # one read of the stored weights
    }
    if screened:
        # the screen leaves zeros in A and reads the rows in 4 bits; its own products are in another unit and take half as long
        work["weights_stats"] = dict(bound="hbm", amount=a_bytes + w.B * w.N * w.C / 2, limit="the zeros of A")
        work["weights_write"] = dict(bound=mm, amount=f["weights"] * ef.get("weights_write", 0.0), equiv=f["weights"],
                                     limit="latency: a list of marked tiles and dependent gathers per 32 sources")
    return work


def roofline_entry(name, work, avg_us, traffic=None):
    """achieved = work of the kernel as built / duration against the MI355X peak of its roof; equiv_* the
    same for the textbook count; traffic_* from the HBM bytes rocprofv3 counted for this kernel."""
    wk = work[name]
    bound = wk["bound"]
    sec = avg_us * 1e-6
    if bound == "hbm":
        out = {"kernel": name, "bound": "hbm", "achieved": wk["amount"] / sec / 1e9, "peak": PEAK["hbm"], "unit": "GB/s"}
    else:
        out = {"kernel": name, "bound": "mfma", "achieved": wk["amount"] / sec / 1e12, "peak": PEAK[bound],
               "unit": "TOP/s" if bound == "i8" else "TFLOP/s", "mfma_dtype": bound}
    out["frac"] = out["achieved"] / out["peak"]
    out["traffic"] = traffic
    if "equiv" in wk:
        scale = 1e9 if bound == "hbm" else 1e12
        out["equiv_achieved"] = wk["equiv"] / sec / scale
        if bound != "i8":   # (the textbook count is in flops of another unit there: a rate, no fraction)
            out["equiv_frac"] = out["equiv_achieved"] / out["peak"]
    if traffic:
        out["traffic_GBps"] = traffic / sec / 1e9
        out["traffic_frac_of_hbm"] = out["traffic_GBps"] / PEAK["hbm"]
    if "limit" in wk:
        out["binding_limit"] = wk["limit"]
    return out


def greedy_rounds(w, steps):
    """Selection (toma_select) of the workload's tokens with 1/16 ... 3/4 of each region kept: the greedy
    kernel runs one round per pick, so its duration over the number of picks gives the cost of a round and
    of what does not depend on the rounds (reading S, the first keys, writing the picks)."""
    import torch
    from paper_2509_10918_amd import binding as tb
    from paper_2509_10918_amd import synth
    X = torch.from_numpy(np.ascontiguousarray(synth.make_inputs(w)["X"], dtype=np.float32)).to("cuda")
    X = X.to(torch.bfloat16 if w.dtype == "bf16" else torch.float32).contiguous()
    rows = []
    for d_loc in sorted({max(w.n_loc // 16, 1), w.n_loc // 8, w.n_loc // 4, 3 * w.n_loc // 8, w.n_loc // 2, 3 * w.n_loc // 4}):
        desc = tb.make_desc(w.B, w.H, w.W, w.C, w.tile_h, w.tile_w, d_loc, 1, w.tau, w.dtype)
        ws = tb.alloc_workspace(desc)
        idx = torch.empty((w.B, w.P, d_loc), dtype=torch.int32, device="cuda")
        for _ in range(5):
            tb.toma_select(desc, X, idx, None, None, ws)
        tb.toma_profile_enable(True)
        tb.toma_profile_read("greedy")
        for _ in range(steps):
            tb.toma_select(desc, X, idx, None, None, ws)
        torch.cuda.synchronize()
        n, total = tb.toma_profile_read("greedy")
        tb.toma_profile_enable(False)
        rows.append((d_loc, total * 1e3 / n))
    d = np.array([r[0] for r in rows], float)
    t = np.array([r[1] for r in rows], float)
    slope, fixed = np.polyfit(d, t, 1)
    print(f"# greedy kernel of {w.name}: {w.B * w.P} regions of {w.n_loc} tokens, one workgroup each; average us per launch")
    print(f"# command: python bench.py --workload {w.name} --greedy-rounds --steps {steps}")
    print(f"{'picks per region':>18}{'us':>10}{'us per pick':>14}")
    for dl, us in rows:
        print(f"{dl:>18}{us:>10.2f}{us / dl:>14.3f}")
    print(f"linear fit: {fixed:.1f} us + {slope:.3f} us per round ({slope * 2400:.0f} clocks at 2.4 GHz); the first rounds cost "
          f"more than the later ones (every column changes at the first pick, a handful later)")


def greedy_parts(w):
    """One selection of the workload's tokens through the greedy kernel that times the parts of its rounds
    (toma_profile_greedy_parts): shader clocks per round and part, per wave, averaged over the regions."""
    import torch
    from paper_2509_10918_amd import binding as tb
    from paper_2509_10918_amd import synth
    X = torch.from_numpy(np.ascontiguousarray(synth.make_inputs(w)["X"], dtype=np.float32)).to("cuda")
    X = X.to(torch.bfloat16 if w.dtype == "bf16" else torch.float32).contiguous()
    desc = tb.make_desc(w.B, w.H, w.W, w.C, w.tile_h, w.tile_w, w.d_loc, 1, w.tau, w.dtype)
    ws = tb.alloc_workspace(desc)
    waves = (w.n_loc // 16 + 1) // 2
    idx = torch.empty((w.B, w.P, w.d_loc), dtype=torch.int32, device="cuda")
    ref = torch.empty_like(idx)
    parts = torch.zeros((w.B * w.P, waves, 8), dtype=torch.int64, device="cuda")
    tb.toma_select(desc, X, ref, None, None, ws)
    for _ in range(3):
        tb.toma_profile_greedy_parts(desc, X, idx, parts, ws)
    torch.cuda.synchronize()
    assert torch.equal(idx, ref), "the timing variant must pick what toma_select picks"
    p = parts.cpu().numpy().astype(np.float64)
    rounds = p[:, :, 5]
    assert np.all(rounds == w.d_loc)
    per = p[:, :, :5] / rounds[:, :, None]          # clocks per round and part
    names = ["keys, argmax", "post row, barrier", "own columns", "changed columns", "second barrier"]
    print(f"# greedy kernel of {w.name}: shader clocks per round and part (sums over all {w.d_loc} rounds of a region / "
          f"{w.d_loc}), mean over the {w.B * w.P} regions; each part includes one read of the cycle counter (about 30 clocks)")
    print(f"# command: python bench.py --workload {w.name} --greedy-parts")
    print(f"{'wave':>6}" + "".join(f"{n:>20}" for n in names) + f"{'sum':>10}{'changed columns / round':>26}")
    mean = per.mean(axis=0)
    chg = (p[:, :, 6] / rounds).mean(axis=0)
    for wv in range(waves):
        print(f"{wv:>6}" + "".join(f"{mean[wv, i]:>20.0f}" for i in range(5)) + f"{mean[wv].sum():>10.0f}{chg[wv]:>26.2f}")
    busiest = per[:, :, 3].max(axis=1).mean()
    print(f"all waves: {mean.sum(axis=1).mean():.0f} clocks per round; changed columns per round over all waves "
          f"{chg.sum():.2f}; the wave with the most work in 'changed columns' spends {busiest:.0f} there (mean over regions)")


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=200)
    ap.add_argument("--warmup", type=int, default=20)
    ap.add_argument("--workload", default="sdxl1")
    ap.add_argument("--merge-regions", default="global", choices=["global", "tile"])
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--report", default=None, help="also write a per-kernel table (text) to this path")
    ap.add_argument("--report-append", action="store_true", help="append to the report instead of replacing it")
    ap.add_argument("--traffic-probe", action="store_true",
                    help="for rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE runs: three uncached layer calls and one "
                         "256 MiB device copy (the calibration kernel), nothing else")
    ap.add_argument("--greedy-rounds", action="store_true",
                    help="time the selection of this workload at several numbers of picks per region (the greedy "
                         "kernel's rounds) and print what a round costs; nothing else")
    ap.add_argument("--greedy-parts", action="store_true",
                    help="one selection of this workload through the greedy kernel that times the parts of its "
                         "rounds (regions of 256 or 64 tokens); prints clocks per round and part; nothing else")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py: this build runs on ONE GPU (no collectives, no sharding); --gpus must be 1",
              file=sys.stderr)
        sys.exit(2)

    import torch
    from paper_2509_10918_amd import binding as tb
    from paper_2509_10918_amd import synth

    w = synth.WORKLOADS[args.workload]
    if args.greedy_rounds:
        greedy_rounds(w, args.steps)
        return
    if args.greedy_parts:
        greedy_parts(w)
        return
    R = 1 if args.merge_regions == "global" else w.P
    inp = synth.make_inputs(w)
    tdt = torch.bfloat16 if w.dtype == "bf16" else torch.float32
    esize = 2 if w.dtype == "bf16" else 4

    def dev(a):
        return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to("cuda").to(tdt).contiguous()

    desc = tb.make_desc(w.B, w.H, w.W, w.C, w.tile_h, w.tile_w, w.d_loc, R, w.tau, w.dtype)
    attn = tb.toma_attn_desc(w.heads, w.head_dim, w.T_extra)
    X = dev(inp["X"])
    Xe = dev(inp["X_extra"]) if inp["X_extra"] is not None else None
    Wq, Wk, Wv = dev(inp["Wq"]), dev(inp["Wk"]), dev(inp["Wv"])
    ws = tb.alloc_workspace(desc, attn)
    idx, A, Z, amap = tb.alloc_cache(desc)
    Y = torch.empty((w.B, w.N, w.C), dtype=tdt, device="cuda")
    Ye = torch.empty((w.B, w.T_extra, w.C), dtype=tdt, device="cuda") if w.T_extra else None

    # a denoising-like sequence keeps every step's tokens resident and follows the reuse schedule
    # (destinations re-selected / weights recomputed every few steps, cached otherwise)
    seq = w.steps > 1
    if seq:
        X_steps = [dev(x) for x in inp["X_steps"]]
        plan = [0 if sel else (tb.TOMA_REUSE_IDX if rew else tb.TOMA_REUSE_A)
                for sel, rew in synth.reuse_schedule(w)]

    def call(flags, x=None):
        tb.toma_layer(desc, attn, flags, X if x is None else x, Xe, idx, A, Z, amap, Wq, Wk, Wv, None, Y, Ye, ws)

    def timed(flags, steps):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for i in range(steps):
            if seq and flags is None:
                call(plan[i % w.steps], X_steps[i % w.steps])
            else:
                call(flags)
        torch.cuda.synchronize()
        return (time.perf_counter() - t0) * 1e3 / steps     # ms per step

    if args.traffic_probe:
        src = torch.empty(256 << 20, dtype=torch.uint8, device="cuda").random_(0, 255)
        dst = torch.empty_like(src)
        for _ in range(3):
            call(0)
            dst.copy_(src)
        torch.cuda.synchronize()
        print(json.dumps({"traffic_probe": w.name, "merge_regions": R, "layer_calls": 3, "copy_bytes": 256 << 20}))
        return

    main_flags = None if seq else 0
    for _ in range(max(args.warmup, 1)):
        call(0)
    ms = timed(main_flags, args.steps)
    ms_idx = timed(tb.TOMA_REUSE_IDX, args.steps)
    ms_a = timed(tb.TOMA_REUSE_A, args.steps)
    # the same calls with the weights recomputed inside merge and unmerge instead of stored (Sec. 4.2.1)
    sub = max(args.steps // 2, 5)
    ms_rc = timed(tb.TOMA_RECOMPUTE_WEIGHTS, sub)
    ms_rc_idx = timed(tb.TOMA_RECOMPUTE_WEIGHTS | tb.TOMA_REUSE_IDX, sub)
    per_position = None
    ms_full = ms
    if seq:
        ms_full = timed(0, max(args.steps // 4, w.steps))
        # per schedule position, HIP events on the launch stream (torch's current stream)
        reps = max(args.steps // w.steps, 3)
        acc = [0.0] * w.steps
        for _ in range(reps):
            for t in range(w.steps):
                e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                e0.record()
                call(plan[t], X_steps[t])
                e1.record()
                e1.synchronize()
                acc[t] += e0.elapsed_time(e1) * 1e3
        per_position = [a / reps for a in acc]

    # per-kernel durations: the same K steps with every launch bracketed by HIP events
    tb.toma_profile_enable(True)
    timed(main_flags, args.steps)
    per_kernel = {}
    for name in tb.toma_profile_kernel_names():
        n, total = tb.toma_profile_read(name)
        if n:
            per_kernel[name] = {"launches_per_step": n / args.steps, "avg_us": total * 1e3 / n,
                                "us_per_step": total * 1e3 / args.steps}
    timed(tb.TOMA_RECOMPUTE_WEIGHTS | tb.TOMA_REUSE_IDX, sub)
    recompute_kernels = {}
    for name in ("weights_stats", "lse", "merge_recompute", "unmerge_recompute"):
        n, total = tb.toma_profile_read(name)
        if n:
            recompute_kernels[name] = total * 1e3 / n
    tb.toma_profile_enable(False)
    # products actually executed by the block-skipping merge / unmerge: counted from the block map
    call(0)
    torch.cuda.synchronize()
    exec_frac = {}
    if amap is not None:
        nblk_d, nblk_s = (w.D // R + 127) // 128, (w.N // R) // 32
        m = amap.cpu().numpy()[: w.B * R * nblk_d * nblk_s].reshape(w.B * R, nblk_d, nblk_s)
        for which, name in ((0, "merge"), (1, "unmerge")):
            tile = tb.toma_profile_map_product(desc, which)
            if tile is not None:
                exec_frac[name] = executed_fraction(m, desc, which, tile, esize)
        tile = tb.toma_profile_map_product(desc, 2)
        if tile is not None and "weights_write" in per_kernel:
            # tiles of (tile[0] sources x tile[1] destinations) that hold a nonzero block: a lower bound on
            # the tiles the write pass computes (it also computes tiles whose weights all round to zero but
            # lie less than e^-110 below their row's sum)
            spt, dpt = max(tile[0] // 32, 1), max(tile[1] // 128, 1)
            occ = m != 0
            z, db, sb = occ.shape
            pad_d, pad_s = (-db) % dpt, (-sb) % spt
            occ = np.pad(occ, ((0, 0), (0, pad_d), (0, pad_s)))
            exec_frac["weights_write"] = float(occ.reshape(z, (db + pad_d) // dpt, dpt, (sb + pad_s) // spt, spt).any(axis=(2, 4)).mean())
    screened = "weights_bounds" in per_kernel
    if screened and w.N % 32 == 0:
        # tiles of 32 sources x 16 destinations (in grid order inside their region) that hold a nonzero weight: a lower
        # bound on the tiles computed
        rank = idx.sort(dim=-1).indices + (torch.arange(w.P, device="cuda") * w.d_loc).view(1, w.P, 1)
        share = 0.0
        for b in range(w.B):
            rows = (A.view(w.B, w.D, w.N // 32, 32)[b] != 0).any(dim=-1)[rank[b].reshape(-1)]
            rows = torch.nn.functional.pad(rows, (0, 0, 0, (-w.D) % 16))
            share += float(rows.view(-1, 16, w.N // 32).any(dim=1).float().mean()) / w.B
        exec_frac["weights_write"] = share
    work = kernel_work(w, R, esize, exec_frac, int8_gram="limbs" in per_kernel, screened=screened)
    # HBM bytes per launch from rocprofv3 FETCH_SIZE / WRITE_SIZE runs of this command (profiles/)
    traffic = {}
    try:
        with open(os.path.join(ROOT, "profiles", "hbm_traffic.json")) as fh:
            rec = json.load(fh)[w.name][args.merge_regions]
        traffic = {k: t["read_bytes"] + t["written_bytes"] for k, t in rec.items()}
    except (OSError, KeyError, ValueError):
        pass
    for name, rec in per_kernel.items():
        rec.update({k: v for k, v in roofline_entry(name, work, rec["avg_us"], traffic.get(name)).items()
                    if k != "kernel"})
    if "merge" in exec_frac:
        for name in ("merge", "unmerge", "weights_write"):
            if name in per_kernel and name in exec_frac:
                per_kernel[name]["executed_share_of_k_steps" if name != "weights_write" else "executed_share_of_tiles_lower_bound"] = exec_frac[name]
    dominant = max(per_kernel, key=lambda k: per_kernel[k]["us_per_step"])
    roofline = roofline_entry(dominant, work, per_kernel[dominant]["avg_us"], traffic.get(dominant))
    roofline["avg_us"] = per_kernel[dominant]["avg_us"]
    roofline["traffic_source"] = "profiles/hbm_traffic.json (rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE runs of this command)"
    mfma_k = [k for k in per_kernel if per_kernel[k]["bound"] == "mfma" and k not in ("gram", "limbs")]
    mfma_flops = sum(work[k]["amount"] * per_kernel[k]["launches_per_step"] for k in mfma_k)
    mfma_equiv = sum(work[k].get("equiv", work[k]["amount"]) * per_kernel[k]["launches_per_step"] for k in mfma_k)
    mfma_us = sum(per_kernel[k]["us_per_step"] for k in mfma_k)
    mfma_us += per_kernel.get("split_finish", {"us_per_step": 0.0})["us_per_step"]   # part of the split products
    mm_peak = PEAK["bf16" if w.dtype == "bf16" else "f32"]

    out = {
        "metric": METRIC, "value": ms * 1e3, "unit": "us", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": ms, "higher_is_better": False, "scaling": "weak",
        "vs_baseline": None, "dtype": w.dtype, "data": "synthetic",
        "config": {"workload": f"{w.name}: B={w.B}, {w.H}x{w.W} tokens (N={w.N}), C={w.C}, "
                               f"{w.tile_h}x{w.tile_w} regions (P={w.P}), keep {w.keep:g} (D={w.D}), tau={w.tau}, "
                               f"{w.heads} heads x {w.head_dim}, extra tokens {w.T_extra}, "
                               f"merge_regions={R} ({args.merge_regions})",
                   "call": ("toma_layer along the reuse schedule (amortised over the sequence)" if seq else
                            "toma_layer, nothing cached (select + weights + merge + attention + unmerge)")},
        "roofline": roofline,
        "us_idx_cached": ms_idx * 1e3, "us_idx_and_weights_cached": ms_a * 1e3,
        "recomputed_weights": {"us_nothing_cached": ms_rc * 1e3, "us_idx_cached": ms_rc_idx * 1e3,
                               "kernel_avg_us": recompute_kernels,
                               "note": "toma_layer with TOMA_RECOMPUTE_WEIGHTS: no A is written or read; compare "
                                       "us_idx_cached here with the stored-weights us_idx_cached"},
        "sequence": None if not seq else {
            "schedule": ["select+weights" if f == 0 else ("weights" if f == tb.TOMA_REUSE_IDX else "cached") for f in plan],
            "us_per_position": per_position, "us_amortised": ms * 1e3, "us_nothing_cached": ms_full * 1e3},
        "mfma_stages": {"tflops": mfma_flops / (mfma_us * 1e-6) / 1e12 if mfma_us else None,
                        "frac_of_peak": (mfma_flops / (mfma_us * 1e-6) / 1e12) / mm_peak if mfma_us else None,
                        "equiv_dense_tflops": mfma_equiv / (mfma_us * 1e-6) / 1e12 if mfma_us else None,
                        "equiv_dense_frac_of_peak": (mfma_equiv / (mfma_us * 1e-6) / 1e12) / mm_peak if mfma_us else None,
                        "us_per_step": mfma_us,
                        "note": "weights, merge, QKV, attention, unmerge; tflops counts the products executed "
                                "(merge / unmerge skip the K steps whose blocks of A are empty), equiv_dense the full ones"},
        "kernels": per_kernel,
    }

    # the two unmerges of Sec. 4.2.2 side by side (App. E.4 compares them end to end): transpose against
    # Moore-Penrose, where the latter's region size limit allows it
    if R == w.P and w.d_loc <= 128:
        O_in = torch.randn((w.B, w.D + w.T_extra, w.C), device="cuda").to(tdt)
        reps = max(args.steps // 4, 10)

        def time_it(fn):
            fn()
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(reps):
                fn()
            torch.cuda.synchronize()
            return (time.perf_counter() - t0) * 1e6 / reps

        t_us = time_it(lambda: tb.toma_unmerge(desc, A, Z, amap, O_in, Y, ws))
        tb.toma_profile_enable(True)
        p_us = time_it(lambda: tb.toma_unmerge_pinv(desc, A, Z, O_in, 1e-2, Y, ws))
        parts = {}
        for name in ("pinv_eig", "pinv_apply"):
            n, total = tb.toma_profile_read(name)
            parts[name + "_us"] = total * 1e3 / max(n, 1)
        tb.toma_profile_enable(False)
        out["unmerge_variants"] = {"transpose_us": t_us, "pseudo_inverse_us": p_us, "rcond": 1e-2, **parts,
                                   "context": "paper, SDXL end to end: 4.8 s / image with the transpose, 10.1 s with the "
                                              "pseudo-inverse (App. E.4, hardware not stated)"}

    if not args.no_cpu_baseline:
        from oracle import toma_oracle as orc
        f64 = lambda a: None if a is None else np.asarray(a, dtype=np.float64)
        # bounded sample: the whole call when it is a few seconds of CPU work, else one sample of the
        # batch in region-local mode (stated in the record)
        heavy = w.N > 8192
        ob = 1 if heavy else w.B
        oR = w.P if heavy else R
        od = orc.make_desc(ob, w.H, w.W, w.C, w.tile_h, w.tile_w, w.d_loc, oR, w.tau)
        ox = f64(inp["X"][:ob])
        oxe = None if inp["X_extra"] is None else f64(inp["X_extra"][:ob])
        t0 = time.perf_counter()
        ref = orc.layer(od, ox, f64(inp["Wq"]), f64(inp["Wk"]), f64(inp["Wv"]), heads=w.heads, Xe=oxe)
        cpu_s = time.perf_counter() - t0
        sample = ("1 full layer call of the same workload (all samples, all regions)" if not heavy else
                  f"1 full layer call on sample 0 only (B=1 of {w.B}), region-local merge, step 0")
        out["cpu_baseline"] = {"value": cpu_s * 1e6, "unit": "us", "cores": orc.threads(), "kind": "oracle",
                               "sample": sample}
        # parity of this very run: picks against the oracle (whole workload, or sample 0 of a heavy one),
        # the library's own near-tie report, and the oracle's decision grid against plain fp64
        gain_d = torch.empty((w.B, w.P, w.d_loc), dtype=torch.float32, device="cuda")
        gap_d = torch.empty_like(gain_d)
        idx_d = torch.empty((w.B, w.P, w.d_loc), dtype=torch.int32, device="cuda")
        tb.toma_select(desc, X, idx_d, gain_d, gap_d, ws)
        torch.cuda.synchronize()
        idx_gpu = idx_d.cpu().numpy()[:ob]
        gain_g, gap_g = gain_d.cpu().numpy().astype(np.float64), gap_d.cpu().numpy().astype(np.float64)
        rel_gap = ref["gap"] / np.maximum(ref["gain"], 1e-30)
        # plain definition: similarities not rounded to the grid (sim_bits = 0)
        od0 = orc.make_desc(ob, w.H, w.W, w.C, w.tile_h, w.tile_w, w.d_loc, oR, w.tau, sim_bits=0)
        idx0, gain0, gap0 = orc.select(od0, ox)
        rel0 = gap0 / np.maximum(gain0, 1e-30)
        _, _, token_of = orc.region_map(w.H, w.W, w.tile_h, w.tile_w)
        differing = unexcused = 0
        worst = 0.0
        for b in range(ob):
            for p in range(w.P):
                if np.array_equal(idx_gpu[b, p], idx0[b, p]):
                    continue
                differing += 1
                first = int(np.nonzero(idx_gpu[b, p] != idx0[b, p])[0][0])
                unexcused += int(not rel0[b, p, first] < 1e-6)
                loc = {int(t): l for l, t in enumerate(token_of[p])}
                picks = np.array([loc[int(t)] for t in idx_gpu[b, p]], np.int32)
                _, deficit, _ = orc.check_picks(orc.cosine(ox[b, token_of[p]]), picks)
                worst = max(worst, float(deficit.max()))
        out["parity"] = {
            "scope": "whole workload" if not heavy else "sample 0",
            "regions_with_different_picks": int((~np.all(idx_gpu == ref["idx"], axis=2)).sum()),
            "near_tie_steps_reported_by_the_library": int((gap_g[..., :-1] < 1e-6 * np.maximum(gain_g[..., :-1], 1e-30)).sum()),
            "exact_tie_steps_reported_by_the_library": int((gap_g[..., :-1] == 0).sum()),
            "near_tie_steps_oracle": int((rel_gap[..., :-1] < 1e-6).sum()),
            "exact_tie_steps_oracle": int((ref["gap"][..., :-1] == 0).sum()),
            "picks_vs_ungridded_oracle": {"regions_differing": differing, "unexcused": unexcused, "worst_deficit": worst,
                                          "note": "plain fp64 similarities break mathematically tied candidates by "
                                                  "rounding noise, the 2^-30 grid by the lowest index; unexcused = first "
                                                  "differences not at a step plain fp64 flags as a near tie (< 1e-6); "
                                                  "worst_deficit = how far below the best candidate, judged by plain "
                                                  "similarities, any pick of the library lies (relative)"},
            "clamped_destinations": int(ref["clamps"]),
        }
        if not heavy:
            call(0)
            torch.cuda.synchronize()
            y = Y.to(torch.float64).cpu().numpy()
            out["parity"]["max_rel_err_Y"] = float(np.abs(y - ref["Y"]).max() / np.abs(ref["Y"]).max())
    out["context"] = {"paper": "merge 38.8 us / unmerge 40.5 us at N=1024 on RTX6000 (Table 6); SDXL/Flux "
                               "end-to-end latency -24% / -23% (abstract); other hardware, context only"}
    if args.report:
        with open(args.report, "a" if args.report_append else "w") as fh:
            cb = out.get("cpu_baseline")
            fh.write(f"## {out['config']['workload']}\n"
                     f"command: python bench.py --workload {w.name} --merge-regions {args.merge_regions} --steps {args.steps} "
                     f"--warmup {args.warmup}\n"
                     f"us per layer call: nothing cached {ms_full * 1e3 if seq else ms * 1e3:.1f}; idx cached {ms_idx * 1e3:.1f}; "
                     f"idx + weights cached {ms_a * 1e3:.1f}" + (f"; along the reuse schedule {ms * 1e3:.1f}" if seq else "") + "\n")
            fh.write(f"with recomputed weights (no stored A): nothing cached {ms_rc * 1e3:.1f}; idx cached {ms_rc_idx * 1e3:.1f} "
                     f"(" + ", ".join(f"{k} {v:.1f}" for k, v in recompute_kernels.items()) + ")\n")
            if "unmerge_variants" in out:
                uv = out["unmerge_variants"]
                fh.write(f"unmerge alone: transpose {uv['transpose_us']:.1f} us, Moore-Penrose (rcond {uv['rcond']:g}) "
                         f"{uv['pseudo_inverse_us']:.1f} us (eigen-decomposition {uv['pinv_eig_us']:.1f}, apply {uv['pinv_apply_us']:.1f})\n")
            if cb:
                fh.write(f"fp64 oracle on {cb['cores']} host threads: {cb['value'] / 1e6:.2f} s ({cb['sample']})\n")
            ms_ = out["mfma_stages"]
            if ms_["tflops"]:
                fh.write(f"matrix-core stages: {ms_['tflops']:.0f} TFLOP/s executed = {ms_['frac_of_peak']:.3f} of peak "
                         f"({ms_['equiv_dense_tflops']:.0f} counting skipped blocks as done) over {ms_['us_per_step']:.1f} us\n")
            fh.write(f"{'kernel':<15}{'launch/step':>12}{'avg us':>10}{'achieved':>12}{'unit':>9}{'frac':>8}{'equiv frac':>12}{'HBM MB':>9}\n")
            for k, r in sorted(per_kernel.items(), key=lambda kv: -kv[1]["us_per_step"]):
                eq = f"{r['equiv_frac']:.3f}" if "equiv_frac" in r else "-"
                tr = f"{r['traffic'] / 1e6:.1f}" if r.get("traffic") else "-"
                fh.write(f"{k:<15}{r['launches_per_step']:>12.1f}{r['avg_us']:>10.2f}{r['achieved']:>12.2f}"
                         f"{r['unit']:>9}{r['frac']:>8.3f}{eq:>12}{tr:>9}\n")
            fh.write("\n")
    print(json.dumps(out))


if __name__ == "__main__":
    main()

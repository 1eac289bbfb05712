#!/usr/bin/env python3
"""Benchmark of the ECC hot path on one MI355X.

A step is one ecc_hard call (batch-global range, thresholds, coefficient sweep, histogram,
merge, scan) over workload C2: a batch of 16 2D 4096x4096 float32 smoothed Gaussian random
fields, 1024 equal-width bins over the batch-global [min, max] found on the device.  Inputs are
resident in HBM before the timed region.  The same run also times, as `extra` fields of the one
JSON line, the other four workloads (C4 3D 512^3 float32, C1 256^2 uint8, C3 256^3 uint16, C5
soft forward + backward), each with a roofline entry of its own and -- for the three that fit
the 256 MB Infinity Cache -- a cold variant that rotates over copies totalling more than 256 MB;
the hard path with the range supplied; directional curves; the grid sizes of the paper's
Tables 1-2; and the CPU oracle on the host cores (a baseline, not the target).

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--quick]
    python bench.py --only c1|c2|c2r|c3|c4|c4r|c5|dir|soft3d|scan|step|sizes|batches|calib    one workload, no JSON (profiling runs)

Counter-based figures (HBM traffic, VALU / LDS instruction counts) cannot be taken inside this
process; they come from rocprofv3 runs of `bench.py --only <workload>` summarised by
`python -m paper_2510_20271_amd.profile_summary` into profiles/counters.json, which this script
reads (null when the file has no entry).
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0       # MI355X published HBM3E peak
VALU_PEAK_TLANEOPS = 39.32  # 256 CUs x 4 SIMDs x 16 lanes x 2.4 GHz: vector lane-operations per second (x 1e12)
CACHE_MB = 256              # Infinity Cache; cold variants rotate over more than this


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def time_steps(fn, steps, warmup):
    import torch
    for _ in range(warmup):
        fn()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        fn()
    torch.cuda.synchronize()
    return (time.perf_counter() - t0) / steps * 1e3  # ms per step


def kernel_ms(api, fn, steps, warmup):
    """(mean duration of the call's dominant kernel -- HIP events recorded by the library on the call's
    stream --, wall time per call, launches measured) over the same `steps` calls."""
    import torch
    for _ in range(warmup):
        fn()
    torch.cuda.synchronize()
    api.ecc_profile_begin(steps)
    t0 = time.perf_counter()
    for _ in range(steps):
        fn()
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) / steps * 1e3
    k, n = api.ecc_profile_end()
    return k, ms, n


def load_counters():
    path = os.path.join(ROOT, "profiles", "counters.json")
    if os.path.exists(path):
        return json.load(open(path)).get("kernels", {})
    return {}


def roofline_hbm(alg_bytes, k_ms, kernel, counters, note=None):
    achieved = alg_bytes / (k_ms * 1e-3) / 1e9
    c = counters or {}
    traffic = None
    if "fetch_bytes" in c and "write_bytes" in c:
        traffic = int(c["fetch_bytes"] + c["write_bytes"])
    r = {"bound": "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
         "frac": round(achieved / HBM_PEAK_GBS, 4), "traffic": traffic, "kernel": kernel, "kernel_ms": round(k_ms, 4),
         "algorithmic_bytes_per_launch": int(alg_bytes)}
    if traffic is not None:
        r["traffic_source"] = "rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE (profiles/counters.json)"
    if "SQ_INSTS_VALU" in c:
        r["valu_lane_ops_per_launch"] = int(c["SQ_INSTS_VALU"] * 64)
        r["valu_frac_of_peak"] = round(c["SQ_INSTS_VALU"] * 64 / (k_ms * 1e-3) / 1e12 / VALU_PEAK_TLANEOPS, 4)
    if note:
        r["note"] = note
    return r


def roofline_alu(k_ms, kernel, counters, alg_bytes, note):
    """A kernel nearer to the vector units' limit than to the memory's: achieved = lane-operations issued (SQ_INSTS_VALU x 64, from
    the rocprofv3 run) per second of the kernel's duration measured here."""
    c = counters or {}
    if "SQ_INSTS_VALU" not in c:
        return {"bound": "alu", "achieved": None, "peak": VALU_PEAK_TLANEOPS, "unit": "Tlane-op/s", "frac": None,
                "traffic": None, "kernel": kernel, "kernel_ms": round(k_ms, 4), "note": note}
    ach = c["SQ_INSTS_VALU"] * 64 / (k_ms * 1e-3) / 1e12
    r = {"bound": "alu", "achieved": round(ach, 2), "peak": VALU_PEAK_TLANEOPS, "unit": "Tlane-op/s",
         "frac": round(ach / VALU_PEAK_TLANEOPS, 4),
         "traffic": int(c["fetch_bytes"] + c["write_bytes"]) if "fetch_bytes" in c else None, "kernel": kernel,
         "kernel_ms": round(k_ms, 4), "algorithmic_bytes_per_launch": int(alg_bytes),
         "hbm_frac_by_algorithmic_bytes": round(alg_bytes / (k_ms * 1e-3) / 1e9 / HBM_PEAK_GBS, 4), "note": note}
    for k in ("SQ_INSTS_LDS", "SQ_LDS_BANK_CONFLICT", "SQ_ACTIVE_INST_LDS"):
        if k in c:
            r[k] = int(c[k])
    return r


def step_host_times(args, torch, synth):
    """A training step of the layer (32 x 512^2, 128 thresholds; input, thresholds and angle learned): the step among others,
    and how long the host takes to put a forward and a backward pass into an idle device's queue."""
    from paper_2510_20271_amd.layer import SoftECCLayer
    x = torch.from_numpy(synth.config_c5()).cuda()
    m = SoftECCLayer(2, 128, float(x.min()), float(x.max()), alpha=0.01, lam=20.0, theta=[0.3]).cuda()
    x.requires_grad_()
    g = torch.ones(32, 128, device="cuda")
    host = [0.0, 0.0]

    def step():
        t0 = time.perf_counter()
        chi = m(x)
        t1 = time.perf_counter()
        torch.autograd.grad(chi, [x, m.tau, m.theta], g)
        host[0], host[1] = host[0] + t1 - t0, host[1] + time.perf_counter() - t1

    for _ in range(args.warmup):
        step()
    n = 10 * args.steps
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(n):
        step()
    torch.cuda.synchronize()
    among = (time.perf_counter() - t0) / n * 1e6
    host[:] = 0.0, 0.0
    for _ in range(n):
        step()
        torch.cuda.synchronize()
    log(f"[bench] step 32 x 512^2: {among:.1f} us; host alone: forward {host[0] / n * 1e6:.1f}, backward {host[1] / n * 1e6:.1f} us")


# "New" kernel times of the paper's Tables 1 and 2 (ms, one RTX A6000; dtype, bins and timing
# method not stated there): context beside the sizes below, not a target.
PAPER_MS = {(128, 128): 0.0165, (256, 256): 0.0174, (512, 512): 0.021, (1024, 1024): 0.032,
            (2048, 2048): 0.11, (4096, 4096): 0.408, (8192, 8192): 1.6, (128, 128, 128): 0.1,
            (256, 256, 256): 0.71, (512, 512, 512): 5.61, (1024, 1024, 1024): 48.47}


def size_rows(args, np, torch, api, synth, field_2d=None, field_3d=None):
    """One float32 smoothed random field of each size of the paper's Tables 1-2, 1024 bins over the range
    found on the device (the whole hot path per call).  The generator smooths with wrap-around, so a
    field tiles seamlessly: 8192^2 is a 4096^2 field tiled 2 x 2, 1024^3 a 512^3 field tiled 2 x 2 x 2
    (exact duplicates across tiles are ties like any other)."""
    rows = []
    for shape in PAPER_MS:
        nd = len(shape)
        if shape == (8192, 8192):
            X = np.tile(field_2d if field_2d is not None else synth.grf((4096, 4096), 4.0, 4242), (2, 2))
        elif shape == (4096, 4096) and field_2d is not None:
            X = field_2d
        elif shape == (1024, 1024, 1024):
            X = np.tile(field_3d if field_3d is not None else synth.grf((512, 512, 512), 3.0, 4242), (2, 2, 2))
        elif shape == (512, 512, 512) and field_3d is not None:
            X = field_3d
        else:
            X = synth.grf(shape, 4.0 if nd == 2 else 3.0, 4242)
        g = torch.from_numpy(np.ascontiguousarray(X)[None]).cuda()
        ws = torch.empty(api.ecc_workspace_bytes(shape, 1, 1024), dtype=torch.uint8, device="cuda")
        cv = torch.empty((1, 1024), dtype=torch.int64, device="cuda")
        ms = time_steps(lambda: api.ecc_hard(g, nd, 1024, curve=cv, workspace=ws), args.steps, args.warmup)
        n = int(np.prod(shape))
        rows.append({"shape": "x".join(map(str, shape)), "ms": round(ms, 4), "gvoxel_per_s": round(n / ms / 1e6, 1),
                     "curve_ends_at_one": bool(int(cv[0, -1]) == 1), "paper_ms_rtx_a6000": PAPER_MS[shape]})
        log(f"[bench] size {rows[-1]['shape']:>14}: {ms:8.4f} ms  {rows[-1]['gvoxel_per_s']:8.1f} Gvoxel/s"
            f"   (paper, RTX A6000: {PAPER_MS[shape]} ms)")
        del g, ws, cv, X
        torch.cuda.empty_cache()
    return rows


def batch_rows(args, np, torch, api, synth):
    """Batches of small float32 images and sets of directions (what a topological layer or a directional
    transform calls with; not a workload of the paper): whole calls, 256 bins, range found on the device."""
    rows = []
    cases = [("hard", 1024, (28, 28), 0), ("hard", 256, (64, 64), 0), ("hard", 256, (256, 256), 0), ("hard", 32, (512, 512), 0),
             ("hard", 16, (1024, 1024), 0), ("hard", 16, (64, 64, 64), 0), ("dir", 1, (256, 256), 64), ("dir", 8, (128, 128), 32)]
    for kind, B, shape, ndir in cases:
        nd = len(shape)
        base = np.stack([synth.grf(shape, 2.0, 900 + i) for i in range(min(B, 4))])
        g = torch.from_numpy(np.ascontiguousarray(base[np.arange(B) % base.shape[0]])).cuda()
        rows_out = B * max(ndir, 1)
        cv = torch.empty((rows_out, 256) if not ndir else (ndir, B, 256), dtype=torch.int64, device="cuda")
        if ndir:
            U = np.random.default_rng(5).standard_normal((ndir, nd)).astype(np.float32)
            u = torch.from_numpy(U / np.linalg.norm(U, axis=1, keepdims=True)).cuda()
            ws = torch.empty(api.ecc_workspace_bytes_dir(shape, B, ndir, 256), dtype=torch.uint8, device="cuda")
            step = lambda: api.ecc_hard_dir(g, nd, u, 1e-3, 256, curve=cv, workspace=ws)
        else:
            ws = torch.empty(api.ecc_workspace_bytes(shape, B, 256), dtype=torch.uint8, device="cuda")
            step = lambda: api.ecc_hard(g, nd, 256, curve=cv, workspace=ws)
        ms = time_steps(step, args.steps, args.warmup)
        n = int(np.prod(shape)) * rows_out
        name = (f"{ndir} directions x " if ndir else "") + f"{B} x " + "x".join(map(str, shape))
        rows.append({"workload": name, "ms": round(ms, 4), "gvoxel_per_s": round(n / ms / 1e6, 1)})
        log(f"[bench] batch {name:>32}: {ms:8.4f} ms  {rows[-1]['gvoxel_per_s']:8.1f} Gvoxel/s")
        del g, ws, cv
        torch.cuda.empty_cache()
    return rows


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--quick", action="store_true", help="C2 only: skip the other workloads and the CPU baseline")
    ap.add_argument("--only", default="", help="profiling aid: run one of c1, c2, c2r, c3, c4, c4r, c5, dir, soft3d, sizes, "
                                               "batches, scan (an int16 volume over a known range), step (a training "
                                               "step of the layer), calib (a plain 1 GiB copy); no JSON")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py: this build runs on ONE GPU; --gpus must be 1 (the path shards by batch item / "
              "z-slab with one all-reduce of the histogram, which this single-GPU build does not include)", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch
    from paper_2510_20271_amd import _lib, api, synth

    _lib.load()  # fails loudly when the HIP library is missing
    assert torch.cuda.is_available(), "bench.py needs a GPU"
    torch.cuda.set_device(0)
    only = args.only
    full = only == "" and not args.quick
    counters = load_counters()
    BINS = 1024
    extra = {}
    rooflines = {}

    def want(*names):
        return full or only in names

    if only == "calib":
        # counter calibration: a plain device copy of exactly 1 GiB read + 1 GiB written per launch
        src = torch.empty(1 << 28, dtype=torch.float32, device="cuda").normal_()
        dst = torch.empty_like(src)
        for _ in range(args.steps):
            dst.copy_(src)
        torch.cuda.synchronize()
        log("[bench] calib: copied 1 GiB x %d" % args.steps)
        return

    def rotating(make_copy, one_bytes):
        """Copies of an input totalling more than the Infinity Cache, for the cold variants."""
        n = int(CACHE_MB * (1 << 20) * 1.05 // one_bytes) + 1
        return [make_copy() for _ in range(n)]

    # ---------------- C2: the headline workload --------------------------------
    field_2d = None
    if only in ("", "c2", "c2r"):
        t0 = time.perf_counter()
        X2 = synth.config_c2()
        log(f"[bench] generated C2 {X2.shape} in {time.perf_counter() - t0:.1f}s")
        g2 = torch.from_numpy(X2).cuda()
        ws2 = torch.empty(api.ecc_workspace_bytes(X2.shape[1:], X2.shape[0], BINS), dtype=torch.uint8, device="cuda")
        curve2 = torch.empty((X2.shape[0], BINS), dtype=torch.int64, device="cuda")
        nvox = X2.size
        alg_bytes = 4.0 * nvox  # one float32 read per vertex per sweep launch
        if only != "c2r":
            sweep_ms, ms, nl = kernel_ms(api, lambda: api.ecc_hard(g2, 2, BINS, curve=curve2, workspace=ws2), args.steps,
                                         args.warmup)
            value = nvox / (ms * 1e-3) / 1e9
            roofline = roofline_hbm(alg_bytes, sweep_ms, "sweep2d_list_kernel (coefficient sweep + range + "
                                    "critical-vertex lists)", counters.get("c2"))
            roofline["launches_timed"] = nl
            roofline["whole_call_hbm_frac"] = round(alg_bytes / (ms * 1e-3) / 1e9 / HBM_PEAK_GBS, 4)
            log(f"[bench] C2: {ms:.4f} ms/step, {value:.1f} Gvoxel/s, sweep kernel {sweep_ms:.4f} ms")
        if full or only == "c2r":
            rng2 = (float(X2.min()), float(X2.max()))
            k_r, ms_r, _ = kernel_ms(api, lambda: api.ecc_hard(g2, 2, BINS, range=rng2, curve=curve2, workspace=ws2),
                                     args.steps, args.warmup)
            extra["c2_range_supplied"] = {"ms_per_step": round(ms_r, 4), "gvoxel_per_s": round(nvox / ms_r / 1e6, 1)}
            rooflines["c2_range_supplied"] = roofline_hbm(alg_bytes, k_r, "sweep2d_kernel (histogram mode)",
                                                          counters.get("c2r"))
            log(f"[bench] C2, range supplied: {ms_r:.4f} ms/step, sweep kernel {k_r:.4f} ms")
        if full:
            # CPU oracle on the same batch, as it stands
            from oracle import ecc_oracle as O
            from oracle import ecc_oracle_c as OC
            api.ecc_hard(g2, 2, BINS, curve=curve2, workspace=ws2)
            nitem = X2.shape[0]  # the whole batch: a couple of seconds on the host cores
            t0 = time.perf_counter()
            lo, hi = X2.min(), X2.max()
            ref = OC.ecc_hard_batch(X2[:nitem], O.thresholds_equal_width(lo, hi, BINS))
            dt = time.perf_counter() - t0
            cpu = {"value": round(nitem * X2[0].size / dt / 1e9, 4), "unit": "Gvoxel/s", "cores": OC.threads(),
                   "kind": "oracle", "sample": f"the whole C2 batch, {nitem} items, thresholds from its min/max "
                   f"({dt:.1f} s of host time)"}
            extra["c2_matches_oracle"] = bool(np.array_equal(curve2.cpu().numpy(), ref))
            # the same batch as float16
            g2h = g2.half()
            wsh = torch.empty(api.ecc_workspace_bytes_dtype(X2.shape[1:], X2.shape[0], api.ECC_F16, BINS),
                              dtype=torch.uint8, device="cuda")
            ms_h = time_steps(lambda: api.ecc_hard(g2h, 2, BINS, curve=curve2, workspace=wsh), args.steps, args.warmup)
            extra["c2_float16"] = {"ms_per_step": round(ms_h, 4), "gvoxel_per_s": round(nvox / ms_h / 1e6, 1)}
            log(f"[bench] C2 as float16: {ms_h:.4f} ms/step")
            del g2h, wsh
            field_2d = X2[0].copy()
        if only in ("c2", "c2r"):
            return
        del g2, ws2, X2
        torch.cuda.empty_cache()

    # ---------------- C4: 3D 512^3 float32 -------------------------------------
    field_3d = None
    if want("c4", "c4r"):
        t0 = time.perf_counter()
        X4 = synth.config_c4()[None]
        log(f"[bench] generated C4 {X4.shape} in {time.perf_counter() - t0:.1f}s")
        g4 = torch.from_numpy(X4).cuda()
        ws4 = torch.empty(api.ecc_workspace_bytes(X4.shape[1:], 1, BINS), dtype=torch.uint8, device="cuda")
        curve4 = torch.empty((1, BINS), dtype=torch.int64, device="cuda")
        b4 = 4.0 * X4.size
        c4 = {"workload": "C4: 3D 512^3 float32 GRF sigma=3, 1024 bins"}
        if only != "c4r":
            sweep4, ms4, _ = kernel_ms(api, lambda: api.ecc_hard(g4, 3, BINS, curve=curve4, workspace=ws4), args.steps,
                                       args.warmup)
            c4.update({"ms_per_step_auto_range": round(ms4, 4), "gvoxel_per_s_auto_range": round(X4.size / ms4 / 1e6, 1)})
            rooflines["c4"] = roofline_hbm(b4, sweep4, "sweep3d_list_kernel (coefficient sweep + range + lists)",
                                           counters.get("c4"), note="target of this build: frac >= 0.60; not met: the kernel "
                                           "is bound by vector instruction issue before it is bound by memory (see "
                                           "valu_frac_of_peak)")
            rooflines["c4"]["whole_call_hbm_frac"] = round(b4 / (ms4 * 1e-3) / 1e9 / HBM_PEAK_GBS, 4)
            log(f"[bench] C4: {ms4:.4f} ms/step, sweep kernel {sweep4:.4f} ms")
        if full or only == "c4r":
            rng4 = (float(X4.min()), float(X4.max()))
            k4r, ms4r, _ = kernel_ms(api, lambda: api.ecc_hard(g4, 3, BINS, range=rng4, curve=curve4, workspace=ws4),
                                     args.steps, args.warmup)
            c4.update({"ms_per_step_range_supplied": round(ms4r, 4),
                       "gvoxel_per_s_range_supplied": round(X4.size / ms4r / 1e6, 1)})
            rooflines["c4_range_supplied"] = roofline_hbm(b4, k4r, "sweep3d_kernel (histogram mode)", counters.get("c4r"))
            log(f"[bench] C4, range supplied: {ms4r:.4f} ms/step, sweep kernel {k4r:.4f} ms")
        extra["c4"] = c4
        if only in ("c4", "c4r"):
            return
        field_3d = X4[0]
        del g4, ws4
        torch.cuda.empty_cache()

    # ---------------- C1 / C3: integer levels, one bin per level ----------------
    if want("c1", "c3"):
        for name, nd, bins in (("c1", 2, 256), ("c3", 3, 4096)):
            if only and only != name:
                continue
            X = (synth.config_c1() if name == "c1" else synth.config_c3())[None]
            if X.dtype == np.uint16:
                gi = torch.from_numpy(X.view(np.int16)).cuda().view(torch.uint16)
            else:
                gi = torch.from_numpy(X).cuda()
            wsi = torch.empty(api.ecc_workspace_bytes(X.shape[1:], 1, bins), dtype=torch.uint8, device="cuda")
            cvi = torch.empty((1, bins), dtype=torch.int64, device="cuda")
            swi, msi, _ = kernel_ms(api, lambda: api.ecc_hard(gi, nd, bins, curve=cvi, workspace=wsi), args.steps, args.warmup)
            # cold: rotate over copies totalling more than the Infinity Cache
            copies = rotating(lambda: gi.clone(), X.nbytes)
            it = [0]

            def cold():
                it[0] = (it[0] + 1) % len(copies)
                api.ecc_hard(copies[it[0]], nd, bins, curve=cvi, workspace=wsi)
            ncold = max(args.steps, 2 * len(copies)) if name == "c3" else 512
            swc, msc, _ = kernel_ms(api, cold, ncold, len(copies) if name == "c3" else 64)
            extra[name] = {"workload": {"c1": "C1: 2D 256^2 uint8 i.i.d., 256 levels (launch-latency bound, 2 launches)",
                                        "c3": "C3: 3D 256^3 uint16 i.i.d., 4096 levels"}[name],
                           "us_per_step": round(msi * 1e3, 2), "sweep_kernel_us": round(swi * 1e3, 2),
                           "gvoxel_per_s": round(X.size / msi / 1e6, 2),
                           "cold_us_per_step": round(msc * 1e3, 2), "cold_sweep_kernel_us": round(swc * 1e3, 2),
                           "cold_copies": len(copies)}
            if name == "c3":
                rooflines["c3"] = roofline_alu(swi, "sweep3dp_kernel<uint16> (levels, LDS histogram)", counters.get("c3"),
                                               X.nbytes, "2 bytes per vertex: HBM is idle by construction; half of the vector "
                                               "units' issue slots (stencil, then the 60 % of the vertices that are "
                                               "critical, binned from registers), the rest the march of three waves a "
                                               "SIMD, LDS updates and the blocks' histograms")
                rooflines["c3"]["cold_kernel_ms"] = round(swc, 4)
            else:
                rooflines["c1"] = roofline_hbm(float(X.nbytes), swi, "sweep_generic_kernel<uint8> (one thread per vertex)",
                                               counters.get("c1"), note="64 KiB input: the call is two dependent "
                                               "launches of a few microseconds each; a fraction of HBM peak says nothing here")
                rooflines["c1"]["cold_kernel_ms"] = round(swc, 4)
                rooflines["c1"]["launches_per_call"] = 2
            log(f"[bench] {name}: {msi * 1e3:.1f} us/step, sweep {swi * 1e3:.1f} us; cold {msc * 1e3:.1f} us/step, "
                f"sweep {swc * 1e3:.1f} us ({len(copies)} copies)")
            del gi, copies
            torch.cuda.empty_cache()
        if only in ("c1", "c3"):
            return

    # ---------------- directional curves: 16 directions of one 4096^2 field --------
    if want("dir"):
        Xd = (field_2d if field_2d is not None else synth.grf((4096, 4096), 4.0, 2002))[None]
        th = np.linspace(0.0, np.pi, 16, endpoint=False)
        Ud = np.stack([np.cos(th), np.sin(th)], 1).astype(np.float32)
        gd, ud = torch.from_numpy(Xd).cuda(), torch.from_numpy(Ud).cuda()
        wsd = torch.empty(api.ecc_workspace_bytes_dir(Xd.shape[1:], 1, 16, BINS), dtype=torch.uint8, device="cuda")
        cvd = torch.empty((16, 1, BINS), dtype=torch.int64, device="cuda")
        swd, msd, _ = kernel_ms(api, lambda: api.ecc_hard_dir(gd, 2, ud, 1e-4, BINS, curve=cvd, workspace=wsd), args.steps,
                                args.warmup)
        extra["directional"] = {"workload": "16 directions x one 2D 4096^2 float32 GRF (alpha = 1e-4 per pixel), 1024 "
                                            "bins over the range of all tilted fields, found on the device",
                                "ms_per_step": round(msd, 4), "sweep_kernel_ms": round(swd, 4),
                                "gvoxel_per_s": round(16 * Xd.size / msd / 1e6, 1),
                                "note": "the field (64 MiB) is read once per direction; re-reads are served by "
                                        "the L2 / Infinity Cache, so vertices/s may pass the HBM roofline of a "
                                        "single read"}
        log(f"[bench] directional: {msd:.4f} ms/step (16 x 4096^2), sweep kernel {swd:.4f} ms")
        del gd, Xd
        torch.cuda.empty_cache()
        if only == "dir":
            return

    # ---------------- C5: soft forward + backward -------------------------------
    if want("c5"):
        X5 = synth.config_c5()
        p = synth.soft_params_c5(X5)
        T = len(p["tau"])
        B5 = X5.shape[0]
        g5 = torch.from_numpy(X5).cuda()
        u5, tau5 = torch.from_numpy(p["u"]).cuda(), torch.from_numpy(p["tau"]).cuda()
        G5 = torch.from_numpy(synth.upstream_grad(B5, T)).cuda()
        ws5 = torch.empty(api.ecc_workspace_bytes(X5.shape[1:], B5, T), dtype=torch.uint8, device="cuda")
        st5 = torch.empty(api.ecc_soft_state_bytes(X5.shape[1:], B5), dtype=torch.uint8, device="cuda")
        chi = torch.empty((B5, T), dtype=torch.float32, device="cuda")
        gx = torch.empty_like(g5)
        dt_ = torch.empty_like(chi)
        du_ = torch.empty((B5, T, 2), dtype=torch.float32, device="cuda")
        a5 = (2, u5, p["alpha"], tau5, p["lam"])

        def fwd(g=g5):
            api.ecc_soft_fwd(g, *a5, chi=chi, workspace=ws5)

        def bwd(g=g5):
            api.ecc_soft_bwd(g, *a5, grad_chi=G5, grad_X=gx, dchi_dtau=dt_, dchi_du=du_, workspace=ws5)

        def fwd_save(g=g5):
            api.ecc_soft_fwd_save(g, *a5, chi=chi, dchi_dtau=dt_, dchi_du=du_, state=st5, workspace=ws5)

        def bwd_saved(g=g5):
            api.ecc_soft_bwd_saved(g, *a5, st5, grad_chi=G5, grad_X=gx, workspace=ws5)

        k_f, ms_f, _ = kernel_ms(api, fwd, args.steps, args.warmup)
        k_b, ms_b, _ = kernel_ms(api, bwd, args.steps, args.warmup)
        k_fs, ms_fs, _ = kernel_ms(api, fwd_save, args.steps, args.warmup)
        k_bs, ms_bs, _ = kernel_ms(api, bwd_saved, args.steps, args.warmup)
        ms_pair = time_steps(lambda: (fwd(), bwd()), args.steps, args.warmup)
        ms_saved = time_steps(lambda: (fwd_save(), bwd_saved()), args.steps, args.warmup)
        # cold: rotate over copies of the batch totalling more than the Infinity Cache
        copies = rotating(lambda: g5.clone(), X5.nbytes)
        it = [0]

        def cold_step():
            it[0] = (it[0] + 1) % len(copies)
            fwd_save(copies[it[0]])
            bwd_saved(copies[it[0]])
        ms_cold = time_steps(cold_step, max(args.steps, 2 * len(copies)), len(copies))
        K = int((api.ecc_coeff(g5, 2) != 0).sum().item())
        pairs = K * T  # (critical vertex, threshold) pairs: the sigmoids Eq. 6 / Eq. 8-10 need per pass
        nb = float(X5.nbytes)
        extra["c5_soft"] = {"workload": "C5: soft fwd+bwd, 32 x 512^2 float32, T=128, lambda=20, alpha=0.01; outputs chi, "
                                        "dchi/dtau, dchi/du, grad_X",
                            "ms_fwd_plus_bwd": round(ms_saved, 4),
                            "ms_fwd_plus_bwd_cold": round(ms_cold, 4), "cold_copies": len(copies),
                            "entry_points": "ecc_soft_fwd_save (chi, dchi/dtau, dchi/du, saved critical vertices) + "
                                            "ecc_soft_bwd_saved (grad_X from the saved list)",
                            "ms_fwd_save": round(ms_fs, 4), "ms_bwd_saved": round(ms_bs, 4),
                            "stateless_pair": {"entry_points": "ecc_soft_fwd + ecc_soft_bwd (two sweeps of the grid)",
                                               "ms_fwd_plus_bwd": round(ms_pair, 4), "ms_fwd": round(ms_f, 4),
                                               "ms_bwd": round(ms_b, 4)},
                            "critical_vertices": K, "pairs_per_pass": pairs, "dense_pairs": int(X5.size) * T,
                            "pairs_note": "pairs_per_pass = critical vertices x thresholds, what Eq. 6 / Eq. 8-10 need; of "
                                          "these, entries whose sigmoids are all 0 or 1 to 2^-64 are not evaluated (a tilt "
                                          "of 0.01 per pixel against thresholds over the field's own range saturates most "
                                          "of the image), so the rates below are upper bounds of the sigmoids evaluated",
                            "gpairs_per_s_fwd_kernel": round(pairs / (k_f * 1e-3) / 1e9, 2),
                            "gpairs_per_s_fwd_save_kernel": round(pairs / (k_fs * 1e-3) / 1e9, 2),
                            "gpairs_per_s_bwd_kernel": round(pairs / (k_b * 1e-3) / 1e9, 2),
                            "gpairs_per_s_bwd_saved_kernel": round(pairs / (k_bs * 1e-3) / 1e9, 2)}
        note5 = ("bytes floor: the grid read once (forward), read + grad_X written (backward); the kernels are bound by "
                 "launch latency and the march of 3072 short-lived waves, not by bandwidth")
        rooflines["c5_fwd"] = roofline_hbm(nb, k_f, "soft2d_fwd_kernel", counters.get("c5_fwd"), note=note5)
        rooflines["c5_bwd"] = roofline_hbm(2 * nb, k_b, "soft2d_bwd_kernel", counters.get("c5_bwd"), note=note5)
        rooflines["c5_fwd_save"] = roofline_hbm(nb, k_fs, "soft2d_fwd_save_kernel", counters.get("c5_fwd_save"), note=note5)
        rooflines["c5_bwd_saved"] = roofline_hbm(nb, k_bs, "soft2d_bwd_saved_kernel (grad_X written; the grid is not read)",
                                                 counters.get("c5_bwd_saved"), note=note5)
        log(f"[bench] C5 soft: fwd_save+bwd_saved {ms_saved:.4f} ms (cold {ms_cold:.4f}); fwd_save {ms_fs:.4f} (kernel "
            f"{k_fs:.4f}), bwd_saved {ms_bs:.4f} (kernel {k_bs:.4f}); stateless fwd+bwd {ms_pair:.4f}: fwd {ms_f:.4f} "
            f"(kernel {k_f:.4f}), bwd {ms_b:.4f} (kernel {k_b:.4f}); K={K}")
        if only == "c5":
            return
        if full:
            from oracle import ecc_oracle as O
            t0 = time.perf_counter()
            O.soft_fwd_batch(X5[:2], p["u"], p["alpha"], p["tau"], p["lam"])
            O.soft_bwd_batch(X5[:2], p["u"], p["alpha"], p["tau"], p["lam"], G5[:2].cpu().numpy())
            dt = time.perf_counter() - t0
            extra["c5_soft"]["cpu_oracle_ms_full_batch_extrapolated"] = round(dt / 2 * B5 * 1e3, 1)
            extra["c5_soft"]["cpu_oracle_sample"] = "2 of 32 items, numpy float64"
        del copies, g5
        torch.cuda.empty_cache()

    # ---------------- soft forward + backward on a volume (fused 3D path) ---------
    if want("soft3d"):
        V = synth.grf((256, 256, 256), 3.0, 5151)[None]
        T3 = 64
        gv = torch.from_numpy(V).cuda()
        uv = torch.tensor([0.48, -0.6, 0.64], dtype=torch.float32, device="cuda")
        tv = torch.linspace(float(V.min()), float(V.max()), T3, device="cuda")
        Gv = torch.from_numpy(synth.upstream_grad(1, T3)).cuda()
        wsv = torch.empty(api.ecc_workspace_bytes(V.shape[1:], 1, T3), dtype=torch.uint8, device="cuda")
        gxv = torch.empty_like(gv)

        def stepv():
            api.ecc_soft_fwd(gv, 3, uv, 0.01, tv, 20.0, workspace=wsv)
            api.ecc_soft_bwd(gv, 3, uv, 0.01, tv, 20.0, grad_chi=Gv, grad_X=gxv, workspace=wsv)
        msv = time_steps(stepv, args.steps, args.warmup)
        stv = torch.empty(api.ecc_soft_state_bytes(V.shape[1:], 1), dtype=torch.uint8, device="cuda")
        chv = torch.empty((1, T3), dtype=torch.float32, device="cuda")
        dtv, duv = torch.empty_like(chv), torch.empty((1, T3, 3), dtype=torch.float32, device="cuda")

        def stepv_saved():
            api.ecc_soft_fwd_save(gv, 3, uv, 0.01, tv, 20.0, chi=chv, dchi_dtau=dtv, dchi_du=duv, state=stv, workspace=wsv)
            api.ecc_soft_bwd_saved(gv, 3, uv, 0.01, tv, 20.0, stv, grad_chi=Gv, grad_X=gxv, workspace=wsv)
        mss = time_steps(stepv_saved, args.steps, args.warmup)
        extra["soft_3d"] = {"workload": "soft fwd+bwd, one 256^3 float32 GRF sigma=3, T=64, lambda=20, alpha=0.01",
                            "ms_fwd_plus_bwd": round(mss, 4), "entry_points": "ecc_soft_fwd_save + ecc_soft_bwd_saved",
                            "ms_stateless_fwd_plus_bwd": round(msv, 4)}
        log(f"[bench] soft 3D 256^3: fwd_save+bwd_saved {mss:.4f} ms, stateless fwd+bwd {msv:.4f} ms")
        del gv, gxv, wsv, stv
        torch.cuda.empty_cache()
        if only == "soft3d":
            return

    if only == "scan":
        gs = torch.from_numpy((synth.grf((193, 229, 193), 2.0, 6161) * 2000).astype(np.int16)[None]).cuda()
        mss = time_steps(lambda: api.ecc_hard(gs, 3, BINS, range=(-4000.0, 4000.0), superlevel=True), args.steps, args.warmup)
        log(f"[bench] scan 193x229x193 int16: {mss * 1e3:.1f} us/step")
        return
    if only == "step":
        step_host_times(args, torch, synth)
        return

    # ---------------- the grid sizes of the paper's Tables 1-2 -------------------
    if want("sizes"):
        extra["size_sweep"] = {"workload": "one float32 smoothed random field per size of the paper's Tables 1-2, 1024 "
                                           "bins, range found on the device (whole call); 8192^2 and 1024^3 are periodic "
                                           "fields tiled 2x",
                               "rows": size_rows(args, np, torch, api, synth, field_2d, field_3d)}
        if only == "sizes":
            return

    # ---------------- batches of small images, sets of directions ----------------
    if want("batches"):
        extra["batches"] = {"workload": "batches of small float32 smoothed random fields and sets of directions, 256 bins, "
                                        "range found on the device (whole call)",
                            "rows": batch_rows(args, np, torch, api, synth)}
        if only == "batches":
            return

    extra["rooflines"] = rooflines
    line = {
        "metric": "hard_ecc_throughput", "value": round(value, 2), "unit": "Gvoxel/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": round(ms, 4), "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": "C2: hard ECC, batch 16 of 2D 4096x4096 float32 smoothed Gaussian random fields "
                               "(sigma=4 px), 1024 equal-width bins over the batch-global [min,max] found on the "
                               "device (single read pass: the sweep tracks the range and lists the critical "
                               "vertices, which are binned afterwards)", "bins": BINS, "batch": 16},
        "roofline": roofline,
    }
    if full:
        line["cpu_baseline"] = cpu
    line["extra"] = extra
    print(json.dumps(line), flush=True)


if __name__ == "__main__":
    main()

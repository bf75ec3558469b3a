#!/usr/bin/env python3
"""Benchmark of the DCNv4 operator on one MI355X at the InternImage stage-1 shape
(N=64, 56x56, C=128, G=8, 3x3, stride 1, pad 1), synthetic seeded inputs.

A step of the headline leg is one fp16 forward pass (the leg the 60 %-of-HBM-peak bar is
quoted on); the same run also times the fp32 forward and the fp32 and fp16 backward (grad_x,
grad_offset, grad_mask) at the same shape and reports them under "legs".  Every leg rotates
over several buffer sets whose total size exceeds the 256 MB memory-side cache, so a launch
does not find its inputs in cache ("cold"); the back-to-back rate on one buffer set is
reported beside it as "hot".  Durations come from HIP events recorded on the stream the
kernels are launched on.  Prints ONE JSON line.
"""
import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0          # MI355X HBM3E, published peak


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=200)
    ap.add_argument("--warmup", type=int, default=20)
    ap.add_argument("--sets", type=int, default=4, help="buffer sets rotated per leg")
    ap.add_argument("--legs", default="fwd_f16,fwd_f32,bwd_f32,bwd_f16,fwd_f16_merged,bwd_f32_merged,fwd_f16_softmax,bwd_f32_softmax,"
                                      "module_f16,modulelite_f16,module_f32,modulelite_f32,module_f16_dw",
                    help="fwd|bwd _ f16|f32 [_merged: offsets and mask values in one [N,Ho,Wo,G,32] buffer | "
                         "_softmax: the mask tensor holds logits, normalised over the 9 taps (DCNv3 form)]")
    ap.add_argument("--workload", default="c2")
    ap.add_argument("--more-workloads", default="c3_28,c3_14,c3_7,c4",
                    help="further workloads whose fp16 forward is timed and reported under legs as fwd_f16@<name>")
    ap.add_argument("--paper-shapes", action="store_true",
                    help="also time the forward (fp32 and fp16) at the ten shapes of the paper's Tab. 2 and 3")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--cpu-seconds", type=float, default=10.0)
    ap.add_argument("--cold-only", action="store_true", help="skip the back-to-back (hot) timing loop")
    ap.add_argument("--calibrate-copy", action="store_true",
                    help="also run one 256 MiB device-to-device copy (a dispatch of known size, for scaling "
                         "profiler byte counters)")
    ap.add_argument("--opt", action="append", default=[], metavar="KEY=VALUE",
                    help="library tuning option (dcnv4_set_option), repeatable")
    return ap.parse_args()


def ensure_built():
    from paper_2401_06197_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        from paper_2401_06197_amd import build
        build.build()
    return binding


def measured_traffic(leg, workload, kernel=None):
    """HBM bytes per launch of the leg's kernel as measured with rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE
    (scaled by a copy of known size); read from the committed profile summary.  None if there is no
    summary, or if it was taken on another kernel than the one that ran now (`kernel`)."""
    # (c5, the training-step config, is the c2 shape: the backward summaries carry its name)
    path = os.path.join(ROOT, "profiles", f"{leg}_{workload}_hbm_traffic.md")
    if not os.path.exists(path) and workload == "c2":
        path = os.path.join(ROOT, "profiles", f"{leg}_c5_hbm_traffic.md")
    traffic, profiled = None, None
    try:
        for line in open(path):
            if line.startswith("traffic_bytes_per_launch"):
                traffic = int(line.split("=")[1].split()[0])
            if line.startswith("kernel"):
                profiled = line.split("=", 1)[1].strip().strip("`")
    except OSError:
        return None
    if kernel is not None and profiled != kernel:
        return None
    return traffic


def copy_ceiling(torch, stream, nbytes, steps):
    """GB/s (bytes read + bytes written) of a plain device-to-device copy of nbytes/2 bytes, i.e. of the
    same total traffic as the headline kernel's algorithmic bytes: what this machine's memory system gives
    a kernel that does nothing but stream."""
    half = max(1 << 20, (nbytes // 2) & ~255)
    srcs = [torch.empty(half, dtype=torch.uint8, device="cuda:0").fill_(i + 1) for i in range(4)]
    dsts = [torch.empty_like(t) for t in srcs]
    with torch.cuda.stream(stream):
        for i in range(8):
            dsts[i % 4].copy_(srcs[i % 4])
        start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        stream.synchronize()
        start.record(stream)
        for i in range(steps):
            dsts[i % 4].copy_(srcs[i % 4])
        stop.record(stream)
        stop.synchronize()
    us = start.elapsed_time(stop) / steps * 1e3
    return {"bytes_moved": 2 * half, "us_per_copy": round(us, 3), "GBps": 2 * half / (us * 1e-6) / 1e9,
            "frac_of_hbm_peak": 2 * half / (us * 1e-6) / 1e9 / HBM_PEAK_GBS}


def time_leg(torch, stream, launch, nsets, steps, warmup, cold_only=False):
    """Average duration of one launch(set_index) in ms: cold (rotating sets) and hot (set 0 only)."""
    out = {}
    for label, pick in (("cold", lambda i: i % nsets), ("hot", lambda i: 0)):
        if cold_only and label == "hot":
            out["hot"] = float("nan")
            continue
        for i in range(warmup):
            launch(pick(i))
        start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        stream.synchronize()
        torch.cuda.synchronize()
        start.record(stream)
        for i in range(steps):
            launch(pick(i))
        stop.record(stream)
        stop.synchronize()
        torch.cuda.synchronize()
        out[label] = start.elapsed_time(stop) / steps
    return out


def run_leg(torch, dcn, lib, stream, cfg, leg, a, host_inputs, steps, keep_output=False):
    """Times one leg ("fwd_f16", "bwd_f32", ...) on workload cfg; returns (record, first output or None)."""
    from paper_2401_06197_amd.synth import make_inputs, merge_offset_mask
    dev = torch.device("cuda:0")
    Ho, Wo = cfg.out_hw
    out_elems = cfg.N * Ho * Wo * cfg.C
    geo = dict(kernel=cfg.kernel, stride=cfg.stride, pad=cfg.pad, dilation=cfg.dilation, offset_scale=cfg.offset_scale)
    direction, dt = leg.split("_")[:2]
    merged = leg.endswith("_merged")
    softmax = leg.endswith("_softmax")
    tdt = {"f16": torch.float16, "f32": torch.float32}[dt]
    code = {"f16": dcn.DCNV4_F16, "f32": dcn.DCNV4_F32}[dt]
    if (cfg.name, dt) not in host_inputs:
        host_inputs[(cfg.name, dt)] = make_inputs(cfg, dt, seed=0)
    base = {k: torch.from_numpy(v).to(dev) for k, v in host_inputs[(cfg.name, dt)].items()}
    if merged:
        h = host_inputs[(cfg.name, dt)]
        base = {"x": base["x"], "grad_y": base["grad_y"], "om": torch.from_numpy(merge_offset_mask(h["offset"], h["mask"])).to(dev)}
    # enough buffer sets that a launch does not find its inputs in the 256 MB memory-side cache
    one_set = sum(v.numel() * v.element_size() for v in base.values())
    nsets = max(a.sets, min(16, -(-(320 << 20) // one_set)))
    sets = [base] + [{k: v.clone() for k, v in base.items()} for _ in range(nsets - 1)]
    if direction == "fwd":
        outs = [torch.empty((cfg.N, Ho, Wo, cfg.C), dtype=tdt, device=dev) for _ in range(nsets)]
        if merged:
            alg = dcn.dcnv4_forward_merged_algorithmic_bytes(cfg.N, cfg.H, cfg.W, cfg.G, cfg.Cg, Ho, Wo, code)
            argv = [dcn.dcnv4_forward_merged(s["x"], s["om"], out=o, stream=stream, prepare_only=True, **geo)
                    for s, o in zip(sets, outs)]
            fn = lib.dcnv4_forward_merged
        else:
            alg = dcn.dcnv4_forward_algorithmic_bytes(cfg.N, cfg.H, cfg.W, cfg.G, cfg.Cg, Ho, Wo, code)
            argv = [dcn.dcnv4_forward(s["x"], s["offset"], s["mask"], out=o, stream=stream, prepare_only=True, **geo)
                    for s, o in zip(sets, outs)]
            fn = lib.dcnv4_forward_softmax if softmax else lib.dcnv4_forward
    elif merged:
        outs = [(torch.empty_like(s["x"]), torch.empty_like(s["om"])) for s in sets]
        alg = dcn.dcnv4_backward_merged_algorithmic_bytes(cfg.N, cfg.H, cfg.W, cfg.G, cfg.Cg, Ho, Wo, code)
        argv = [dcn.dcnv4_backward_merged(s["x"], s["om"], s["grad_y"], out=o, stream=stream, prepare_only=True, **geo)
                for s, o in zip(sets, outs)]
        fn = lib.dcnv4_backward_merged
    else:
        outs = [(torch.empty_like(s["x"]), torch.empty_like(s["offset"]), torch.empty_like(s["mask"])) for s in sets]
        alg = dcn.dcnv4_backward_algorithmic_bytes(cfg.N, cfg.H, cfg.W, cfg.G, cfg.Cg, Ho, Wo, code)
        argv = [dcn.dcnv4_backward(s["x"], s["offset"], s["mask"], s["grad_y"], out=o, stream=stream,
                                   prepare_only=True, **geo) for s, o in zip(sets, outs)]
        fn = lib.dcnv4_backward_softmax if softmax else lib.dcnv4_backward

    def launch(i):
        rc = fn(*argv[i])
        if rc:
            raise dcn.Dcnv4Error(rc, leg)
    torch.cuda.synchronize()
    t = time_leg(torch, stream, launch, nsets, steps, a.warmup, a.cold_only)
    rec = {
        "workload": cfg.name,
        "kernel": dcn.dcnv4_last_kernel_name(direction == "bwd"),
        "steps": steps,
        "us_per_launch": round(t["cold"] * 1e3, 3),
        "out_elems_per_s": out_elems / (t["cold"] * 1e-3),
        "algorithmic_bytes": alg,
        "GBps": alg / (t["cold"] * 1e-3) / 1e9,
        "frac_of_hbm_peak": alg / (t["cold"] * 1e-3) / 1e9 / HBM_PEAK_GBS,
        "hot_us_per_launch": None if a.cold_only else round(t["hot"] * 1e3, 3),
        "hot_GBps": None if a.cold_only else alg / (t["hot"] * 1e-3) / 1e9,
        "buffer_sets": nsets,
    }
    rec["traffic"] = measured_traffic(leg, cfg.name, rec["kernel"])
    y = outs[0].float().cpu().numpy() if (keep_output and direction == "fwd") else None
    del sets, outs, base
    torch.cuda.empty_cache()
    return rec, y


def run_module_leg(torch, dcn, lib, stream, cfg, leg, a, steps):
    """Times the module forward ("module_f16": both projections; "modulelite_f16": without them; suffix "_dw":
    with the depthwise convolution in front of the offset/scalar layer) on workload
    cfg.  Bytes: every tensor between the layers counted once per write and once per read."""
    from paper_2401_06197_amd.synth import make_inputs, make_module_params
    dev = torch.device("cuda:0")
    kind, dt = leg.split("_")[:2]
    light = kind == "modulelite"
    dw = leg.endswith("_dw")
    tdt = {"f16": torch.float16, "f32": torch.float32}[dt]
    es = 2 if dt == "f16" else 4
    x0 = torch.from_numpy(make_inputs(cfg, dt, seed=0)["x"]).to(dev)
    prm = {k: torch.from_numpy(v).to(dev) for k, v in make_module_params(cfg, dt, seed=0, lightweight=light, depthwise=dw).items()}
    P = cfg.N * cfg.H * cfg.W
    moved = P * es * ((2 * cfg.C + 2 * 32 * cfg.G) if light else (6 * cfg.C + 2 * 32 * cfg.G)) + (P * es * 3 * cfg.C if dw else 0)
    one_set = 2 * x0.numel() * es + dcn.dcnv4_module_workspace_bytes(cfg.N, cfg.H, cfg.W, cfg.G, cfg.Cg, {"f16": 1, "f32": 0}[dt], light, dw)
    nsets = max(a.sets, min(16, -(-(320 << 20) // one_set)))
    xs = [x0] + [x0.clone() for _ in range(nsets - 1)]
    ys = [torch.empty_like(x0) for _ in range(nsets)]
    wss = [torch.empty(one_set - 2 * x0.numel() * es, dtype=torch.uint8, device=dev) for _ in range(nsets)]
    geo = dict(kernel=cfg.kernel, stride=cfg.stride, pad=cfg.pad, dilation=cfg.dilation, offset_scale=cfg.offset_scale)
    argv = [dcn.dcnv4_module_forward(x, prm["w_om_padded"], prm["b_om_padded"], cfg.G, w_in=prm.get("w_in"), b_in=prm.get("b_in"),
                                     w_out=prm.get("w_out"), b_out=prm.get("b_out"), w_dw=prm.get("w_dw"), b_dw=prm.get("b_dw"), workspace=w, out=y, stream=stream,
                                     prepare_only=True, **geo) for x, y, w in zip(xs, ys, wss)]

    def launch(i):
        rc = lib.dcnv4_module_forward(*argv[i])
        if rc:
            raise dcn.Dcnv4Error(rc, leg)
    torch.cuda.synchronize()
    t = time_leg(torch, stream, launch, nsets, steps, a.warmup, a.cold_only)
    rec = {"workload": cfg.name, "kernel": "linear layers + " + str(dcn.dcnv4_last_kernel_name(0)), "steps": steps,
           "us_per_launch": round(t["cold"] * 1e3, 3), "out_elems_per_s": P * cfg.C / (t["cold"] * 1e-3),
           "moved_bytes": moved, "GBps": moved / (t["cold"] * 1e-3) / 1e9,
           "frac_of_hbm_peak": moved / (t["cold"] * 1e-3) / 1e9 / HBM_PEAK_GBS,
           "hot_us_per_launch": None if a.cold_only else round(t["hot"] * 1e3, 3), "buffer_sets": nsets}
    del xs, ys, wss, prm
    torch.cuda.empty_cache()
    return rec


# the paper's module-level numbers (appendix, A100, microseconds, fp32 / fp16; full module, lightweight): context
PAPER_A100_MODULE_US = {"paper_56x56x128": ((1280, 873), (762, 547)), "paper_28x28x256": ((738, 483), (419, 313)),
                        "paper_14x14x512": ((452, 324), (375, 192)), "paper_7x7x1024": ((334, 265), (306, 130)),
                        "paper_14x14x768": ((787, 463), (389, 249))}

# the paper's op-level numbers (Tab. 2 and 3, A100 80GB SXM, microseconds, fp32 / fp16): context, not a target
PAPER_A100_US = {"paper_56x56x128": (606, 404), "paper_28x28x256": (303, 230), "paper_14x14x512": (145, 123),
                 "paper_7x7x1024": (73.0, 68.0), "paper_14x14x768": (224, 147), "paper_200x320x128": (210, 136),
                 "paper_100x160x256": (124, 89.5), "paper_50x80x512": (70.7, 58.9), "paper_25x40x1024": (45.2, 42.6),
                 "paper_64x64x768": (103, 67.2)}


def main():
    a = parse()
    if a.gpus != 1:
        print(f"bench.py: this build runs on ONE GPU (the operator needs no exchange between GPUs; "
              f"each GPU would take N/{a.gpus} images); --gpus {a.gpus} is not run", file=sys.stderr)
        sys.exit(2)
    import numpy as np
    import torch
    dcn = ensure_built()
    lib = dcn.load_library()
    for kv in a.opt:
        k, v = kv.split("=")
        dcn.dcnv4_set_option(k, int(v))
    from paper_2401_06197_amd.synth import CONFIGS

    if not torch.cuda.is_available():
        print("bench.py: no GPU visible", file=sys.stderr)
        sys.exit(1)
    cfg = CONFIGS[a.workload]
    Ho, Wo = cfg.out_hw
    out_elems = cfg.N * Ho * Wo * cfg.C
    dev = torch.device("cuda:0")
    stream = torch.cuda.Stream(device=dev)
    geo = dict(kernel=cfg.kernel, stride=cfg.stride, pad=cfg.pad, dilation=cfg.dilation, offset_scale=cfg.offset_scale)
    if a.calibrate_copy:
        src = torch.empty(256 << 20, dtype=torch.uint8, device=dev).fill_(1)
        dst = torch.empty_like(src)
        dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst
    legs_wanted = [s for s in a.legs.split(",") if s]
    if not legs_wanted or legs_wanted[0].startswith("module"):
        print("bench.py: the first leg is the headline and must be an operator leg (fwd_* or bwd_*)", file=sys.stderr)
        sys.exit(2)
    legs = {}
    host_inputs = {}
    head_y = None
    for leg in legs_wanted:
        steps = a.steps if leg.startswith("fwd") else max(1, a.steps // 4)
        if leg.startswith("module"):
            legs[leg] = run_module_leg(torch, dcn, lib, stream, cfg, leg, a, steps)
            continue
        legs[leg], y = run_leg(torch, dcn, lib, stream, cfg, leg, a, host_inputs, steps, keep_output=leg == legs_wanted[0])
        if leg == legs_wanted[0]:
            head_y = y
    head = legs_wanted[0]
    hl = legs[head]
    head_inputs = host_inputs[(cfg.name, head.split("_")[1])]
    host_inputs = {k: v for k, v in host_inputs.items() if k == (cfg.name, head.split("_")[1])}

    # the other workloads (fp16 forward), and on request the paper's own benchmark shapes
    for name in [w for w in a.more_workloads.split(",") if w and w != cfg.name]:
        legs[f"fwd_f16@{name}"], _ = run_leg(torch, dcn, lib, stream, CONFIGS[name], "fwd_f16", a, {}, a.steps)
    if a.paper_shapes:
        for name, (us32, us16) in PAPER_A100_US.items():
            for leg, ref_us in (("fwd_f32", us32), ("fwd_f16", us16)):
                r, _ = run_leg(torch, dcn, lib, stream, CONFIGS[name], leg, a, {}, a.steps)
                r["paper_a100_us"] = ref_us
                legs[f"{leg}@{name}"] = r
        for name, (full, lite) in PAPER_A100_MODULE_US.items():
            for leg, ref_us in (("module_f32", full[0]), ("module_f16", full[1]), ("modulelite_f32", lite[0]), ("modulelite_f16", lite[1])):
                r = run_module_leg(torch, dcn, lib, stream, CONFIGS[name], leg, a, max(1, a.steps // 4))
                r["paper_a100_us"] = ref_us
                legs[f"{leg}@{name}"] = r

    rec = {
        "metric": "DCNv4 fwd/bwd output elems/s and achieved HBM GB/s (% of peak) at 56x56x128",
        "value": hl["out_elems_per_s"],
        "unit": "output elems/s",
        "n_gpus": 1,
        "steps": hl["steps"],
        "warmup": a.warmup,
        "ms_per_step": hl["us_per_launch"] / 1e3,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": head.split("_")[1],
        "data": "synthetic",
        "config": {"workload": f"{cfg.name}: N={cfg.N} {cfg.H}x{cfg.W} C={cfg.C} G={cfg.G} 3x3 s1 p1, leg {head}",
                   "offset_std_px": cfg.sigma, "cache": "cold (rotating buffer sets)"},
        "roofline": {"bound": "hbm", "kernel": hl["kernel"], "achieved": hl["GBps"], "peak": HBM_PEAK_GBS,
                     "unit": "GB/s", "frac": hl["frac_of_hbm_peak"], "traffic": hl["traffic"]},
        "copy_ceiling": copy_ceiling(torch, stream, hl["algorithmic_bytes"], max(20, a.steps // 4)),
        "legs": legs,
    }

    if not a.no_cpu_baseline:
        import ctypes
        import oracle
        t = head_inputs
        reps, spent, ref = 0, 0.0, None
        while spent < a.cpu_seconds and reps < 40:
            t0 = time.perf_counter()
            ref = oracle.forward(t["x"], t["offset"], t["mask"], **geo)
            spent += time.perf_counter() - t0
            reps += 1
        rec["cpu_baseline"] = {
            "value": out_elems * reps / spent, "unit": "output elems/s", "cores": oracle.threads(), "kind": "oracle",
            "sample": f"{reps} full forward passes of the same workload (double precision, {spent:.1f} s)",
        }
        # the same oracle on one host thread, on the first images of the batch (a bounded sample)
        try:
            omp = ctypes.CDLL("libgomp.so.1")
            many = oracle.threads()
            n1 = max(1, cfg.N // 16)
            omp.omp_set_num_threads(1)
            t0 = time.perf_counter()
            oracle.forward(t["x"][:n1], t["offset"][:n1], t["mask"][:n1], **geo)
            dt1 = time.perf_counter() - t0
            omp.omp_set_num_threads(many)
            rec["cpu_baseline"]["single_thread"] = {
                "value": (out_elems // cfg.N) * n1 / dt1, "unit": "output elems/s", "cores": 1,
                "sample": f"one forward pass over the first {n1} of {cfg.N} images ({dt1:.1f} s)"}
        except OSError:
            pass
        # the oracle's backward on the same shape in fp32 (one pass over the whole batch: well under a second)
        try:
            from paper_2401_06197_amd.synth import make_inputs
            nb = cfg.N
            tb = {k: v[:nb] for k, v in make_inputs(cfg, "f32", seed=0).items()}
            t0 = time.perf_counter()
            oracle.backward(tb["x"], tb["offset"], tb["mask"], tb["grad_y"], **geo)
            dtb = time.perf_counter() - t0
            rec["cpu_baseline"]["backward"] = {
                "value": (out_elems // cfg.N) * nb / dtb, "unit": "output elems/s", "cores": oracle.threads(), "kind": "oracle",
                "sample": f"one backward pass (grad_x, grad_offset, grad_mask; double precision) over the first {nb} of {cfg.N} images ({dtb:.1f} s)"}
        except MemoryError:
            pass
        if head_y is not None:
            err = np.abs(head_y - ref)
            tol = 2e-2 if head.endswith("f16") else 1e-5
            big = np.abs(ref) >= 1.0
            rec["parity"] = {"max_abs_err": float(err.max()),
                             "max_rel_err": float((err[big] / np.abs(ref[big])).max()) if big.any() else None,
                             "max_rel_err_note": "over outputs with |reference| >= 1",
                             "max_err_over_tolerance": float((err / (tol + tol * np.abs(ref))).max()),
                             "within_tol": bool(np.all(err <= tol + tol * np.abs(ref)))}
    print(json.dumps(rec))


if __name__ == "__main__":
    main()

#!/usr/bin/env python3
"""Benchmark of the HDC classification hot path on one MI355X.

Workload: the speech-feature-shaped configuration (617 int8 features,
26 classes, D = 10240): class hypervectors are trained on its 6238 training
vectors (GPU encode + majority bundle), then a batch of fresh queries drawn
from the same mixture is classified by the fused kernel (encode -> sign ->
Hamming -> argmin).  One timed step classifies the whole batch with the plain
(unapproximated) configuration; ``value`` is queries/s of those steps.

The tuned configuration is chosen the way the paper's tuner does it
(Sec. 3 / 5.2): every candidate of the (D', stride, dtype) grid is evaluated
on 2000 sweep queries in one persistent launch (hdc_eval_configs), and the
fastest one whose accuracy is within 1 point of the plain configuration is
kept; it is then timed on the same batch.  Also reported: per-call latency
p50/p99 at the configuration's test-set size (1559 queries), the training
time, the sweep time, a roofline line for the fused kernel (int8 MFMA), and
the CPU oracle timed on a bounded sample.

Usage: python bench.py [--gpus 1] [--steps 20] [--warmup 3] [--batch 262144]
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

MFMA_INT8_PEAK_TOPS = 5000.0      # MI355X dense int8 MFMA, 5.0 POP/s
HBM_PEAK_GBS = 8000.0
MFMA_FP32_PEAK_TFLOPS = 157.3
SWEEP_SHARED = 4               # hdc tile id of the shared sweep path
# 32-bit VALU issue rate: 256 CUs x 4 SIMDs x 16 lanes x 2.4 GHz (the fp32
# vector peak of 157.3 TFLOP/s counts an FMA as two flops and packs two lanes)
VALU_PEAK_TOPS = 256 * 4 * 16 * 2.4e9 / 1e12


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=30)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--batch", type=int, default=1 << 18)
    ap.add_argument("--latency-calls", type=int, default=200)
    ap.add_argument("--cpu-sample", type=int, default=98304)
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--ceilings", action="store_true", help="also measure the device ceilings (random-operand "
                    "int8 MFMA loop, HBM read stream) beside the published peaks")
    ap.add_argument("--no-extras", action="store_true", help="only the timed plain steps (profiling)")
    ap.add_argument("--only", default="", help="comma list of the extra sections to run (profiling): train, "
                    "bundle, sweep (with the tuned selection and per-call latency), hamming, adc, cosine, "
                    "encode_side, retrain, ladder, serving, plain_fp32")
    ap.add_argument("--no-autotune", action="store_true", help="built-in tile choices, no tuning launches")
    ap.add_argument("--classify-tile", default=None,
                    help="tile variant of the headline classifier by name (dma_2x2, dma_2x3, ...): no tuning for it")
    ap.add_argument("--classify-form", default="auto", choices=["auto", "int8", "int8shift"],
                    help="projection form of the int8 classifier: the +-1 projection (int8), the shifted one "
                         "(int8shift: weights p + 1, the same results), or whichever the tuning times faster")
    ap.add_argument("--serve-seconds", type=float, default=3.0, help="length of each open-loop serving run")
    ap.add_argument("--serve-budgets", default="16G,64M,5M",
                    help="HBM budgets of the open-loop serving runs (in-flight request bytes)")
    ap.add_argument("--serve-saturation-seconds", type=float, default=3.0,
                    help="length of the closed-loop saturation run (0: none)")
    ap.add_argument("--serve-poll-us", type=float, default=10.0,
                    help="how long the serving loop sleeps when it has nothing to launch or complete")
    ap.add_argument("--full-out", default=os.path.join(ROOT, "gpurun_out", "bench_full.json"),
                    help="where the full result record is written (the last stdout line is a summary of it)")
    return ap.parse_args()


def log(*a):
    print("[bench]", *a, file=sys.stderr, flush=True)


def cpu_model() -> str:
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def _r(v, nd=4):
    """Round floats for the summary line (3-4 significant digits)."""
    if isinstance(v, float):
        return float("%.*g" % (nd, v))
    if isinstance(v, dict):
        return {k: _r(x, nd) for k, x in v.items()}
    if isinstance(v, (list, tuple)):
        return [_r(x, nd) for x in v]
    return v


def _pick(d, *keys):
    return {k: d[k] for k in keys if isinstance(d, dict) and k in d}


def compact(out: dict) -> dict:
    """The one-line summary printed last: the contract fields, the headline
    roofline and CPU baseline, and a few figures of every other section (the
    full record goes to a file).  Stays well under 4 KB."""
    c = _pick(out, "metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better",
              "scaling", "vs_baseline", "dtype", "data", "accuracy_plain", "p50_ms", "p99_ms")
    c["config"] = _pick(out.get("config", {}), "workload", "F", "K", "D", "batch", "parallelism",
                        "projection_form")
    if "roofline" in out:
        c["roofline"] = _pick(out["roofline"], "bound", "achieved", "peak", "unit", "frac", "traffic", "kernel",
                              "ms_per_launch", "tile")
    if "cpu_baseline" in out:
        c["cpu_baseline"] = _pick(out["cpu_baseline"], "value", "unit", "cores", "kind", "sample", "cpu_model",
                                  "tuned_value", "single_thread_value")
    if "tuned" in out:
        t = out["tuned"]
        c["tuned"] = dict(_pick(t, "config", "value", "ms_per_step", "accuracy", "speedup_vs_plain"),
                          p99_ms=out.get("latency", {}).get("tuned", {}).get("p99_ms"))
    extras = {}
    if "latency" in out:
        extras["latency_1559"] = {k: _pick(v, "p50_ms", "p99_ms") for k, v in out["latency"].items()}
    if "train" in out:
        extras["train_ms"] = out["train"]["ms"]
    for key in ("sweep", "bundle", "plain_fp32"):
        if key in out:
            sec = out[key]
            extras[key] = dict(_pick(sec, "ms", "slots", "queries_per_s", "accuracy", "test_accuracy", "GB_s",
                                     "per_config_ms", "shared_ms"),
                               **({"frac": sec["roofline"]["frac"], "bound": sec["roofline"]["bound"]}
                                  if "roofline" in sec else {}))
    if "hamming_unfused" in out:
        extras["hamming_mfma_GB_s"] = {k.split()[0] + k.split()[1]: v["mfma"]["GB_s"]
                                       for k, v in out["hamming_unfused"].items()}
    if "ladder" in out:
        extras["ladder"] = {wl: {t: _pick(v, "flip_rate", "accuracy") for t, v in r.items()
                                 if isinstance(v, dict) and "flip_rate" in v}
                            for wl, r in out["ladder"].items()}
    if "serving" in out:
        sv = out["serving"]
        extras["serving"] = {m: dict(_pick(sv[m], "p50_ms", "p99_ms", "queries_per_s"),
                                     saturation_qps=sv[m].get("runs", {}).get("saturation", {}).get("queries_per_s"),
                                     saturation_4096_qps=sv[m].get("runs", {}).get("saturation_4096", {})
                                     .get("queries_per_s"),
                                     p99_by_budget={b: r.get("p99_ms") for b, r in sv[m].get("runs", {}).items()
                                                    if not b.startswith("saturation")})
                             for m in ("plain", "tuned") if m in sv}
    for key in ("cosine", "adc", "retrain"):
        if key in out and "roofline" in out[key]:
            extras[key + "_frac"] = out[key]["roofline"]["frac"]
    if "ceilings" in out:
        extras["ceilings"] = {"mfma_i8_TOPs_best": max(out["ceilings"]["mfma_i8_TOPs"].values()),
                              "mfma_i8_shifted_TOPs_best": max(out["ceilings"]["mfma_i8_shifted_TOPs"].values()),
                              "hbm_read_GBs_best": max(out["ceilings"]["hbm_read_GBs"].values())}
    if extras:
        c["extras"] = extras
    c["full_record"] = out.get("full_record")
    return _r(c)


def traffic_key(tile: str, form: str) -> str:
    """Key of the headline launch's record in profiles/traffic.json."""
    return "k_encode_classify_speech_b262144_" + tile + ("_shift" if form == "int8shift" else "")


def measured_traffic(key: str, batch: int, tile: str):
    """HBM bytes per launch of a kernel from profiles/traffic.json (rocprofv3
    FETCH_SIZE / WRITE_SIZE, copy-calibrated), or None when the kernel's
    sources changed since the counters were taken, the batch differs or the
    launch uses another tile variant."""
    try:
        t = json.load(open(os.path.join(ROOT, "profiles", "traffic.json")))[key]
        h = hashlib.sha256(b"".join(open(os.path.join(ROOT, f), "rb").read() for f in t["sources"])).hexdigest()
    except (OSError, KeyError, ValueError):
        return None
    if h != t["sha256"] or int(t["batch"]) != batch or t.get("tile") != tile:
        return None
    return float(t["bytes_per_launch"])


def main():
    args = parse()
    world = int(os.environ.get("WORLD_SIZE", "1"))
    if args.gpus != 1 or world != 1:
        print("bench.py runs on exactly one GPU: the library has no multi-GPU path "
              "(queries or sweep slots would shard across GPUs without communication); "
              "got --gpus %d, WORLD_SIZE %d" % (args.gpus, world), file=sys.stderr)
        sys.exit(2)

    import torch
    from paper_2606_26547_amd import datagen as dg
    from paper_2606_26547_amd import hdc, tuner

    torch.cuda.set_device(0)
    dev = "cuda"
    N = args.batch

    # ------------------------------------------------------------ data
    t0 = time.time()
    sp = dg.SpeechLike(2)
    ds = sp.dataset()
    F, K, D = ds.F, ds.K, ds.D
    Xq, yq = sp.queries(N, stream=10)
    Xs, ys = sp.queries(dg.C4["n_queries"], stream=4)          # sweep queries
    log("data ready in %.1fs: F=%d K=%d D=%d batch=%d" % (time.time() - t0, F, K, D, N))

    Pd = hdc.pad_cols(ds.P, dev)
    # the model's projection in the shifted forms (made once with the model;
    # int8 / E4M3 classification on them gives the same labels and distances)
    Ps = hdc.shift_projection(Pd, F)
    shifted_P = {t: hdc.shift_projection(Pd, F, compute=ts) for t, ts in hdc.SHIFTED.items()
                 if hdc.shift_supported("classify", F, K, ts)}
    Xtr = hdc.pad_cols(ds.X_train, dev)
    ytr = torch.as_tensor(ds.y_train).to(dev)
    Xqd = hdc.pad_cols(Xq, dev)
    yqd = torch.as_tensor(yq).to(dev)
    Xsd = hdc.pad_cols(Xs, dev)
    ysd = torch.as_tensor(ys).to(dev)
    Xte = hdc.pad_cols(ds.X_test, dev)
    ws_b = torch.empty(hdc.lib().hdc_bundle_workspace_bytes(Xtr.shape[0], D, K), dtype=torch.uint8, device=dev)
    Htr = torch.zeros((Xtr.shape[0], hdc.words(D)), dtype=torch.int64, device=dev)

    tiles_in_use = {"encode": 0, "encode_form": "int8"}

    def train():
        form = tiles_in_use["encode_form"]
        hdc.encode(Xtr, F, Ps if form == "int8shift" else Pd, D, form, out=Htr, tile=tiles_in_use["encode"])
        return hdc.bundle(Htr, D, ytr, K, ws_b)

    Cw, _ = train()
    torch.cuda.synchronize()

    def event_loop(fn, steps, warmup):
        for _ in range(warmup):
            fn()
        torch.cuda.synchronize()
        ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(steps)]
        t = time.perf_counter()
        for a, b in ev:
            a.record()
            fn()
            b.record()
        torch.cuda.synchronize()
        wall = time.perf_counter() - t
        durs = [a.elapsed_time(b) for a, b in ev]          # ms, on the launch stream
        return wall * 1e3 / steps, float(np.mean(durs)), durs

    # ------------------------------------------------------------ tile autotuning
    # the buckets this run launches: the speech classifier and encoder and
    # the configuration sweep (2000 queries, the 256 sampled slots)
    from paper_2606_26547_amd import autotune as AT
    slots = [(d, k, 0, t) for (d, k, t) in dg.sweep_slots(4)]
    tile_shapes = [AT.Shape("encode", F, 1, D, 8192), AT.Shape("sweep", F, K, D, dg.C4["n_queries"], cfgs=slots)]
    t0 = time.time()
    tiles = AT.autotune(tile_shapes) if not args.no_autotune else []
    # the headline classifier is tuned at the batch it is timed on, in both
    # projection forms; its variants give identical labels, so a 1% margin
    # is enough
    forms = ["int8", "int8shift"] if args.classify_form == "auto" else [args.classify_form]
    forms = [f for f in forms if f == "int8" or hdc.shift_supported("classify", F, K)]
    cls_choice = {}
    if not args.no_autotune and not args.classify_tile:
        for form in forms:
            cls_choice[form] = AT.tune(AT.Shape("classify", F, K, D, N, compute=form), margin=0.01)
            tiles.append(cls_choice[form])
    table = AT.TileTable.from_choices(tiles)
    # the form whose chosen variant timed fastest (without timings the
    # shifted one where it has kernels: it measured faster on every box)
    cls_form = min(forms, key=lambda f: cls_choice[f].variants[cls_choice[f].chosen_name]) if cls_choice \
        else forms[-1]
    cls_tile_id = table.get("classify", "int8", cls_form, F, K)
    if args.classify_tile:
        cls_tile_id = {v: k for k, v in hdc.TILE_NAMES["classify"].items()}[args.classify_tile]
    P_cls = Ps if cls_form == "int8shift" else Pd
    # the training encode takes the classifier's projection form (the
    # shifted one with its built-in 2x2 shape)
    if cls_form == "int8shift" and hdc.shift_supported("encode", F, 1):
        tiles_in_use.update(encode=0, encode_form="int8shift")
    else:
        tiles_in_use["encode"] = table.get("encode", "int8", "int8", F, 1)
    sweep_tile = table.get("sweep", "int8", "int8", F, K)
    cls_tile = hdc.TILE_NAMES["classify"][cls_tile_id or hdc.tile_variants("classify", "int8", cls_form, F, K)[0]]
    log("tiles (%.1fs): %s" % (time.time() - t0, {c.shape.kind: (c.chosen_name, {k: round(v, 3) for k, v in
                                                                                 c.variants.items()})
                                                  for c in tiles}))

    # ------------------------------------------------------------ plain steps
    plain = hdc.Prepared(Cw, D, cls_form, tile=cls_tile_id)
    labels = torch.empty(N, dtype=torch.int32, device=dev)
    ms_step, ms_kernel, _ = event_loop(lambda: plain(Xqd, F, P_cls, labels), args.steps, args.warmup)
    acc_plain = float((labels == yqd).float().mean().item())
    qps = N / (ms_step / 1e3)
    ops = 2.0 * F * D * N                      # algorithmic encode ops per launch (pad not counted)
    achieved = ops / (ms_kernel / 1e3) / 1e12
    log("plain: %.3f ms/step (kernel %.3f ms) -> %.3e q/s, %.1f TOP/s, acc %.4f" %
        (ms_step, ms_kernel, qps, achieved, acc_plain))

    out = {
        "metric": "queries/s (encode+Hamming argmin) plain vs tuned at <=1% acc loss; p99 ms",
        "value": qps,
        "unit": "queries/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "int8",
        "data": "synthetic (seeded c2 Gaussian-mixture generator; ISOLET-shaped, no real dataset)",
        "config": {"workload": "speech-shaped HDC classify, int8 features F=617, K=26 classes, D=10240, "
                               "plain config, batch of %d fresh queries; model bundled from 6238 train vectors" % N,
                   "F": F, "K": K, "D": D, "batch": N, "parallelism": "none (1 GPU)",
                   "projection_form": cls_form},
        "accuracy_plain": acc_plain,
        "tiles": AT.to_json(tiles) if tiles else None,
        "roofline": {"bound": "mfma", "kernel": "k_encode<int8, classify>", "achieved": achieved,
                     "peak": MFMA_INT8_PEAK_TOPS, "unit": "TOP/s", "frac": achieved / MFMA_INT8_PEAK_TOPS,
                     "traffic": measured_traffic(traffic_key(cls_tile, cls_form), N, cls_tile),
                     "tile": cls_tile, "form": cls_form,
                     "traffic_unit": "bytes per launch (HBM read + write, profiles/traffic.json)",
                     "ms_per_launch": ms_kernel,
                     "ops_per_launch": ops},
    }

    only = set(x for x in args.only.split(",") if x)

    def want(name):
        return not args.no_extras and (not only or name in only)

    if want("train"):
        # -------------------------------------------------------- training
        ms_train, _, _ = event_loop(train, 5, 1)
        _, ms_bundle_tr, _ = event_loop(lambda: hdc.bundle(Htr, D, ytr, K, ws_b), 20, 3)
        out["train"] = {"ms": ms_train, "n_train": int(Xtr.shape[0]), "bundle_ms": ms_bundle_tr,
                        "encode_form": tiles_in_use["encode_form"],
                        "note": "encode of the training set + majority bundle (bundle_ms: the bundle alone, "
                                "device time)"}
    if want("bundle"):
        # -------------------------------------------------------- bundling at HBM scale
        out["bundle"] = bundle_bench(dev, hdc, torch, event_loop)
    if want("sweep"):
        # -------------------------------------------------------- sweep + tuned selection
        grid = [(d, k, 0, t) for (d, k, t) in dg.sweep_grid()]
        tuner.sweep(Xsd, F, ysd, Pd, D, Cw, slots, tile=sweep_tile)   # warm-up launch
        torch.cuda.synchronize()
        t = time.perf_counter()
        res = tuner.sweep(Xsd, F, ysd, Pd, D, Cw, slots, tile=sweep_tile)
        sweep_wall_ms = (time.perf_counter() - t) * 1e3
        # device time of the launch (configurations up, slot setup, class
        # operands, persistent kernel, results down into pinned memory) with
        # events on the launch stream
        sweep_out = torch.empty(16 * len(slots), dtype=torch.uint8, pin_memory=True)
        ws_sw = torch.empty(hdc.lib().hdc_eval_configs_workspace_bytes(len(slots), F, D, K), dtype=torch.uint8,
                            device=dev)
        # the configuration table is built once and reused by each launch
        arrs = {t: hdc.config_array(slots, t) for t in (0, SWEEP_SHARED, sweep_tile)}
        sweep_ms_by = {}
        for t in (0, SWEEP_SHARED):
            _, sweep_ms_by[t], _ = event_loop(lambda: hdc.eval_configs(Xsd, F, ysd, Pd, D, Cw, arrs[t], ws=ws_sw,
                                                                       out=sweep_out), 5, 1)
        sweep_ms = sweep_ms_by.get(sweep_tile) or event_loop(
            lambda: hdc.eval_configs(Xsd, F, ysd, Pd, D, Cw, arrs[sweep_tile], ws=ws_sw, out=sweep_out), 5, 1)[1]
        # algorithmic encode work of the 256 slots: 2 F |S| per query
        sweep_ops = sum(2.0 * F * hdc.dims_count(s_, d_, k_) * Xsd.shape[0] for (d_, k_, s_, _) in slots)
        # what the shared path encodes: the union of the slots' sets once for
        # the int8 / bf16 slots and once for the E4M3 slots
        shared_ops = sum(2.0 * F * D * Xsd.shape[0] for dt in ("int8", "fp8")
                         if any(s_[3] in ((dt, "bf16") if dt == "int8" else (dt,)) for s_ in slots))
        grid_res = tuner.sweep(Xsd, F, ysd, Pd, D, Cw, grid, tile=sweep_tile)
        best, plain_r = tuner.select_tuned(
            grid_res, (D, 1, 0, "int8"), 1.0,
            timer=lambda c: tuner.time_config(c, Xqd, F, Pd, D, Cw, tile=cls_tile_id,
                                              shifted=shifted_P if cls_form == "int8shift" else None))
        pc_ms, sh_ms = sweep_ms_by[0], sweep_ms_by[SWEEP_SHARED]
        out["sweep"] = {"slots": len(slots), "distinct": len(set(slots)), "queries": int(Xsd.shape[0]),
                        "tile": hdc.TILE_NAMES["sweep"].get(sweep_tile, "built-in"),
                        "ms": sweep_ms, "wall_ms": sweep_wall_ms, "one_call": True,
                        "per_config_ms": pc_ms, "shared_ms": sh_ms, "shared_speedup": pc_ms / sh_ms,
                        "roofline": {"bound": "mfma", "achieved": sweep_ops / (pc_ms / 1e3) / 1e12,
                                     "peak": MFMA_INT8_PEAK_TOPS, "unit": "TOP/s",
                                     "frac": sweep_ops / (pc_ms / 1e3) / 1e12 / MFMA_INT8_PEAK_TOPS,
                                     "ops_per_launch": sweep_ops,
                                     "note": "per-configuration path: sum over slots of 2 F |S| x queries "
                                             "(int8 peak for every slot dtype; bf16 slots run at half that "
                                             "rate)"},
                        "shared_roofline": {"bound": "mfma", "achieved": shared_ops / (sh_ms / 1e3) / 1e12,
                                            "peak": MFMA_INT8_PEAK_TOPS, "unit": "TOP/s",
                                            "frac": shared_ops / (sh_ms / 1e3) / 1e12 / MFMA_INT8_PEAK_TOPS,
                                            "ops_per_launch": shared_ops,
                                            "note": "shared path: the two encodings of the union (2 F D x "
                                                    "queries each) over the whole call; the masked Hamming "
                                                    "search (FP4 matrix cores) is not counted"}}
        d, k, s, tdt = best.cfg
        t_form = cls_form if tdt == "int8" else tdt
        if tdt == "fp8" and cls_form == "int8shift" and "fp8" in shifted_P:
            t_form = "fp8shift"
        P_t = shifted_P.get(tdt, Pd) if t_form.endswith("shift") else Pd
        tuned = hdc.Prepared(Cw, D, t_form, s, d, k, tile=cls_tile_id if tdt == "int8" else 0)
        tl = torch.empty(N, dtype=torch.int32, device=dev)
        ms_t, ms_tk, _ = event_loop(lambda: tuned(Xqd, F, P_t, tl), args.steps, args.warmup)
        acc_t = float((tl == yqd).float().mean().item())
        out["tuned"] = {"config": {"d_trunc": d, "stride": k, "start": s, "dtype": tdt},
                        "value": N / (ms_t / 1e3), "ms_per_step": ms_t, "accuracy": acc_t,
                        "speedup_vs_plain": ms_step / ms_t,
                        "sweep_accuracy": best.accuracy, "sweep_accuracy_plain": plain_r.accuracy,
                        "rule": "fastest grid config with sweep accuracy >= plain - 1 pt"}
        log("tuned %s: %.3f ms/step, acc %.4f, speedup %.2fx" % (best.cfg, ms_t, acc_t, ms_step / ms_t))
        # -------------------------------------------------------- latency at config size
        lat = {}
        nte = int(Xte.shape[0])
        for name, prep, Pp in (("plain", plain, P_cls), ("tuned", tuned, P_t)):
            lab = torch.empty(nte, dtype=torch.int32, device=dev)
            for _ in range(10):
                prep(Xte, F, Pp, lab)
            torch.cuda.synchronize()
            ts = []
            for _ in range(args.latency_calls):
                t = time.perf_counter()
                prep(Xte, F, Pp, lab)
                torch.cuda.synchronize()
                ts.append((time.perf_counter() - t) * 1e3)
            lat[name] = {"p50_ms": float(np.percentile(ts, 50)), "p99_ms": float(np.percentile(ts, 99)),
                         "queries_per_call": nte}
        out["latency"] = lat
        out["p99_ms"] = lat["plain"]["p99_ms"]
    if want("hamming"):
        # -------------------------------------------------------- unfused Hamming search
        # packed query hypervectors (2^20 rows) against resident class bits:
        # bytes = the queries read once (class words are cached), HBM-bound.
        # "mfma": prepared classes on the matrix cores; "popcount": the
        # workspace-free search.
        ham = {}
        for name, (Kh, nbits) in (("speech K=26 D=10240", (26, 10240)), ("image K=10 D=8192", (10, 8192)),
                                  ("K=100 D=10240", (100, 10240))):
            nq = 1 << 20
            W = nbits // 64
            Q = torch.randint(-(1 << 62), 1 << 62, (nq, W), dtype=torch.int64, device=dev)
            Ch = torch.randint(-(1 << 62), 1 << 62, (Kh, W), dtype=torch.int64, device=dev)
            lab_h = torch.empty(nq, dtype=torch.int32, device=dev)
            lab_p = torch.empty(nq, dtype=torch.int32, device=dev)
            hp = hdc.HammingPrepared(Ch, 0, nbits, 1)
            row = {"queries": nq}
            for kind, fn in (("mfma", lambda: hp(Q, out=lab_h)),
                             ("popcount", lambda: hdc.lib().hdc_hamming_argmin(
                                 hdc._stream(), hdc._ptr(Q), nq, W, hdc._ptr(Ch), Kh, W, nbits, hdc.Dims(0, nbits, 1),
                                 hdc._ptr(lab_p), None, None))):
                _, ms_hk, _ = event_loop(fn, 10, 2)
                gbs = nq * W * 8 / (ms_hk / 1e3) / 1e9
                row[kind] = {"ms": ms_hk, "GB_s": gbs, "frac_of_hbm_peak": gbs / HBM_PEAK_GBS,
                             "queries_per_s": nq / (ms_hk / 1e3)}
            row["agree"] = bool(torch.equal(lab_h, lab_p))
            ham[name] = row
            del Q, Ch, hp
        out["hamming_unfused"] = ham
        log("hamming GB/s: %s" % {k: (round(v["mfma"]["GB_s"], 1), round(v["popcount"]["GB_s"], 1), v["agree"])
                                  for k, v in ham.items()})
    if want("plain_fp32"):
        # -------------------------------------------------------- the plain fp32 workload
        out["plain_fp32"] = plain_fp32(dev, dg, hdc, torch, event_loop, N)
    if want("adc"):
        # -------------------------------------------------------- ADC-chunked similarity
        out["adc"] = adc_emulation(dev, hdc, torch, event_loop, ds, Xte, Pd, Cw, F, D)
    if want("cosine"):
        # -------------------------------------------------------- cosine similarity
        out["cosine"] = cosine_similarity(dev, hdc, torch, event_loop, ds, Xtr, ytr, Xte, Pd, F, K, D)
    if want("encode_side"):
        # -------------------------------------------------------- encode-side knobs
        out["encode_side"] = encode_side(dev, hdc, dg, torch, np, event_loop, sp, Xtr, ytr, Xte, Pd, Xqd, yqd,
                                         F, K, D)
    if want("retrain"):
        # -------------------------------------------------------- retraining epochs
        out["retrain"] = retraining(dev, hdc, torch, event_loop, ds, Xtr, ytr, Xte, Pd, F, K, D)
    if want("ladder"):
        # -------------------------------------------------------- precision ladder
        out["ladder"] = ladder(dev, dg, hdc, tuner, torch, np, event_loop, ds, Xte, Pd, Cw, Xqd, F, D)
    if want("serving"):
        # -------------------------------------------------------- serving
        if args.serve_seconds > 0:
            out["serving"] = serving(args, dev, dg, hdc, tuner, torch)

    if args.ceilings:
        # ------------------------------------------------------------ device ceilings
        from paper_2606_26547_amd import ceilings
        out["ceilings"] = ceilings.measure()
        log("ceilings: %s" % out["ceilings"])

    # ------------------------------------------------------------ CPU oracle

    if not args.no_cpu:
        from oracle import oracle as O
        n_cpu = min(args.cpu_sample, N)
        Cref = Cw.cpu().numpy().view(np.uint64)
        t = time.perf_counter()
        lab_cpu = O.classify(Xq[:n_cpu], ds.P, Cref)
        dt = time.perf_counter() - t
        agree = float((lab_cpu == labels[:n_cpu].cpu().numpy()).mean())
        out["cpu_baseline"] = {"value": n_cpu / dt, "unit": "queries/s", "cores": O.threads(), "kind": "oracle",
                               "cpu_model": cpu_model(), "host_cpus": os.cpu_count(),
                               "sample": "first %d queries of the batch, plain config (exact int encode + "
                                         "bit-by-bit Hamming + argmin), %.1fs" % (n_cpu, dt),
                               "labels_agree_with_gpu": agree}
        # the tuned configuration on a smaller sample, and one thread
        if "tuned" in out:
            tc = out["tuned"]["config"]
            n_t = max(1, n_cpu // 3)
            t = time.perf_counter()
            O.classify(Xq[:n_t], ds.P, Cref, tc["dtype"], tc["start"], tc["d_trunc"], tc["stride"])
            out["cpu_baseline"]["tuned_value"] = n_t / (time.perf_counter() - t)
        n_1 = 1024
        t = time.perf_counter()
        O.classify(Xq[:n_1], ds.P, Cref, threads=1)
        out["cpu_baseline"]["single_thread_value"] = n_1 / (time.perf_counter() - t)
        log("cpu oracle: %.1f q/s on %d threads (agree %.4f), tuned %.1f q/s, one thread %.1f q/s" %
            (n_cpu / dt, O.threads(), agree, out["cpu_baseline"].get("tuned_value", 0.0),
             out["cpu_baseline"]["single_thread_value"]))
        if not args.no_extras and not only:
            out["cpu_baseline"]["rows"] = oracle_rows(O, np, ds, F, K, D)

    out["full_record"] = args.full_out
    try:
        os.makedirs(os.path.dirname(args.full_out), exist_ok=True)
        with open(args.full_out, "w") as f:
            json.dump(out, f, indent=1)
    except OSError as e:
        log("could not write the full record to %s: %s" % (args.full_out, e))
        out["full_record"] = None
    print(json.dumps(compact(out)), flush=True)


def plain_fp32(dev, dg, hdc, torch, event_loop, N):
    """The plain fp32 workload (64 fp32 features, 10 classes, D = 2048, no
    approximation): fp32 encode of the 1000 training vectors, majority
    bundle, fused fp32 classify of the 200 test vectors, then a batch of N
    further queries of the same mixture for throughput (fp32 MFMA)."""
    d = dg.config_c1(1)
    F, K, D = d.X_train.shape[1], d.K, d.P.shape[0]
    Pd = hdc.pad_cols(d.P, dev)
    Xtr, Xte = hdc.pad_cols(d.X_train, dev), hdc.pad_cols(d.X_test, dev)
    ytr = torch.as_tensor(d.y_train).to(dev)
    Htr = hdc.encode(Xtr, F, Pd, D, "fp32")
    Cw, _ = hdc.bundle(Htr, D, ytr, K)
    lab = hdc.classify(Xte, F, Pd, D, Cw, "fp32")
    acc = float((lab.cpu().numpy() == d.y_test).mean())
    Xq, yq = dg.c1_queries(N, 1, stream=3)
    Xqd = hdc.pad_cols(Xq, dev)
    prep = hdc.Prepared(Cw, D, "fp32")
    lq = torch.empty(N, dtype=torch.int32, device=dev)
    _, ms, _ = event_loop(lambda: prep(Xqd, F, Pd, lq), 10, 2)
    acc_b = float((lq.cpu().numpy() == yq).mean())
    flops = 2.0 * F * D * N
    tf = flops / (ms / 1e3) / 1e12
    log("plain fp32: test accuracy %.3f, batch %d: %.3f ms, %.3e q/s, %.1f TFLOP/s" % (acc, N, ms, N / ms * 1e3, tf))
    del Xqd
    return {"F": F, "K": K, "D": D, "test_accuracy": acc, "batch": N, "batch_accuracy": acc_b, "ms": ms,
            "queries_per_s": N / (ms / 1e3),
            "roofline": {"bound": "mfma", "achieved": tf, "peak": MFMA_FP32_PEAK_TFLOPS, "unit": "TFLOP/s",
                         "frac": tf / MFMA_FP32_PEAK_TFLOPS, "flops_per_launch": flops,
                         "note": "2 F D per query on v_mfma_f32_32x32x2_f32 (fp32 dense peak)"}}


def bundle_bench(dev, hdc, torch, event_loop, n=1 << 20, nbits=10240, K=26):
    """Majority bundling of 2^20 random 10240-bit rows (1.34 GB) into 26
    classes, random labels: HBM-bound (every row read once)."""
    W = nbits // 64
    H = torch.randint(-(1 << 62), 1 << 62, (n, W), dtype=torch.int64, device=dev)
    y = torch.randint(0, K, (n,), dtype=torch.int32, device=dev)
    ws = torch.empty(hdc.lib().hdc_bundle_workspace_bytes(n, nbits, K), dtype=torch.uint8, device=dev)
    _, ms, _ = event_loop(lambda: hdc.bundle(H, nbits, y, K, ws), 10, 2)
    nbytes = n * W * 8 + n * 4 + K * W * 8        # rows + labels read, class words written
    gbs = nbytes / (ms / 1e3) / 1e9
    log("bundle 2^20 x %d bits: %.3f ms, %.0f GB/s" % (nbits, ms, gbs))
    del H
    return {"rows": n, "nbits": nbits, "K": K, "ms": ms, "GB_s": gbs,
            "roofline": {"bound": "hbm", "achieved": gbs, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                         "frac": gbs / HBM_PEAK_GBS, "bytes_per_launch": nbytes,
                         "note": "algorithmic bytes: every row and label read once, class words written"}}


def oracle_rows(O, np, ds, F, K, D):
    """The oracle timed on a bounded sample of each path beside the headline
    one (same shapes as the GPU figures in the sections above; seeded
    random operands, whose values do not change the oracle's work)."""
    g = np.random.default_rng(77)
    W = D // 64
    rows = {}

    def timed(name, n, unit, fn, sample):
        t = time.perf_counter()
        fn()
        dt = time.perf_counter() - t
        rows[name] = {"value": n / dt, "unit": unit, "cores": O.threads(), "kind": "oracle",
                      "sample": "%s, %.2fs" % (sample, dt)}

    Q = g.integers(0, 2 ** 63, size=(1 << 18, W), dtype=np.int64).view(np.uint64)
    C = g.integers(0, 2 ** 63, size=(K, W), dtype=np.int64).view(np.uint64)
    acc = g.integers(-300, 301, size=(K, D), dtype=np.int32)
    timed("hamming_search", 1 << 18, "queries/s", lambda: O.argmin(O.hamming_popcount(Q, C, 0, D, 1)),
          "262144 queries x %d classes x %d bits, popcount distances + argmin" % (K, D))
    timed("cosine", 4096, "queries/s", lambda: O.argmax_f64(O.cosine_scores(Q[:4096], acc, 0, D, 1)),
          "4096 queries x %d classes x %d dimensions" % (K, D))
    timed("adc", 4096, "queries/s", lambda: O.argmax(O.adc_scores(Q[:4096], C, 0, D, 1, 8, 2, -3, 128)),
          "4096 queries, ADC (8, 2, -3, 128)")
    X = np.ascontiguousarray(ds.X_train[:4096])
    timed("feature_perforation_stride2", 4096, "queries/s", lambda: O.encode_fperf(X, ds.P, 0, F, 2),
          "4096 speech rows, feature stride 2, D = %d" % D)
    L = 128
    lev = g.integers(0, L, size=(256, F)).astype(np.uint16)
    IDh = g.integers(0, 2 ** 63, size=(F, W), dtype=np.int64).view(np.uint64)
    LVh = g.integers(0, 2 ** 63, size=(L, W), dtype=np.int64).view(np.uint64)
    timed("level_id_encode", 256, "rows/s", lambda: O.level_id_encode(lev, IDh, LVh, D),
          "256 rows x %d features, L = %d, D = %d" % (F, L, D))
    n_tr = ds.X_train.shape[0]
    H = g.integers(0, 2 ** 63, size=(n_tr, W), dtype=np.int64).view(np.uint64)
    acc_tr = O.class_acc(H, ds.y_train, K, D)

    def epochs():
        for _ in range(20):
            pred, _ = O.argmin(O.hamming_popcount(H, O.binarize(acc_tr, D), 0, D, 1))
            O.retrain_epoch(H, ds.y_train, pred, acc_tr, D)
    timed("retrain_epoch", 20 * n_tr, "training rows/s", epochs,
          "20 epochs over %d training rows (predict + update), D = %d" % (n_tr, D))
    log("cpu oracle rows: %s" % {k: "%.3g %s" % (v["value"], v["unit"]) for k, v in rows.items()})
    return rows


def adc_emulation(dev, hdc, torch, event_loop, ds, Xte, Pd, Cw, F, D):
    """Dot-product similarity over 128-element chunks with ADC quantisation
    (the in-memory accelerator knobs): test accuracy of the speech model for
    the paper's reference ADC setting and the settings its tuner picked, and
    the search throughput on 2^20 query hypervectors."""
    yte = torch.as_tensor(ds.y_test).to(dev)
    Hte = hdc.encode(Xte, F, Pd, D)
    settings = {"reference 8b step1 [-127,128]": (8, 1, -127, 128), "tuned 8b step2 [-3,128]": (8, 2, -3, 128),
                "6b step9 [-3,128]": (6, 9, -3, 128), "4b step16 [-127,128]": (4, 16, -127, 128)}
    res = {"hamming_accuracy": float((hdc.hamming_argmin(Hte, Cw, 0, D, 1)[0] == yte).float().mean().item())}
    for name, a in settings.items():
        lab, _, _ = hdc.adc_argmax(Hte, Cw, 0, D, 1, a)
        res[name] = {"adc": list(a), "accuracy": float((lab == yte).float().mean().item())}
    nq = 1 << 20
    Q = torch.randint(-(1 << 62), 1 << 62, (nq, D // 64), dtype=torch.int64, device=dev)
    _, ms, _ = event_loop(lambda: hdc.adc_argmax(Q, Cw, 0, D, 1, (8, 2, -3, 128)), 5, 1)
    res["search_2^20"] = {"ms": ms, "GB_s": nq * D / 8 / (ms / 1e3) / 1e9, "queries_per_s": nq / (ms / 1e3),
                          "form": "one call, VALU popcount partials"}
    # prepared form: partials on FP4 matrix cores, the ADC table on the VALU
    ap = hdc.AdcPrepared(Cw, 0, D, 1)
    lab_p = torch.empty(nq, dtype=torch.int32, device=dev)
    _, ms_p, _ = event_loop(lambda: ap(Q, (8, 2, -3, 128), out=lab_p), 5, 1)
    res["search_2^20_prepared"] = {"ms": ms_p, "GB_s": nq * D / 8 / (ms_p / 1e3) / 1e9,
                                   "queries_per_s": nq / (ms_p / 1e3),
                                   "agrees_with_one_call": bool(torch.equal(
                                       lab_p, hdc.adc_argmax(Q, Cw, 0, D, 1, (8, 2, -3, 128))[0]))}
    # the prepared search's bound: per (query, class, 128-dimension chunk)
    # the partial's conversion, table index and add on the VALU (3
    # operations; the two FP4 MFMAs per chunk and tile take less time)
    ops = nq * Cw.shape[0] * (D / 128) * 3
    res["roofline"] = {"bound": "alu", "kernel": "k_adc_mfma", "achieved": ops / (ms_p / 1e3) / 1e12,
                       "peak": VALU_PEAK_TOPS, "unit": "TOP/s", "frac": ops / (ms_p / 1e3) / 1e12 / VALU_PEAK_TOPS,
                       "ops_per_launch": ops}
    del Q
    log("adc: %s" % {k: (v["accuracy"] if isinstance(v, dict) and "accuracy" in v else v) for k, v in res.items()})
    return res


def cosine_similarity(dev, hdc, torch, event_loop, ds, Xtr, ytr, Xte, Pd, F, K, D):
    """Cosine similarity against the integer class accumulators (no
    binarisation) beside Hamming against their signs: test accuracy of the
    speech model after bundling and after retraining, under truncation and
    perforation, and the search throughput on 2^20 query hypervectors."""
    from paper_2606_26547_amd import train
    H = hdc.encode(Xtr, F, Pd, D)
    Hte = hdc.encode(Xte, F, Pd, D)
    yte = torch.as_tensor(ds.y_test).to(dev)
    res = {}
    for epochs in (0, 3):
        Cw, acc, _ = train.fit(H, D, ytr, K, epochs)
        row = {"max_abs_acc": int(acc.abs().max().item())}
        for name, (s, e, k) in {"full": (0, D, 1), "D'=4096": (0, 4096, 1), "stride 4": (0, D, 4)}.items():
            ham = hdc.HammingPrepared(Cw, s, e, k)(Hte)[0]
            cos = hdc.CosinePrepared(acc, s, e, k)(Hte)[0]
            row[name] = {"hamming": float((ham == yte).float().mean().item()),
                         "cosine": float((cos == yte).float().mean().item())}
        res["epochs=%d" % epochs] = row
    nq = 1 << 20
    Q = torch.randint(-(1 << 62), 1 << 62, (nq, D // 64), dtype=torch.int64, device=dev)
    lab = torch.empty(nq, dtype=torch.int32, device=dev)
    cp = hdc.CosinePrepared(acc, 0, D, 1)
    _, ms, _ = event_loop(lambda: cp(Q, out=lab), 10, 2)
    res["search_2^20"] = {"ms": ms, "GB_s": nq * D / 8 / (ms / 1e3) / 1e9, "queries_per_s": nq / (ms / 1e3),
                          "int8_tops": 2 * nq * D * 32 * 2 / (ms / 1e3) / 1e12}
    # matrix cores: two parts of each class sum times 32 queries, 32 dimensions
    # and a class tile of 32, 2 * 2 * n * D * 32 ops executed for K <= 32: on
    # FP6 digits while the sums over S stay within +-255, else in int8 (the
    # peak the rate is put against)
    ops = 2 * 2 * nq * D * 32
    res["roofline"] = {"bound": "mfma", "achieved": ops / (ms / 1e3) / 1e12, "peak": MFMA_INT8_PEAK_TOPS,
                       "unit": "TOP/s", "frac": ops / (ms / 1e3) / 1e12 / MFMA_INT8_PEAK_TOPS, "ops_per_launch": ops,
                       "algorithmic_ops_per_launch": 2 * nq * D * K}
    del Q
    log("cosine: %s, 2^20 search %.3f ms" % ({k: v["full"] for k, v in res.items() if k.startswith("epochs")}, ms))
    return res


def encode_side(dev, hdc, dg, torch, np, event_loop, sp, Xtr, ytr, Xte, Pd, Xqd, yqd, F, K, D):
    """The encoder's own knobs on the speech workload: (a) perforating the
    reduction over features (gather the columns, encode, bundle, classify)
    -- test accuracy and the time of gather + fused classify on the bench
    batch; (b) Level-ID encoding from the unquantised features -- test
    accuracy for a few (levels, D) and the time of quantise + encode +
    prepared Hamming search on the bench batch."""
    yte = torch.as_tensor(sp.float_split()[3]).to(dev)
    res = {"feature_perforation": {}, "level_id": {}}
    n = Xqd.shape[0]
    lab = torch.empty(n, dtype=torch.int32, device=dev)
    for k in (1, 2, 4):
        nf = hdc.dims_count(0, F, k)
        Pg = hdc.feature_perforate(Pd, F, 0, F, k)
        Htr = hdc.encode(hdc.feature_perforate(Xtr, F, 0, F, k), nf, Pg, D)
        Cw, _ = hdc.bundle(Htr, D, ytr, K)
        acc_te = float((hdc.classify(hdc.feature_perforate(Xte, F, 0, F, k), nf, Pg, D, Cw) == yte)
                       .float().mean().item())
        prep = hdc.Prepared(Cw, D, "int8")
        Xg = torch.empty((n, max(64, (nf + 63) // 64 * 64)), dtype=torch.int8, device=dev)

        def step():
            hdc.feature_perforate(Xqd, F, 0, F, k, out=Xg)
            prep(Xg, nf, Pg, lab)
        ms_wall, ms, _ = event_loop(step, 5, 1)
        ops = 2.0 * n * nf * D                 # algorithmic encode ops of the perforated product
        res["feature_perforation"]["stride %d" % k] = {
            "features": nf, "test_accuracy": acc_te, "batch_accuracy": float((lab == yqd).float().mean().item()),
            "ms": ms, "queries_per_s": n / (ms / 1e3),
            "roofline": {"bound": "mfma", "achieved": ops / (ms / 1e3) / 1e12, "peak": MFMA_INT8_PEAK_TOPS,
                         "unit": "TOP/s", "frac": ops / (ms / 1e3) / 1e12 / MFMA_INT8_PEAK_TOPS,
                         "note": "gather + fused classify per batch"}}
    Xtr_f, ytr_f, Xte_f, _ = sp.float_split()
    lo, hi = dg.feature_ranges(Xtr_f)
    lo_d, hi_d = torch.as_tensor(lo).to(dev), torch.as_tensor(hi).to(dev)
    Xtr_d, Xte_d = torch.as_tensor(Xtr_f).to(dev), torch.as_tensor(Xte_f).to(dev)
    Xq_f = torch.as_tensor(sp.mix.sample(yqd.cpu().numpy(), dg.rng(2, 99))).to(dev)
    for L, Dl in ((16, 1024), (128, 1024), (128, 10240)):
        ID = torch.as_tensor(dg.id_hypervectors(F, Dl, 21).view(np.int64)).to(dev)
        LV = torch.as_tensor(dg.level_hypervectors(L, Dl, 22).view(np.int64)).to(dev)
        Htr = hdc.level_id_encode(hdc.level_quantize(Xtr_d, lo_d, hi_d, L), ID, LV, Dl)
        Cw, _ = hdc.bundle(Htr, Dl, ytr, K)
        Hte = hdc.level_id_encode(hdc.level_quantize(Xte_d, lo_d, hi_d, L), ID, LV, Dl)
        hp = hdc.HammingPrepared(Cw, 0, Dl, 1)
        acc_te = float((hp(Hte)[0] == yte).float().mean().item())
        lev = hdc.level_quantize(Xq_f, lo_d, hi_d, L)
        Hq = torch.empty((n, Dl // 64), dtype=torch.int64, device=dev)

        def step():
            hdc.level_quantize(Xq_f, lo_d, hi_d, L, out=lev)
            hdc.level_id_encode(lev, ID, LV, Dl, out=Hq)
            hp(Hq, out=lab)
        ms_wall, ms, _ = event_loop(step, 3, 1)
        _, ms_enc, _ = event_loop(lambda: hdc.level_id_encode(lev, ID, LV, Dl, out=Hq), 3, 1)
        # VALU-bound: about 3 operations per (row, feature, 32 dimensions): 2.8
        # in the carry-save tree, whose first adders bind, and the level address
        ops = n * F * (Dl / 32) * 3
        res["level_id"]["L=%d D=%d" % (L, Dl)] = {
            "test_accuracy": acc_te, "batch_accuracy": float((lab == yqd).float().mean().item()),
            "ms": ms, "queries_per_s": n / (ms / 1e3), "encode_ms": ms_enc,
            "word_features_per_s": n * F * (Dl / 32) / (ms_enc / 1e3),
            "roofline": {"bound": "alu", "achieved": ops / (ms_enc / 1e3) / 1e12, "peak": VALU_PEAK_TOPS,
                         "unit": "TOP/s", "frac": ops / (ms_enc / 1e3) / 1e12 / VALU_PEAK_TOPS,
                         "ops_per_launch": ops}}
    log("encode-side: %s" % {g: {k: (round(v["test_accuracy"], 4), round(v["ms"], 3)) for k, v in r.items()}
                             for g, r in res.items()})
    return res


def retraining(dev, hdc, torch, event_loop, ds, Xtr, ytr, Xte, Pd, F, K, D, epochs=6):
    """Retraining epochs on the speech workload (the apps' TRAIN_ITERATIONS):
    training-set errors and test accuracy after each epoch, and the device
    time of one epoch (predict all 6238 training rows + accumulator update)."""
    from paper_2606_26547_amd import train
    H = hdc.encode(Xtr, F, Pd, D)
    yte = torch.as_tensor(ds.y_test).to(dev)
    acc_by_epoch, wrong = [], []
    for e in range(epochs + 1):
        Cw, _, w = train.fit(H, D, ytr, K, e)
        lab = hdc.classify(Xte, F, Pd, D, Cw)
        acc_by_epoch.append(float((lab == yte).float().mean().item()))
        if w:
            wrong.append(int(w[-1].item()))
    acc, Cw = hdc.class_acc(H, D, ytr, K)
    pred = torch.empty(H.shape[0], dtype=torch.int32, device=dev)

    def epoch():
        hdc.HammingPrepared(Cw, 0, D, 1)(H, out=pred)
        hdc.retrain_epoch(H, D, ytr, pred, acc, Cw)
    _, ms, _ = event_loop(epoch, 5, 1)
    log("retrain: test accuracy by epoch %s, training errors %s, %.3f ms/epoch" %
        ([round(a, 4) for a in acc_by_epoch], wrong, ms))
    return {"test_accuracy_by_epoch": acc_by_epoch, "train_errors_at_epoch_start": wrong, "ms_per_epoch": ms,
            "rule": "mispredicted rows: acc[true] += b, acc[pred] -= b; model = sign(acc)"}


def flip_rate(Ha, Hb, nbits: int) -> float:
    """Fraction of the first nbits bits of each row that differ."""
    a = Ha.cpu().numpy().view(np.uint8)
    b = Hb.cpu().numpy().view(np.uint8)
    diff = np.unpackbits(a ^ b, axis=1, bitorder="little")[:, :nbits]
    return float(diff.mean())


def ladder(dev, dg, hdc, tuner, torch, np_, event_loop, ds, Xte, Pd, Cw, Xqd, F, D):
    """The encoding precision ladder (int8 exact, bf16, fp8 E4M3) on both
    integer workloads: bit flip rate of the query hypervectors against the
    exact int8 encoding, accuracy, and fused-classifier throughput.  Speech:
    its 1559 test queries (throughput on the 262144-query batch).  Image:
    the uint8 workload trained on 60000 images, its 10000 test images, and
    the 27-point (D', stride, dtype) grid of that workload evaluated in one
    launch with the <= 1 point selection rule."""
    res = {}
    yte = torch.as_tensor(ds.y_test).to(dev)
    Hx = hdc.encode(Xte, F, Pd, D, "int8")
    sp = {}
    for t in ("int8", "bf16", "fp8", "fp8split"):
        H = hdc.encode(Xte, F, Pd, D, t)
        lab = hdc.classify(Xte, F, Pd, D, Cw, t)
        prep = hdc.Prepared(Cw, D, t)
        lb = torch.empty(Xqd.shape[0], dtype=torch.int32, device=dev)
        _, ms, _ = event_loop(lambda: prep(Xqd, F, Pd, lb), 5, 1)
        sp[t] = {"flip_rate": flip_rate(H, Hx, D), "accuracy": float((lab == yte).float().mean().item()),
                 "ms_batch": ms, "queries_per_s": Xqd.shape[0] / (ms / 1e3)}
        ts = hdc.SHIFTED.get(t)
        if ts and hdc.shift_supported("classify", F, Cw.shape[0], ts):
            # the same rung on the shifted projection (identical labels)
            Pt = hdc.shift_projection(Pd, F, compute=ts)
            prep_s = hdc.Prepared(Cw, D, ts)
            ls = torch.empty_like(lb)
            _, ms_s, _ = event_loop(lambda: prep_s(Xqd, F, Pt, ls), 5, 1)
            sp[t].update(ms_batch_shifted=ms_s, labels_equal_shifted=bool(torch.equal(ls, lb)))
    res["speech"] = sp
    log("ladder speech: %s" % {t: (round(v["flip_rate"], 5), round(v["accuracy"], 4), round(v["ms_batch"], 3))
                               for t, v in sp.items()})
    img = dg.ImageLike(3).dataset()
    Fi, Ki, Di = img.F, img.K, img.D
    Pi = hdc.pad_cols(img.P, dev)
    Xi_tr = hdc.pad_cols(img.X_train, dev)
    Xi_te = hdc.pad_cols(img.X_test, dev)
    yi_tr = torch.as_tensor(img.y_train, dtype=torch.int32).to(dev)
    yi_te = torch.as_tensor(img.y_test, dtype=torch.int32).to(dev)
    Hi = hdc.encode(Xi_tr, Fi, Pi, Di, "int8")
    Ci, _ = hdc.bundle(Hi, Di, yi_tr, Ki)
    Hx = hdc.encode(Xi_te, Fi, Pi, Di, "int8")
    im = {}
    for t in ("int8", "bf16", "fp8", "fp8split"):
        H = hdc.encode(Xi_te, Fi, Pi, Di, t)
        lab = hdc.classify(Xi_te, Fi, Pi, Di, Ci, t)
        prep = hdc.Prepared(Ci, Di, t)
        lb = torch.empty(Xi_te.shape[0], dtype=torch.int32, device=dev)
        _, ms, _ = event_loop(lambda: prep(Xi_te, Fi, Pi, lb), 5, 1)
        im[t] = {"flip_rate": flip_rate(H, Hx, Di), "accuracy": float((lab == yi_te).float().mean().item()),
                 "ms_10000": ms, "queries_per_s": Xi_te.shape[0] / (ms / 1e3)}
    grid = [(d, k, 0, t) for d in (2048, 4096, 8192) for k in (1, 2, 4) for t in ("int8", "bf16", "fp8")]
    results = tuner.sweep(Xi_te, Fi, yi_te, Pi, Di, Ci, grid)
    best, plain = tuner.select_tuned(results, (Di, 1, 0, "int8"), 1.0,
                                     timer=lambda c: tuner.time_config(c, Xi_te, Fi, Pi, Di, Ci))
    im["grid"] = [{"cfg": list(r.cfg), "accuracy": r.accuracy, "device_us": r.device_us} for r in results]
    im["tuned"] = {"cfg": list(best.cfg), "accuracy": best.accuracy, "accuracy_plain": plain.accuracy}
    res["image"] = im
    log("ladder image: %s; tuned %s" % ({t: (round(v["flip_rate"], 5), round(v["accuracy"], 4)) for t, v in im.items()
                                        if t in ("int8", "bf16", "fp8", "fp8split")}, best.cfg))
    return res


def _bytes(text: str) -> int:
    mult = {"K": 1 << 10, "M": 1 << 20, "G": 1 << 30}
    return int(float(text[:-1]) * mult[text[-1]]) if text[-1] in mult else int(text)


def serving(args, dev, dg, hdc, tuner, torch):
    """The serving loop over the 8 resident serving models, plain and tuned.
    Open loop: a Poisson stream of 2000 requests/s, 95% inference requests of
    1..4096 queries (log-uniform), 5% configuration jobs (16 configurations
    x 512 labelled queries), at each HBM budget for in-flight requests (16 GiB:
    admission never waits; small budgets make it wait); p50 / p99 latency from
    arrival to labels on the host, completed queries per second, peak admitted
    bytes and how many requests waited for budget.  Closed loop: 64
    inference requests kept outstanding, the sustained queries per second
    (the capacity, which the open-loop rate does not reach)."""
    from paper_2606_26547_amd import serve

    srcs = dg.serving_models(5)
    models = [serve.ResidentModel(s.P, s.X_train, s.y_train, s.K) for s in srcs]
    tuned_cfgs = []
    for s, m in zip(srcs, models):
        # per-model tuning: the 24-point grid (D', stride, encoding type) on
        # 2048 labelled queries in one sweep call (shared path), then the
        # cheapest candidates within 1 point re-timed on a 4096-query batch
        Xv, yv = s.queries(2048, 900)
        Xt = hdc.pad_cols(s.queries(4096, 901)[0], dev)
        grid = [(d, k, 0, t) for d in sorted({m.D, m.D // 2, m.D // 4, m.D // 8}) for k in (1, 2)
                for t in ("int8", "bf16", "fp8")]
        res = tuner.sweep(hdc.pad_cols(Xv, dev), m.F, torch.as_tensor(yv).to(dev), m.P, m.D, m.C, grid,
                          tile=SWEEP_SHARED)
        best, plain = tuner.select_tuned(res, (m.D, 1, 0, "int8"), 1.0, max_timed=6,
                                         timer=lambda c, m=m, Xt=Xt: tuner.time_config(c, Xt, m.F, m.P, m.D, m.C,
                                                                                       shifted=m.shifted))
        m.set_tuned(best.cfg)
        tuned_cfgs.append({"F": m.F, "K": m.K, "D": m.D, "tuned": list(best.cfg),
                           "acc_plain": plain.accuracy, "acc_tuned": best.accuracy,
                           "qps_4096_plain": plain.qps, "qps_4096_tuned": best.qps})
    torch.cuda.synchronize()

    def job_cfgs(mi):
        D = models[mi].D
        return [(d, k, 0, t) for d in (D, D // 2, D // 4, D // 8) for k in (1, 2) for t in ("int8", "fp8")]

    budgets = [b for b in args.serve_budgets.split(",") if b]
    report = {"models": tuned_cfgs, "rate_req_s": 2000.0, "seconds": args.serve_seconds,
              "resident_bytes": sum(m.resident_bytes for m in models), "budgets": budgets}
    for mode in ("plain", "tuned"):
        ex = serve.GpuExecutor(models)
        tiles = ex.warm(job_cfgs, tune_tiles=(mode == "plain"))
        if tiles:
            report["tiles"] = {"%s F=%d K=%d D=%d" % (c.shape.kind, c.shape.F, c.shape.K, c.shape.D): c.chosen_name
                               for c in tiles}
        runs = {}
        for bname in budgets:
            srv = serve.Server(ex, budget=_bytes(bname), poll_s=args.serve_poll_us * 1e-6)
            # a short untimed stream first (staging slots, allocator caches)
            for _, f in serve.open_loop(srv, srcs, 2000.0, 0.3, seed=99, tuned=(mode == "tuned"),
                                        job_cfgs=job_cfgs):
                f.result(timeout=300)
            srv.completed.clear()
            srv.sched.blocked = 0
            srv.max_loop_s, srv.loop_stalls = 0.0, 0
            t0 = time.perf_counter()
            futs = serve.open_loop(srv, srcs, 2000.0, args.serve_seconds, seed=7, tuned=(mode == "tuned"),
                                   job_cfgs=job_cfgs)
            for _, f in futs:
                f.result(timeout=300)
            wall = time.perf_counter() - t0
            srv.close()
            rep = srv.latency_report("infer")
            rep["configs_jobs"] = srv.latency_report("configs")
            rep["queries_per_s"] = rep.get("queries", 0) / wall
            rep["peak_admitted_bytes"] = srv.sched.peak_used
            rep["waited_for_budget"] = srv.sched.blocked
            rep["max_loop_ms"] = srv.max_loop_s * 1e3
            rep["loop_passes_over_10ms"] = srv.loop_stalls
            rep["staging_slots"] = ex.nslots
            runs[bname] = rep
            log("serving %s %s: p50 %.3f ms p99 %.3f ms, %d requests, %.0f q/s, %d waited for budget, "
                "longest loop pass %.1f ms (%d over 10 ms), %d staging slots" %
                (mode, bname, rep.get("p50_ms", -1), rep.get("p99_ms", -1), rep.get("requests", 0),
                 rep["queries_per_s"], rep["waited_for_budget"], rep["max_loop_ms"], rep["loop_passes_over_10ms"],
                 ex.nslots))
        if args.serve_saturation_seconds > 0:
            srv = serve.Server(ex, budget=16 << 30, poll_s=args.serve_poll_us * 1e-6)
            q, wall = serve.closed_loop(srv, srcs, 64, args.serve_saturation_seconds, seed=21,
                                        tuned=(mode == "tuned"))
            srv.close()
            runs["saturation"] = {"concurrency": 64, "queries_per_s": q / wall, "seconds": wall}
            log("serving %s saturation: %.0f q/s" % (mode, q / wall))
            # the same with every request at the largest size (4096 queries):
            # per-request host work is amortised, so the device sets the pace
            srv = serve.Server(ex, budget=16 << 30, poll_s=args.serve_poll_us * 1e-6)
            q, wall = serve.closed_loop(srv, srcs, 16, args.serve_saturation_seconds, seed=22,
                                        tuned=(mode == "tuned"), fixed_n=4096)
            srv.close()
            runs["saturation_4096"] = {"concurrency": 16, "request_queries": 4096, "queries_per_s": q / wall,
                                       "seconds": wall}
            log("serving %s saturation, 4096-query requests: %.0f q/s" % (mode, q / wall))
        # the first budget's run is the headline of this mode
        report[mode] = dict(runs[budgets[0]], runs=runs) if budgets else {"runs": runs}
    return report


if __name__ == "__main__":
    main()

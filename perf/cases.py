"""Performance cases of the HDC classification framework.

Each case is one pass of work that a program built on this framework does,
through the public entry points of ``paper_2606_26547_amd`` (``hdc``,
``train``): inference under the approximation knobs, training, the
similarity searches, Level-ID encoding and the configuration sweep.  Sizes
are those of the framework's own workloads (speech: 617 features, 26
classes, 10240 dimensions; image: 784 uint8 features, 10 classes, 8192
dimensions; plain: 64 fp32 features; the resident models of the serving
loop); ``draw`` varies them.  Every input is made on the GPU from the seed.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2606_26547_amd import hdc, train

DEV = "cuda"
TILE_SHARED = 4          # sweep tile: the one the tile autotuner picks for every sweep bucket
SWEEP_TYPES = ("int8", "bf16", "fp8")
SWEEP_STRIDES = (1, 2, 4, 8)
ADC_REFERENCE = (8, 1, -127, 128)
ADC_COARSE = (6, 9, -3, 128)
ADC_FINE = (8, 2, -3, 128)
# the serving loop's resident models: (features, classes, dimensions)
MODELS = ((64, 2, 1024), (96, 5, 1024), (128, 10, 2048), (256, 26, 4096), (512, 50, 8192), (617, 26, 10240),
          (784, 10, 8192), (1024, 100, 16384))


def listed():
    return [
        # one small call: the plain workload's fp32 test set, classes prepared
        # in the call; latency and launches are what it costs
        dict(name="plain_fp32_call", kind="classify", n=200, F=64, K=10, D=2048, x="float32", types="fp32",
             start=0, end=2048, stride=1, dists=False),
        # the speech test set against a resident model: one serving request
        dict(name="speech_request", kind="infer", n=1559, F=617, K=26, D=10240, x="int8", types="int8",
             start=0, end=10240, stride=1, dists=False),
        # bulk inference of the same model (the benchmark's batch) on the
        # projection form its autotuner picks
        dict(name="speech_batch", kind="infer", n=262144, F=617, K=26, D=10240, x="int8", types="int8shift",
             start=0, end=10240, stride=1, dists=False),
        # the image test set, uint8 pixels, one call with the distances
        dict(name="image_test", kind="classify", n=10000, F=784, K=10, D=8192, x="uint8", types="int8",
             start=0, end=8192, stride=1, dists=True),
        # the reduced element types on a batch: bf16, then E4M3, under a
        # truncated and perforated dimension set
        dict(name="speech_reduced_types", kind="infer", n=65536, F=617, K=26, D=10240, x="int8", types="bf16,fp8",
             start=0, end=8192, stride=2, dists=True),
        # training: encode the speech set, class sums, two retraining epochs
        dict(name="speech_fit", kind="fit", n=6238, F=617, K=26, D=10240, x="int8", epochs=2),
        # training: encode and bundle the image set
        dict(name="image_bundle", kind="bundle", n=60000, F=784, K=10, D=8192, x="uint8"),
        # search of stored hypervectors by Hamming distance (unfused path)
        dict(name="hamming_search", kind="hamming", n=1048576, K=26, D=10240, start=0, end=10240, stride=1),
        # cosine ranking against the integer sums of many classes
        dict(name="cosine_search", kind="cosine", n=100003, K=100, D=16384, start=0, end=16384, stride=1),
        # ADC-quantised similarity of the in-memory accelerator
        dict(name="adc_search", kind="adc", n=262144, K=26, D=10240, start=0, end=10240, stride=1, adc="coarse"),
        # Level-ID encoding of continuous features
        dict(name="level_id_encode", kind="level", n=32768, F=617, D=10240, L=128),
        # the tuner's inner loop: many configurations on the same queries
        dict(name="speech_sweep", kind="sweep", n=2000, F=617, K=26, D=10240, x="int8", slots=256, slot_seed=3),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["small", "infer", "wide", "types", "fit", "bundle", "hamming", "cosine", "adc", "level",
                       "sweep"])
    if kind in ("small", "infer", "wide", "types"):
        if kind == "small":          # single calls on small batches, any feature type
            x = rng.choice(["float32", "int8", "uint8"])
            n = _log_int(rng, 1, 4096)
            F = rng.randint(24, 256) if x == "float32" else rng.randint(33, 1024)
            types = rng.choice(["fp32", "bf16", "fp8"] if x == "float32" else ["int8", "int8", "bf16", "fp8"])
        elif kind == "infer":        # int8 bulk inference
            x, n, F, types = "int8", _log_int(rng, 4096, 200000), rng.randint(257, 640), \
                rng.choice(["int8", "int8shift"])
        elif kind == "wide":         # wide uint8 or int8 features
            x, n, F, types = rng.choice(["uint8", "int8"]), _log_int(rng, 2000, 60000), rng.randint(600, 1024), "int8"
        else:                        # reduced element types
            x, n, F, types = rng.choice(["int8", "uint8"]), _log_int(rng, 4096, 65536), rng.randint(100, 784), \
                rng.choice(["bf16", "fp8", "bf16,fp8", "fp8split"])
        D = 64 * rng.randint(16, 160) - rng.choice([0, 0, 24, 63])
        stride = rng.choice([1, 1, 2, 3])
        start = rng.choice([0, 0, 1, 70])
        end = D if rng.random() < 0.5 else rng.randint(max(D // 2, start + 256), D)
        # the shifted projection has kernels for up to two class tiles
        K = _log_int(rng, 2, 60 if types == "int8shift" else 100)
        return dict(kind=rng.choice(["classify", "infer"]), n=n, F=F, K=K, D=D, x=x, types=types, start=start,
                    end=end, stride=stride, dists=rng.random() < 0.3)
    if kind == "fit":
        F, K, D = rng.choice(MODELS)
        return dict(kind="fit", n=_log_int(rng, 500, 30000), F=F, K=K, D=D, x="int8", epochs=rng.randint(0, 3))
    if kind == "bundle":
        return dict(kind="bundle", n=_log_int(rng, 3000, 60000), F=rng.randint(100, 900), K=rng.randint(2, 60),
                    D=64 * rng.randint(16, 128) - rng.choice([0, 0, 17]), x=rng.choice(["uint8", "int8"]))
    if kind in ("hamming", "cosine", "adc"):
        D = 64 * rng.randint(16, 200)
        K = _log_int(rng, 2, 100)
        start = rng.choice([0, 0, 0, 65])
        c = dict(kind=kind, n=_log_int(rng, 1000, 200000), K=K, D=D, start=start,
                 end=rng.randint(max(D // 2, start + 300), D), stride=rng.choice([1, 1, 2, 3]))
        if kind == "adc":
            c["adc"] = rng.choice(["reference", "coarse", "fine"])
        return c
    if kind == "level":
        return dict(kind="level", n=_log_int(rng, 500, 32768), F=rng.randint(60, 640), D=rng.randint(1000, 10240),
                    L=rng.choice([2, 16, 100, 128, 256]))
    F, K, D = rng.choice(MODELS[2:])
    return dict(kind="sweep", n=rng.randint(500, 2500), F=F, K=K, D=D, x=rng.choice(["int8", "uint8"]),
                slots=_log_int(rng, 12, 256), slot_seed=rng.randint(0, 10 ** 6))


# ------------------------------------------------------------------ inputs
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _rand_words(shape, g):
    return torch.randint(-2 ** 63, 2 ** 63 - 1, shape, dtype=torch.int64, device=DEV, generator=g)


def _pack(bits):
    """Bool [n][D] -> int64 words, least significant bit first."""
    n, D = bits.shape
    W = (D + 63) // 64
    full = torch.zeros((n, W * 64), dtype=torch.int64, device=bits.device)
    full[:, :D] = bits
    sh = torch.arange(64, device=bits.device, dtype=torch.int64)
    return (full.view(n, W, 64) << sh).sum(2)


def _unpack(words, D):
    sh = torch.arange(64, device=words.device, dtype=torch.int64)
    return ((words[:, :, None] >> sh) & 1).view(words.shape[0], -1)[:, :D].bool()


def _features(case, g, classes):
    """Class-clustered features: Gaussian clusters quantised to int8 (or as
    fp32), or sparse uint8 pixels whose density follows a class mask."""
    n, F, K = case["n"], case["F"], classes
    y = torch.randint(0, K, (n,), generator=g, device=DEV)
    if case.get("x") == "uint8":
        mask = torch.rand((K, F), generator=g, device=DEV) < 0.3
        dens = torch.where(mask, 0.33, 0.15)
        X = torch.empty((n, F), dtype=torch.uint8, device=DEV)
        for i in range(0, n, 65536):
            d = dens[y[i:i + 65536]]
            on = torch.rand(d.shape, generator=g, device=DEV) < d
            X[i:i + 65536] = torch.randint(1, 256, d.shape, generator=g, device=DEV).mul_(on).to(torch.uint8)
        proto = (mask * 100 + 20).double()
        return X, y, proto
    f32 = case.get("x", "float32") == "float32"
    mu = torch.randn((K, F), generator=g, device=DEV)
    X = torch.empty((n, F), dtype=torch.float32 if f32 else torch.int8, device=DEV)
    for i in range(0, n, 65536):
        m = mu[y[i:i + 65536]]
        z = torch.randn(m.shape, generator=g, device=DEV)
        X[i:i + 65536] = m + 0.5 * z if f32 else ((m + 3.0 * z) * 8.6).round_().clamp_(-127, 127).to(torch.int8)
    return X, y, mu.double()


def _projection(case, g):
    P = torch.randint(0, 2, (case["D"], case["F"]), generator=g, device=DEV, dtype=torch.int8)
    return P.mul_(2).sub_(1)


def _model_inputs(case, seed):
    """Features, labels, projection and class bits (the sign of every class
    prototype's projection)."""
    g = _gen(seed)
    X, y, proto = _features(case, g, case["K"])
    P = _projection(case, g)
    return X, y, P, (proto @ P.double().T) < 0


def _search_inputs(case, seed):
    """Class hypervectors and queries: a class row with 3/8 of its bits
    flipped at random, pad bits zero."""
    g = _gen(seed)
    n, K, D = case["n"], case["K"], case["D"]
    W = (D + 63) // 64
    C = _rand_words((K, W), g)
    if D % 64:
        C[:, -1] &= (1 << (D % 64)) - 1
    y = torch.randint(0, K, (n,), generator=g, device=DEV)
    Q = torch.empty((n, W), dtype=torch.int64, device=DEV)
    for i in range(0, n, 131072):
        m = min(131072, n - i)
        flip = _rand_words((m, W), g) & (_rand_words((m, W), g) | _rand_words((m, W), g))
        Q[i:i + m] = C[y[i:i + m]] ^ flip
    if D % 64:
        Q[:, -1] &= (1 << (D % 64)) - 1
    return Q, C, y


def _class_sums(case, C, seed):
    """Integer class accumulators whose signs follow the class bits: sums of
    240 noisy bipolar rows (even, |a| <= 240)."""
    g = _gen(seed + 17)
    bip = 1.0 - 2.0 * _unpack(C, case["D"]).float()
    a = 60.0 * bip + torch.randn(bip.shape, generator=g, device=DEV) * math.sqrt(240.0)
    return (2 * (a / 2).round()).clamp_(-240, 240).to(torch.int32)


def _level_inputs(case, seed):
    g = _gen(seed)
    X, _, _ = _features(dict(n=case["n"], F=case["F"], x="float32"), g, 26)
    X = X * 3.0
    F, D, L = case["F"], case["D"], case["L"]
    lo, hi = X.min(0).values, X.max(0).values
    ident = torch.rand((F, D), generator=g, device=DEV) < 0.5
    base = torch.rand(D, generator=g, device=DEV) < 0.5
    rank = torch.randperm(D, generator=g, device=DEV)
    flips = torch.arange(L, device=DEV) * (D // 2) // max(L - 1, 1)
    level = base[None, :] ^ (rank[None, :] < flips[:, None])
    return X, lo, hi, ident, level


def _slots(case):
    """Configurations drawn with replacement from the truncation x stride x
    type grid."""
    r = random.Random(case["slot_seed"])
    D = case["D"]
    ends = [D, D * 4 // 5, D * 2 // 5, D // 5, D // 10]
    return [(r.choice(ends), r.choice(SWEEP_STRIDES), 0, r.choice(SWEEP_TYPES)) for _ in range(case["slots"])]


def _adc(case):
    return {"reference": ADC_REFERENCE, "coarse": ADC_COARSE, "fine": ADC_FINE}[case["adc"]]


# ----------------------------------------------------------------- prepare
def prepare(case, seed):
    kind = case["kind"]
    st = dict(case=case)
    if kind in ("classify", "infer", "fit", "bundle", "sweep"):
        X, y, P, cbits = _model_inputs(case, seed)
        st["X"], st["P"] = hdc.pad_cols(X), hdc.pad_cols(P)
        st["y"] = y.to(torch.int32)
        st["C"] = _pack(cbits)
        if kind == "infer":
            st["plans"] = []
            for t in case["types"].split(","):
                plan = hdc.Prepared(st["C"], case["D"], t, case["start"], case["end"], case["stride"])
                shifted = t in hdc.SHIFTED.values()
                st["plans"].append((plan, hdc.shift_projection(st["P"], case["F"], compute=t) if shifted else st["P"]))
        elif kind == "sweep":
            st["cfgs"] = hdc.config_array(_slots(case), TILE_SHARED)
            need = int(hdc.lib().hdc_eval_configs_workspace_bytes(case["slots"], case["F"], case["D"], case["K"]))
            st["ws"] = torch.empty(need, dtype=torch.uint8, device=DEV)
    elif kind == "level":
        X, lo, hi, ident, level = _level_inputs(case, seed)
        st.update(X=X, lo=lo, hi=hi, ID=_pack(ident), LV=_pack(level))
    else:
        Q, C, _ = _search_inputs(case, seed)
        if Q.shape[1] % 2:                      # stored hypervectors have an even row pitch
            Q = torch.nn.functional.pad(Q, (0, 1))
        st["Q"] = Q
        args = (case["start"], case["end"], case["stride"])
        if kind == "hamming":
            st["plan"] = hdc.HammingPrepared(C, *args)
        elif kind == "cosine":
            st["plan"] = hdc.CosinePrepared(_class_sums(case, C, seed), *args)
        else:
            st["plan"] = hdc.AdcPrepared(C, *args)
    return st


# --------------------------------------------------------------------- run
def run(st):
    case = st["case"]
    kind, F, D = case["kind"], case.get("F"), case["D"]
    if kind == "classify":
        out = []
        for t in case["types"].split(","):
            P = st["P"]
            if t in hdc.SHIFTED.values():
                P = hdc.shift_projection(P, F, compute=t)
            out.append(hdc.classify(st["X"], F, P, D, st["C"], t, case["start"], case["end"], case["stride"],
                                    with_dists=case["dists"]))
        return out
    if kind == "infer":
        return [plan(st["X"], F, P, with_dists=case["dists"]) for plan, P in st["plans"]]
    if kind == "fit":
        H = hdc.encode(st["X"], F, st["P"], D)
        C, acc, wrong = train.fit(H, D, st["y"], case["K"], case["epochs"])
        return H, C, acc, wrong
    if kind == "bundle":
        H = hdc.encode(st["X"], F, st["P"], D)
        return (H,) + hdc.bundle(H, D, st["y"], case["K"])
    if kind == "hamming":
        return st["plan"](st["Q"], with_min=True)[:2]
    if kind == "cosine":
        return st["plan"](st["Q"], with_max=True)[:2]
    if kind == "adc":
        return st["plan"](st["Q"], _adc(case), with_max=True)[:2]
    if kind == "level":
        lev = hdc.level_quantize(st["X"], st["lo"], st["hi"], case["L"])
        return lev, hdc.level_id_encode(lev, st["ID"], st["LV"], D)
    # the counts; the records' device_us is a time, not a result
    res = hdc.eval_configs(st["X"], F, st["y"], st["P"], D, st["C"], st["cfgs"], ws=st["ws"])
    return res["correct"], res["n"]


# -------------------------------------------------------------------- work
def _count(case):
    return (case["end"] - case["start"] + case["stride"] - 1) // case["stride"]


def work(case):
    kind, n, D = case["kind"], case["n"], case["D"]
    esz = 4 if case.get("x", "float32") == "float32" else 1
    W8 = (D + 63) // 64 * 8
    if kind in ("classify", "infer"):
        F, K, nd, rungs = case["F"], case["K"], _count(case), len(case["types"].split(","))
        per = n * F * esz + nd * F + K * W8 + 4 * n + (4 * n * K if case["dists"] else 0)
        return {"bytes": rungs * per, "flops": rungs * 2 * n * nd * (F + K)}
    if kind == "fit":
        F, K = case["F"], case["K"]
        return {"bytes": n * F + D * F + n * W8 + 4 * n + 4 * K * D + K * W8,
                "flops": 2 * n * D * F + n * D + case["epochs"] * 2 * n * K * D}
    if kind == "bundle":
        F, K = case["F"], case["K"]
        return {"bytes": n * F + D * F + n * W8 + 4 * n + K * W8 + 4 * K, "flops": 2 * n * D * F + n * D}
    if kind in ("hamming", "cosine", "adc"):
        K, nd = case["K"], _count(case)
        words = (case["end"] + 63) // 64 - case["start"] // 64
        out = {"hamming": 8, "cosine": 12, "adc": 8}[kind]
        cls = K * nd * 4 if kind == "cosine" else K * words * 8
        return {"bytes": n * words * 8 + cls + out * n, "flops": 2 * n * K * nd}
    if kind == "level":
        F, L = case["F"], case["L"]
        return {"bytes": n * F * 4 + n * F * 2 + (F + L) * W8 + n * W8, "flops": 2 * n * F * D}
    # the sweep: the integer and the E4M3 encoding of every query at the
    # longest set, and one comparison per class and dimension of each
    F, K = case["F"], case["K"]
    return {"bytes": n * F + D * F + K * W8 + 4 * n + 8 * case["slots"], "flops": 2 * 2 * n * D * (F + K)}


# ------------------------------------------------------------------- exact
def _rounded(X, t):
    """Features as the compute type holds them, in float64."""
    if t == "bf16":
        return X.float().to(torch.bfloat16).double()
    if t in ("fp8", "fp8shift"):
        return X.float().clamp(-448, 448).to(torch.float8_e4m3fn).double()
    return X.double()


def _sign_bits(X, P, t):
    Xr, Pd = _rounded(X, t), P.double().T.contiguous()
    return torch.cat([(Xr[i:i + 16384] @ Pd) < 0 for i in range(0, Xr.shape[0], 16384)])


def _distances(bits, cls):
    """Bit differences [n][K] (float64, exact)."""
    c = 1.0 - 2.0 * cls.double().T.contiguous()
    nd = bits.shape[1]
    out = [(nd - (1.0 - 2.0 * bits[i:i + 16384].double()) @ c) / 2 for i in range(0, bits.shape[0], 16384)]
    return torch.cat(out)


def _first_min(d):
    """Lowest index of each row's minimum."""
    k = torch.arange(d.shape[1], device=d.device, dtype=d.dtype)
    return ((d * 128 + k).min(1).values % 128).to(torch.int32)


def _first_max(s):
    m = s.max(1, keepdim=True).values
    k = torch.arange(s.shape[1], device=s.device)
    return torch.where(s == m, k, s.shape[1]).min(1).values.to(torch.int32), m[:, 0]


def _sums(bits, y, K):
    one = torch.nn.functional.one_hot(y, K).double().T.contiguous()
    return one @ (1.0 - 2.0 * bits.double())


def exact(case, seed):
    kind, D = case["kind"], case["D"]
    if kind in ("classify", "infer"):
        X, _, P, cls = _model_inputs(case, seed)
        S = slice(case["start"], case["end"], case["stride"])
        out = []
        for t in case["types"].split(","):
            bits = _sign_bits(X, P[S], t)
            d = _distances(bits, cls[:, S])
            out.append((_first_min(d), d.to(torch.int32)) if case["dists"] else _first_min(d))
        return out
    if kind in ("fit", "bundle"):
        X, y, P, _ = _model_inputs(case, seed)
        K = case["K"]
        bits = _sign_bits(X, P, "int8")
        if kind == "bundle":
            return _pack(bits), _pack(_sums(bits, y, K) < 0), torch.bincount(y, minlength=K).to(torch.int32)
        acc, wrong = _sums(bits, y, K), []
        for _ in range(case["epochs"]):
            pred = _first_min(_distances(bits, acc < 0)).long()
            w = pred != y
            acc = acc + _sums(bits[w], y[w], K) - _sums(bits[w], pred[w], K)
            wrong.append(w.sum(dtype=torch.int32).view(1))
        return _pack(bits), _pack(acc < 0), acc.to(torch.int32), wrong
    if kind in ("hamming", "cosine", "adc"):
        Q, C, _ = _search_inputs(case, seed)
        lab, best = [], []
        start, end, stride = case["start"], case["end"], case["stride"]
        S = slice(start, end, stride)
        cls = _unpack(C, D)
        acc = _class_sums(case, C, seed)[:, S].double() if kind == "cosine" else None
        for i in range(0, Q.shape[0], 16384):
            bits = _unpack(Q[i:i + 16384], D)
            if kind == "hamming":
                d = _distances(bits[:, S], cls[:, S])
                lab.append(_first_min(d))
                best.append(d.min(1).values.to(torch.int32))
            elif kind == "cosine":
                s = ((1.0 - 2.0 * bits[:, S].double()) @ acc.T.contiguous()) * (1.0 / (acc * acc).sum(1).sqrt())
                k, m = _first_max(s)
                lab.append(k)
                best.append(m)
            else:
                res, step, floor, ceil = _adc(case)
                keep = torch.zeros(D, dtype=torch.float64, device=DEV)
                keep[S] = 1.0
                s = torch.zeros((bits.shape[0], case["K"]), dtype=torch.float64, device=DEV)
                for c in range(0, D, 128):
                    if not bool(keep[c:c + 128].any()):
                        continue
                    q = (1.0 - 2.0 * bits[:, c:c + 128].double()) * keep[c:c + 128]
                    v = q @ (1.0 - 2.0 * cls[:, c:c + 128].double()).T.contiguous()
                    code = ((v.clamp(floor, ceil) - floor) / step + 0.5).floor().clamp(max=2 ** res - 1)
                    s += floor + step * code
                k, m = _first_max(s)
                lab.append(k)
                best.append(m.to(torch.int32))
        return torch.cat(lab), torch.cat(best)
    if kind == "level":
        X, lo, hi, ident, level = _level_inputs(case, seed)
        L, F = case["L"], case["F"]
        # the quantiser is defined in binary32, one rounding per operation
        w = hi - lo
        v = ((X - lo) * float(L)) / w
        lev = torch.where((w > 0) & (v > 0), v.floor().clamp(max=L - 1), torch.zeros_like(v)).long()
        H = []
        for i in range(0, X.shape[0], 8192):
            cnt = torch.zeros((lev[i:i + 8192].shape[0], D), dtype=torch.int16, device=DEV)
            for f in range(F):
                cnt += (level ^ ident[f])[lev[i:i + 8192, f]]
            H.append(_pack(2 * cnt > F))
        return lev.to(torch.int16), torch.cat(H)
    X, y, P, cls = _model_inputs(case, seed)
    enc = {t: _sign_bits(X, P, t) for t in SWEEP_TYPES}
    seen, correct = {}, []
    for end, stride, start, t in _slots(case):
        key = (end, stride, t)
        if key not in seen:
            S = slice(start, end, stride)
            seen[key] = int((_first_min(_distances(enc[t][:, S], cls[:, S])) == y).sum())
        correct.append(seen[key])
    return np.array(correct, dtype=np.int32), np.full(len(correct), case["n"], dtype=np.int32)

"""Performance cases of the Double Sparsity decode-attention library.

Each case is a piece of work that a program serving a model has the library do
through its public entry points: one decode step of one attention layer, one
decode step over several layers replayed as a HIP graph, dense decode, building
the label cache after a prefill, and a decode step with K/V in host memory.

A case is a dict of plain values:
  kind     "decode"  ds_sparse_decode (or its 4-bit / interleaved variant),
                     with `append` preceded by ds_append_kv of the new token
           "dense"   ds_dense_decode
           "prefill" ds_build_label (label 4: ds_build_label_q4)
           "offload" OffloadDecoder.decode: predict, select, fetch over the
                     host link, attend
  B, Hq, Hkv, L, L_max, r, k   sizes (head dimension 128, fp16 storage)
  label    bits of the label cache, 16 or 4
  layers   layers of a step; more than one: captured once, replayed as a graph
           ("offload" enqueues its layers itself)
  inter    K|V kept interleaved in one array
  idx      the index list is wanted as well
"""
import math

import numpy as np
import torch

import paper_2408_07092_amd as ds
from paper_2408_07092_amd.offload import OffloadDecoder

D = 128
N_OUTLIER, OUTLIER_SCALE = 8, 8.0      # static outlier channels of every KV head, as in the synthetic workloads


def _case(kind, B, Hq, Hkv, L, r=8, k=None, L_max=None, label=16, layers=1, append=False, inter=False, idx=False):
    return {"kind": kind, "B": B, "Hq": Hq, "Hkv": Hkv, "L": L, "L_max": L_max or L, "r": r,
            "k": k if k is not None else max(1, L // 16), "label": label, "layers": layers,
            "append": append, "inter": inter, "idx": idx}


def listed():
    named = {
        # one short conversation, one layer, called eagerly: latency and launch cost
        "layer_4k": _case("decode", 1, 32, 32, 4096),
        # a whole step of a small model at batch 4, caches allocated ahead of the tokens they hold:
        # every layer appends its new token and decodes, the step is replayed as a graph
        "step_8layers_6k": _case("decode", 4, 32, 32, 6000, L_max=8192, layers=8, append=True),
        # the 7B shape at batch 8 with 16 label channels
        "batch8_16k": _case("decode", 8, 32, 32, 16384, r=16),
        # the 7B shape, long context: the headline workload
        "long_64k": _case("decode", 1, 32, 32, 65536),
        # grouped queries, the 70B shape
        "group8_32k": _case("decode", 16, 64, 8, 32768),
        # grouped queries with the label cache kept in 4 bits
        "group4_32k_4bit": _case("decode", 16, 32, 8, 32768, label=4),
        # odd sizes: seven heads to a group, twelve channels, a length that fills no tile, a padded
        # and interleaved cache, and a caller that wants to see which tokens were chosen
        "group7_20011_12ch": _case("decode", 3, 28, 4, 20011, r=12, L_max=24576, inter=True, idx=True),
        # 256K tokens with the caches kept in device memory
        "long_256k": _case("decode", 1, 32, 32, 262144),
        # layers that a model keeps dense, grouped queries
        "dense_group4_32k": _case("dense", 4, 32, 8, 32768),
        # label cache of one layer built after a long prefill, fp16 and 4-bit
        "prefill_64k": _case("prefill", 1, 32, 32, 65536),
        "prefill_b8_16k_4bit": _case("prefill", 8, 32, 8, 16384, r=16, label=4),
        # K/V in pinned host memory: four layers of the 7B shape, query prediction on
        "offload_4layers_16k": _case("offload", 1, 32, 32, 16384, layers=4),
    }
    return [dict(c, name=n) for n, c in named.items()]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(("decode", "dense", "prefill", "offload"), (9, 2, 3, 1))[0]
    while True:
        Hq, Hkv = rng.choice(((32, 32), (32, 32), (8, 8), (40, 40), (32, 16), (32, 8), (64, 8), (28, 4)))
        B = _log(rng, 1, 32)
        L = _log(rng, 256, 262144)
        if rng.random() < 0.4:
            L = max(256, L // 1024 * 1024)
        L_max = L if rng.random() < 0.5 else (L + 2047) // 2048 * 2048
        r = rng.choice((8, 8, 8, 16, 16, 4, 12, 24))
        k = max(1, L // rng.choice((8, 16, 16, 16, 32)))
        label = 4 if rng.random() < 0.25 else 16
        inter, idx, append = (rng.random() < p for p in (0.2, 0.2, 0.4))
        layers = rng.choice((1, 1, 1, 2, 4))
        if kind == "dense":
            r, k, label, layers, inter, idx, append = 8, max(1, L // 16), 16, 1, False, False, False
        elif kind == "prefill":
            k, layers, idx, append, inter = max(1, L // 16), 1, False, False, inter and label == 16
        elif kind == "offload":
            Hq, Hkv, B, label, layers, inter, idx, append = 32, Hkv, min(B, 2), 16, rng.choice((2, 3, 4)), False, False, False
            L, k = min(L, 16384), max(1, min(L, 16384) // 16)
            L_max = L
        elif label == 4:
            inter = append = False
        c = _case(kind, B, Hq, Hkv, L, r, k, L_max, label, layers, append, inter, idx)
        cache = layers * B * Hkv * L_max * D * 4
        if kind == "offload":
            if cache <= (1 << 30):
                return c
        elif cache <= (1 << 32) and work(c)["bytes"] <= (400 << 20):
            return c


# ------------------------------------------------------------------ inputs
def _rows(g, shape, scale, out):
    """Fills out [B, Hkv, L, d] (a view is fine) with N(0, 1) * scale[h, d], one head at a time."""
    for b in range(shape[0]):
        for h in range(shape[1]):
            x = torch.randn((shape[2], D), generator=g, device="cuda", dtype=torch.float32)
            if scale is not None:
                x.mul_(scale[h])
            out[b, h, :shape[2]].copy_(x)


class _Layer:
    pass


def _layer(c, seed, shp):
    B, Hq, Hkv, L, L_max, r = (c[n] for n in ("B", "Hq", "Hkv", "L", "L_max", "r"))
    G = Hq // Hkv
    host = np.random.default_rng([seed & 0x7FFFFFFF, 11])
    scale_h = np.ones((Hkv, D), np.float32)
    for h in range(Hkv):
        scale_h[h, host.choice(D, N_OUTLIER, replace=False)] = OUTLIER_SCALE
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    scale = torch.from_numpy(scale_h).cuda()
    y = _Layer()
    # offline calibration, as a program does once per model
    qc = host.standard_normal((64, Hq, D), dtype=np.float32) * np.repeat(scale_h, G, axis=0)
    kc = host.standard_normal((64, Hkv, D), dtype=np.float32) * scale_h
    ch = ds.ds_calibrate_channels(qc.astype(np.float16), kc.astype(np.float16), r,
                                  ds.DS_CALIB_QK if G == 1 else ds.DS_CALIB_Q)
    y.channels = torch.from_numpy(ch).cuda()
    y.q = (torch.randn((B, Hq, D), generator=g, device="cuda") * scale.repeat_interleave(G, 0)).half()
    if c["inter"]:
        y.K = torch.zeros((B, Hkv, L_max, 2, D), dtype=torch.float16, device="cuda")
        y.V = None
        k_rows, v_rows = y.K[:, :, :, 0], y.K[:, :, :, 1]
    else:
        y.K = torch.zeros((B, Hkv, L_max, D), dtype=torch.float16, device="cuda")
        k_rows = y.K
        y.V = v_rows = None
        if c["kind"] != "prefill":
            y.V = v_rows = torch.zeros((B, Hkv, L_max, D), dtype=torch.float16, device="cuda")
    _rows(g, (B, Hkv, L), scale, k_rows)
    if v_rows is not None:
        _rows(g, (B, Hkv, L), None, v_rows)
    y.amax = None
    if c["label"] == 4:
        y.label = torch.zeros((B, Hkv, L_max, (r + 7) // 8), dtype=torch.int32, device="cuda")
        y.amax = torch.zeros((B, Hkv, r), dtype=torch.float32, device="cuda")
    else:
        y.label = torch.zeros((B, Hkv, L_max, r), dtype=torch.float16, device="cuda")
    if c["kind"] in ("decode", "offload"):
        _build(c, y, shp)
    if c["append"]:
        y.k_new = (torch.randn((B, Hkv, 1, D), generator=g, device="cuda") * scale[:, None]).half()
        y.v_new = torch.randn((B, Hkv, 1, D), generator=g, device="cuda").half()
    if c["kind"] == "offload":
        pinned = []
        for t in (y.K, y.V):
            p = torch.empty(t.shape, dtype=torch.float16, pin_memory=True)
            p.copy_(t)
            pinned.append(p)
        y.K, y.V = pinned
        y.x = torch.randn((B, Hq * D), generator=g, device="cuda").half()
        y.Wq = (torch.randn((Hq * D, Hq * D), generator=g, device="cuda") / math.sqrt(Hq * D)).half()
        y.q_pred = torch.empty_like(y.q)
    return y


def _build(c, y, shp):
    if c["label"] == 4:
        ds.ds_build_label_q4(y.K, y.channels, y.label, y.amax, shp)
    elif c["inter"]:
        ds.ds_build_label_kv(y.K, y.channels, y.label, shp)
    else:
        ds.ds_build_label(y.K, y.channels, y.label, shp)


class _State:
    pass


def prepare(case, seed):
    c = case
    s = _State()
    s.case = c
    s.shp = ds.shape(c["B"], c["Hq"], c["Hkv"], D, c["L"], c["L_max"], c["r"], c["k"])
    s.layers = [_layer(c, seed * 64 + i, s.shp) for i in range(c["layers"])]
    if c["kind"] == "prefill":
        return s
    s.out = torch.zeros((c["layers"], c["B"], c["Hq"], D), dtype=torch.float32, device="cuda")
    s.idx = (torch.zeros((c["layers"], c["B"], c["Hkv"], c["k"]), dtype=torch.int32, device="cuda")
             if c["idx"] else None)
    s.graph = None
    if c["kind"] == "offload":
        s.decoder = OffloadDecoder(s.shp)
        torch.cuda.synchronize()
        return s
    s.ws = ds.ds_workspace_alloc(s.shp)
    torch.cuda.synchronize()
    if c["layers"] > 1:
        side = torch.cuda.Stream()
        with torch.cuda.stream(side):
            _step(s)                        # once outside the capture, as usual
            side.synchronize()
            s.graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(s.graph, stream=side):
                _step(s)
    torch.cuda.synchronize()
    return s


def _step(s):
    c = s.case
    for i, y in enumerate(s.layers):
        out, idx = s.out[i], None if s.idx is None else s.idx[i]
        if c["append"]:
            ds.ds_append_kv(y.k_new, y.v_new, y.K, y.V, y.channels, y.label, s.shp, c["L"] - 1, 1,
                            ds.DS_KV_INTERLEAVED if c["inter"] else ds.DS_KV_SPLIT)
        if c["kind"] == "dense":
            ds.ds_dense_decode(y.q, y.K, y.V, out, s.ws, s.shp)
        elif c["label"] == 4:
            ds.ds_sparse_decode_q4(y.q, y.label, y.amax, y.K, y.V, y.channels, out, idx, s.ws, s.shp)
        elif c["inter"]:
            ds.ds_sparse_decode_kv(y.q, y.label, y.K, y.channels, out, idx, s.ws, s.shp)
        else:
            ds.ds_sparse_decode(y.q, y.label, y.K, y.V, y.channels, out, idx, s.ws, s.shp)


def run(state):
    s, c = state, state.case
    if c["kind"] == "prefill":
        y = s.layers[0]
        _build(c, y, s.shp)
        return {"label": y.label, "amax": y.amax}
    if c["kind"] == "offload":
        s.decoder.decode([(y.q, y.label, y.channels, y.K, y.V) for y in s.layers], list(s.out),
                         [(y.x, y.Wq, y.q_pred) for y in s.layers])
        return {"out": s.out, "q_pred": [y.q_pred for y in s.layers]}
    if s.graph is not None:
        s.graph.replay()
    else:
        _step(s)
    res = {"out": s.out, "idx": s.idx}
    if c["append"]:
        res["caches"] = [(y.K, y.V, y.label) for y in s.layers]
    return res


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    c = case
    units = c["B"] * c["Hkv"]
    token = (c["r"] + 7) // 8 * 4 if c["label"] == 4 else c["r"] * 2      # label bytes of a token
    label = units * c["L"] * token
    io = c["B"] * c["Hq"] * D * (2 + 4)
    if c["kind"] == "prefill":
        return {"bytes": units * c["L"] * D * 2 + label, "flops": 0}
    if c["kind"] == "dense":
        return {"bytes": units * c["L"] * D * 4 + io, "flops": 4 * c["B"] * c["Hq"] * c["L"] * D}
    k = min(c["k"], c["L"])
    nbytes = label + units * k * D * 4 + io
    flops = 2 * units * c["L"] * c["r"] + 4 * c["B"] * c["Hq"] * k * D
    if c["idx"]:
        nbytes += units * k * 4
    if c["append"]:
        nbytes += units * (4 * D * 2 + token)
    if c["kind"] == "offload":
        n = c["Hq"] * D
        nbytes += n * n * 2
        flops += 2 * c["B"] * n * n
    return {"bytes": nbytes * c["layers"], "flops": flops * c["layers"]}


def tolerance(case):
    # Label caches are copies or integer codes.  Outputs of the decode are fp32 sums over exact
    # products: over these ranges they are up to 1.8e-6 from the same sums in 64 bits.  The chosen
    # tokens are decided on scores summed in a fixed order and do not differ.
    if case["kind"] == "prefill":
        return "exact"
    return {"rel": 1e-5}

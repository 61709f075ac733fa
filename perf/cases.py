"""Performance cases: the calls a user of this framework makes, through its public entry points.

Three kinds of call, each named by "op" in a case:

  layer      moe_w4a16_layer / moe_w4a16_routed_layer / moe_w4a16_layer_prepacked ("entry"): the
             int4-weight mixture-of-experts layer, from router output (or logits) to the combined rows
  fp8_layer  fp8_moe_layer: the same layer with e4m3 weights and activations quantised on the fly
  fp8_gemm   fp8_blockwise_gemm: a dense FP8 linear layer

A state holds what a serving program holds before the call: resident weights, the batch's
activations and routing, the output buffer and the workspace.  Inputs are drawn on the GPU from the
seed alone, with the distributions of the benchmark workloads (moe_workloads): activations
0.5 N(0, 1), standard normal logits (plus a power-law bias per expert in the skewed workload),
uniform nibbles and zero points, scales in [0.002, 0.02]; e4m3 codes of Gaussian weights.
"""
import math

import numpy as np
import torch

import paper_2504_16214_amd as M

DTYPES = {"f16": torch.float16, "bf16": torch.bfloat16}


def listed():
    return [
        # The launch-bound end: a toy layer behind its router, one call per token batch.
        dict(name="tiny_routed", op="layer", entry="routed", T=16, K=256, N=512, E=8, topk=2, group=128, dtype="f16", skew=False),
        # One user decoding on the 256-expert layer: eight experts' weights and the latency of the launches.
        dict(name="decode_one_token", op="layer", entry="plain", T=1, K=7168, N=2048, E=256, topk=8, group=128, dtype="f16", skew=False),
        # Few large experts at a serving batch (the 8-expert layer shape): 16 rows per expert.
        dict(name="mixtral_decode", op="layer", entry="plain", T=64, K=4096, N=14336, E=8, topk=2, group=128, dtype="f16", skew=False),
        # A small batch on weights that were repacked offline, the layout a serving program would keep.
        dict(name="decode_prepacked", op="layer", entry="prepacked", T=37, K=7168, N=2048, E=256, topk=8, group=128, dtype="f16", skew=False),
        # The benchmark's decode batch: nearly all 256 experts active, four rows each.
        dict(name="deepseek_decode", op="layer", entry="plain", T=128, K=7168, N=2048, E=256, topk=8, group=128, dtype="f16", skew=False),
        # A ragged mixed batch (chunked prefill beside decode) behind its router, bfloat16.
        dict(name="mixed_batch_bf16", op="layer", entry="routed", T=717, K=7168, N=2048, E=256, topk=8, group=128, dtype="bf16", skew=False),
        # Power-law routing, group 64, an intermediate size that is no power of two: 1 to 900 rows per expert.
        dict(name="skewed_bf16", op="layer", entry="plain", T=1024, K=2048, N=1408, E=64, topk=6, group=64, dtype="bf16", skew=True),
        # A whole prefill chunk.
        dict(name="deepseek_prefill", op="layer", entry="plain", T=4096, K=7168, N=2048, E=256, topk=8, group=128, dtype="f16", skew=False),
        # The FP8 layer at the decode batch and at a prefill chunk.
        dict(name="fp8_moe_decode", op="fp8_layer", T=128, K=7168, N=2048, E=256, topk=8, dtype="bf16"),
        dict(name="fp8_moe_prefill", op="fp8_layer", T=4096, K=7168, N=2048, E=256, topk=8, dtype="bf16"),
        # Dense FP8 linear layers of a 32-billion-parameter transformer: fused QKV at decode, fused gate/up at prefill.
        dict(name="fp8_qkv_decode", op="fp8_gemm", M=64, N=10240, K=5120, dtype="bf16"),
        dict(name="fp8_gateup_prefill", op="fp8_gemm", M=4096, N=51200, K=5120, dtype="bf16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["layer", "layer", "layer", "layer", "fp8_layer", "fp8_layer", "fp8_gemm", "fp8_gemm"])
    dtype = rng.choice(["f16", "bf16"])
    if kind == "fp8_gemm":
        n, k = rng.choice([(10240, 5120), (5120, 8192), (51200, 5120), (5120, 25600),
                           (64 * rng.randint(3, 200), 128 * rng.randint(2, 80))])
        return dict(op=kind, M=_log_int(rng, 1, 4096), N=n, K=k, dtype=dtype)
    if kind == "fp8_layer":
        k, n, e, topk = rng.choice([(7168, 2048, 256, 8), (7168, 2048, 256, 8), (2048, 1408, 64, 6),
                                    (128 * rng.randint(2, 40), 128 * rng.randint(2, 24), rng.randint(4, 96), rng.randint(1, 4))])
        return dict(op=kind, T=_log_int(rng, 1, 4096), K=k, N=n, E=e, topk=topk, dtype=dtype)
    group = 128
    shape = rng.choice(["256 experts", "256 experts", "256 experts", "8 experts", "64 experts", "any"])
    if shape == "256 experts":
        k, n, e, topk, most = 7168, 2048, 256, 8, 4096
    elif shape == "8 experts":
        k, n, e, topk, most = 4096, 14336, 8, 2, 2048
    elif shape == "64 experts":
        k, n, e, topk, most, group = 2048, 1408, 64, 6, 4096, 64
    else:
        group = rng.choice([32, 64, 128])
        k, n = group * rng.randint(2, 4096 // group), group * rng.randint(2, 2048 // group)
        e, topk, most = rng.randint(4, 96), rng.randint(1, 4), 4096
    entry = rng.choice(["plain", "routed", "prepacked"])
    if entry == "prepacked" and (group != 128 or k % 1024 or n % 1024):
        entry = "plain"
    return dict(op=kind, entry=entry, T=_log_int(rng, 1, most), K=k, N=n, E=e, topk=topk, group=group, dtype=dtype,
                skew=rng.random() < 0.25)


# ---- inputs -----------------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _normal(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float32)


def _logits(case, g):
    """Router logits [T, E], and the per-expert bias (None unless the routing is skewed)."""
    logits = _normal(g, case["T"], case["E"])
    if not case.get("skew"):
        return logits, None
    rank = torch.arange(1, case["E"] + 1, dtype=torch.float64, device="cuda")
    return logits, (-2.4 * torch.log(rank)).float()


def _route(logits, bias, topk):
    """Top-k expert ids and the softmax over the chosen logits."""
    z = logits if bias is None else logits + bias
    top, ids = torch.topk(z, topk, dim=1)
    return ids.int().contiguous(), torch.softmax(top.double(), dim=1)


def _int4_weight(g, e, rows, red, group, dtype):
    """Packed words, group scales and zero points of one int4 weight tensor [e, rows, red]."""
    q = torch.randint(-2 ** 31, 2 ** 31, (e, rows, red // 8), generator=g, device="cuda", dtype=torch.int32)
    s = torch.rand(e, rows, red // group, generator=g, device="cuda") * 0.018 + 0.002
    z = torch.randint(0, 16, (e, rows, red // group), generator=g, device="cuda", dtype=torch.uint8)
    return q, s.to(dtype), z


def _e4m3(x):
    return x.clamp(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8)


def _fp8_weight(g, e, rows, red):
    """e4m3 codes of Gaussian weights whose 4.5 sigma maps to 448, and 128 x 128 block scales (sigma about 0.02)."""
    p = (torch.arange(256, device="cuda", dtype=torch.float64) + 0.5) / 256
    table = _e4m3((torch.special.ndtri(p) / 4.5 * 448.0).float())
    w = torch.randint(0, 256, (e, rows, red), generator=g, device="cuda", dtype=torch.uint8)
    for i in range(e):
        w[i] = table[w[i].int()]
    s = torch.rand(e, -(-rows // 128), red // 128, generator=g, device="cuda") + 0.5
    return w, s * (0.02 * 4.5 / 448.0)


def _inputs(case, seed):
    g = _gen(seed)
    if case["op"] == "fp8_gemm":
        m, n, k = case["M"], case["N"], case["K"]
        x = _normal(g, m, k // 128, 128)
        sa = x.abs().amax(dim=2).clamp_min(1e-12) / 448.0
        a = _e4m3((x / sa[:, :, None]).reshape(m, k))
        b, sb = _fp8_weight(g, 1, n, k)
        return dict(A=a, sa=sa, B=b[0], sb=sb[0])
    dtype = DTYPES[case["dtype"]]
    t, k, n, e = case["T"], case["K"], case["N"], case["E"]
    d = dict(X=(0.5 * _normal(g, t, k)).to(dtype))
    d["logits"], d["bias"] = _logits(case, g)
    d["ids"], w = _route(d["logits"], d["bias"], case["topk"])
    d["w"] = w.float()
    if case["op"] == "fp8_layer":
        d["w1"], d["w1s"] = _fp8_weight(g, e, 2 * n, k)
        d["w2"], d["w2s"] = _fp8_weight(g, e, k, n)
    else:
        d["q1"], d["s1"], d["z1"] = _int4_weight(g, e, 2 * n, k, case["group"], dtype)
        d["q2"], d["s2"], d["z2"] = _int4_weight(g, e, k, n, case["group"], dtype)
    return d


def _bytes(n):
    return torch.empty(max(int(n), 256), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    st = _inputs(case, seed)
    st["case"] = case
    dtype = DTYPES[case["dtype"]]
    if case["op"] == "fp8_gemm":
        m, n, k = case["M"], case["N"], case["K"]
        st["out"] = torch.empty(m, n, dtype=dtype, device="cuda")
        need = M.fp8_blockwise_gemm_workspace_bytes(m, n, k)
        st["ws"] = _bytes(need) if need else None
        return st
    t, k, n, e, topk = (case[v] for v in ("T", "K", "N", "E", "topk"))
    st["out"] = torch.empty(t, k, dtype=dtype, device="cuda")
    if case["op"] == "fp8_layer":
        st["ws"] = _bytes(M.fp8_moe_layer_workspace_bytes(t, k, n, e, topk))
        return st
    mdt = M.MOE_F16 if case["dtype"] == "f16" else M.MOE_BF16
    if case["entry"] == "routed":
        st["ws"] = _bytes(M.moe_w4a16_routed_layer_workspace_bytes(t, k, n, e, topk, mdt))
    else:
        st["ws"] = _bytes(M.moe_w4a16_layer_workspace_bytes(t, k, n, e, topk, mdt))
    if case["entry"] == "prepacked":
        for name, paired in (("q1", False), ("q2", True)):
            packed = torch.empty_like(st[name])
            M.moe_repack_qweight(st[name], paired, packed)
            st[name] = packed
    return st


def run(st):
    case = st["case"]
    if case["op"] == "fp8_gemm":
        M.fp8_blockwise_gemm(st["A"], st["sa"], st["B"], st["sb"], st["out"], st["ws"])
    elif case["op"] == "fp8_layer":
        M.fp8_moe_layer(st["X"], st["ids"], st["w"], st["w1"], st["w1s"], st["w2"], st["w2s"], st["out"], st["ws"])
    else:
        weights = (st["q1"], st["s1"], st["z1"], st["q2"], st["s2"], st["z2"])
        if case["entry"] == "routed":
            M.moe_w4a16_routed_layer(st["X"], st["logits"], st["bias"], *weights, st["out"], case["topk"],
                                     case["group"], st["ws"])
        else:
            layer = M.moe_w4a16_layer_prepacked if case["entry"] == "prepacked" else M.moe_w4a16_layer
            layer(st["X"], st["ids"], st["w"], *weights, st["out"], case["group"], st["ws"])
    return st["out"]


# ---- what a pass cannot do without ------------------------------------------------------------

def _active_experts(case):
    """Experts that at least one token is sent to, for one draw of the case's routing."""
    rng = np.random.default_rng(0)
    z = rng.standard_normal((case["T"], case["E"]))
    if case.get("skew"):
        z = z - 2.4 * np.log(np.arange(1, case["E"] + 1))
    return int(np.unique(np.argpartition(-z, case["topk"] - 1, axis=1)[:, :case["topk"]]).size)


def work(case):
    if case["op"] == "fp8_gemm":
        m, n, k = case["M"], case["N"], case["K"]
        return {"bytes": n * k + m * k + 4 * (m * (k // 128) + -(-n // 128) * (k // 128)) + 2 * m * n, "flops": 2 * m * n * k}
    t, k, n, s = case["T"], case["K"], case["N"], case["T"] * case["topk"]
    active = _active_experts(case)
    if case["op"] == "fp8_layer":
        weights = active * (3 * n * k + 4 * 3 * (n // 128) * (k // 128))
    else:
        weights = active * (3 * n * k // 2 + 3 * (3 * n * (k // case["group"])))     # nibbles; 2-byte scale, 1-byte zero point
    routing = 4 * t * case["E"] if case.get("entry") == "routed" else 8 * s
    return {"bytes": weights + routing + 2 * 2 * t * k, "flops": 6 * s * n * k}


# ---- correctness ------------------------------------------------------------------------------

def tolerance(case):
    # About four times the largest 2-norm error against exact() over the ranges (measured: FP8 product 2.1e-4 / 1.66e-3, int4
    # layer 4.4e-4 / 3.5e-3, FP8 layer 1.6e-3 / 2.4e-3 in f16 / bf16).  The product rounds once to 16 bits; the layers round
    # their intermediates too, and in the FP8 layer activation codes move one e4m3 step where an intermediate rounds the
    # other way.
    f16 = case["dtype"] == "f16"
    if case["op"] == "fp8_gemm":
        return {"rel": 8.5e-4 if f16 else 6.8e-3}
    if case["op"] == "fp8_layer":
        return {"rel": 6.5e-3 if f16 else 9.6e-3}
    return {"rel": 1.8e-3 if f16 else 1.4e-2}


def _int4_rows(q, s, z, group):
    """One expert's weight matrix in 64 bits."""
    shifts = torch.arange(0, 32, 4, device=q.device, dtype=torch.int32)
    nib = ((q[:, :, None] >> shifts) & 15).reshape(q.shape[0], -1).double()
    return (nib - z.double().repeat_interleave(group, 1)) * s.double().repeat_interleave(group, 1)


def _fp8_rows(codes, scale):
    """One FP8 weight matrix in 64 bits."""
    w = codes.view(torch.float8_e4m3fn).float().double()
    s = scale.double().repeat_interleave(128, 0)[:w.shape[0]]
    return w * s.repeat_interleave(128, 1)


def _quantised(x):
    """1 x 128 activation tiles through e4m3 and back, codes decided in float32 as the layer defines them."""
    x = x.float().reshape(x.shape[0], -1, 128)
    m = x.abs().amax(dim=2, keepdim=True).clamp_min(1e-4)
    code = _e4m3(x * (torch.full_like(m, 448.0) / m)).view(torch.float8_e4m3fn).float().double()
    return (code * (m / 448.0).double()).reshape(x.shape[0], -1)


def exact(case, seed):
    d = _inputs(case, seed)
    if case["op"] == "fp8_gemm":
        a = d["A"].view(torch.float8_e4m3fn).float().double() * d["sa"].double().repeat_interleave(128, 1)
        return a @ _fp8_rows(d["B"], d["sb"]).t()
    t, k, n, topk = case["T"], case["K"], case["N"], case["topk"]
    dtype = DTYPES[case["dtype"]]
    fp8 = case["op"] == "fp8_layer"
    ids, w = d["ids"].long(), d["w"].double()
    if case.get("entry") == "routed":
        w = _route(d["logits"], d["bias"], topk)[1]
    x = _quantised(d["X"]) if fp8 else d["X"].double()
    y = torch.zeros(t * topk, k, dtype=torch.float64, device="cuda")
    flat = ids.reshape(-1)
    for e in range(case["E"]):
        slots = torch.nonzero(flat == e).flatten()
        if not slots.numel():
            continue
        w1 = _fp8_rows(d["w1"][e], d["w1s"][e]) if fp8 else _int4_rows(d["q1"][e], d["s1"][e], d["z1"][e], case["group"])
        w2 = _fp8_rows(d["w2"][e], d["w2s"][e]) if fp8 else _int4_rows(d["q2"][e], d["s2"][e], d["z2"][e], case["group"])
        h = x[slots // topk] @ w1.t()
        if fp8:      # the two products' operands are 16-bit tensors before they are quantised
            h = h.to(dtype).double()
        gate, up = h[:, :n], h[:, n:]
        act = gate / (1 + torch.exp(-gate)) * up
        if fp8:
            act = _quantised(act.to(dtype))
        y[slots] = act @ w2.t()
    return (y.reshape(t, topk, k) * w[:, :, None]).sum(dim=1)

"""GPU tests of the pass over the activations that shares the launch of the bucketing (up to 2^23 activations, a launch of
its own beyond): the layer's two tiles that read reordered rows, both types, plain and routed, and the FP8 layer, either
side of the line.  The bits must be those of a layer whose activations are prepared by the stand-alone passes: the same
tokens in a call of the other kind (more tokens behind them), or the quantiser's own entry."""
from __future__ import annotations

import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2504_16214_amd as M

DT = {"f16": torch.float16, "bf16": torch.bfloat16}


def weights(E, rows, red, dtype, gen):
    q = torch.randint(-2**31, 2**31, (E, rows, red // 8), device="cuda", dtype=torch.int32, generator=gen)
    s = (torch.rand(E, rows, red // 128, device="cuda", generator=gen) * 0.018 + 0.002).to(DT[dtype])
    z = torch.randint(0, 16, (E, rows, red // 128), device="cuda", dtype=torch.uint8, generator=gen)
    return q, s, z


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("block,T", [(64, 129), (256, 257), (64, 8191), (256, 8192)])
def test_reordered_rows(block, T, dtype):
    """K 1024: T tokens alone (beside the bucketing) against the first T of 8193 (a launch of its own)."""
    K, N, E, more = 1024, 1024, 4, 8193
    gen = torch.Generator("cuda").manual_seed(T)
    X = torch.randn(more, K, device="cuda", generator=gen).to(DT[dtype])
    ids = torch.randint(0, E, (more, 1), device="cuda", dtype=torch.int32, generator=gen)
    w = torch.rand(more, 1, device="cuda", generator=gen)
    w1, w2 = weights(E, 2 * N, K, dtype, gen), weights(E, K, N, dtype, gen)
    outs = []
    M.moe_set_block_m_override(block)
    M.moe_set_reduction_splits(1 if block == 64 else 0)
    try:
        for t in (T, more):
            print(f"[gpu-case] rows beside, block {block} {t} tokens {dtype}", flush=True)
            ws = torch.empty(M.moe_w4a16_layer_workspace_bytes(t, K, N, E, 1, M.MOE_F16 if dtype == "f16" else M.MOE_BF16) + t * (N // 128) * 4 + 256,
                             dtype=torch.uint8, device="cuda")
            out = torch.full((t, K), float("nan"), dtype=DT[dtype], device="cuda")
            M.moe_w4a16_layer(X[:t], ids[:t], w[:t], *w1, *w2, out, 128, ws)
            torch.cuda.synchronize()
            outs.append(out[:T])
    finally:
        M.moe_set_block_m_override(0)
        M.moe_set_reduction_splits(0)
    assert bool(outs[0].isfinite().all()) and torch.equal(outs[0], outs[1])


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("T", [1, 300, 16384, 16385])
def test_quantised_rows(T, dtype):
    """FP8, K 512: the layer against its own steps through the staged entries."""
    K, N, E, topk = 512, 256, 4, 2
    gen = torch.Generator("cuda").manual_seed(T)
    X = torch.randn(T, K, device="cuda", generator=gen).to(DT[dtype])
    ids = torch.stack([torch.randperm(E, device="cuda", generator=gen)[:topk] for _ in range(min(T, 64))]).to(torch.int32).repeat((T + 63) // 64, 1)[:T].contiguous()
    w = torch.rand(T, topk, device="cuda", generator=gen)
    f8 = lambda *s: torch.randn(*s, device="cuda", generator=gen).to(torch.float8_e4m3fn).view(torch.uint8)
    w1, s1 = f8(E, 2 * N, K), torch.rand(E, 2 * N // 128, K // 128, device="cuda", generator=gen) * 0.01
    w2, s2 = f8(E, K, N), torch.rand(E, K // 128, N // 128, device="cuda", generator=gen) * 0.01
    ws = torch.full((M.fp8_moe_layer_workspace_bytes(T, K, N, E, topk),), 255, dtype=torch.uint8, device="cuda")
    out = torch.full((T, K), float("nan"), dtype=DT[dtype], device="cuda")
    print(f"[gpu-case] FP8 rows beside, {T} tokens {dtype}", flush=True)
    M.fp8_moe_layer(X, ids, w, w1, s1, w2, s2, out, ws)
    torch.cuda.synchronize()
    codes = torch.zeros(T, K, dtype=torch.uint8, device="cuda")
    scales = torch.zeros(T, K // 128, dtype=torch.float32, device="cuda")
    M.fp8_quantize_rows(X, codes, scales)
    torch.cuda.synchronize()
    # the codes and scales lie in the workspace as the stand-alone quantiser writes them
    flat = ws.cpu().numpy().tobytes()
    assert codes.cpu().numpy().tobytes() in flat and scales.cpu().numpy().tobytes() in flat
    assert bool(out.isfinite().all())

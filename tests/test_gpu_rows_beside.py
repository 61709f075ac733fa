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
            plan = M.moe_last_gemm_plan()
            assert (plan["mt"] == 16) if block == 256 else (plan["mt"], plan["nt"], plan["ks"]) == (4, 2, 256), "another tile ran"
            outs.append(out[:T])
    finally:
        M.moe_set_block_m_override(0)
        M.moe_set_reduction_splits(0)
    assert bool(outs[0].isfinite().all()) and torch.equal(outs[0], outs[1])


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("block,T", [(64, 64), (64, 65), (256, 64), (256, 65)])
def test_reordered_rows_of_a_routed_layer(block, T, dtype):
    """Beside the router with the bucketing (up to 64 tokens) and beside the bucketing alone: the plain layer's bits."""
    K, N, E, topk = 1024, 1024, 4, 2
    gen = torch.Generator("cuda").manual_seed(T + block)
    X = torch.randn(T, K, device="cuda", generator=gen).to(DT[dtype])
    logits = torch.randn(T, E, device="cuda", generator=gen)
    ids, w = torch.empty(T, topk, dtype=torch.int32, device="cuda"), torch.empty(T, topk, device="cuda")
    M.moe_route_topk(logits, None, ids, w)
    w1, w2 = weights(E, 2 * N, K, dtype, gen), weights(E, K, N, dtype, gen)
    sizes = (T, K, N, E, topk, M.MOE_F16 if dtype == "f16" else M.MOE_BF16)
    sums = T * topk * (N // 128) * 4 + 256
    plain, routed = (torch.full((T, K), float("nan"), dtype=DT[dtype], device="cuda") for _ in range(2))
    M.moe_set_block_m_override(block)
    M.moe_set_reduction_splits(1 if block == 64 else 0)
    try:
        print(f"[gpu-case] rows beside, routed, block {block} {T} tokens {dtype}", flush=True)
        ws = torch.empty(M.moe_w4a16_layer_workspace_bytes(*sizes) + sums, dtype=torch.uint8, device="cuda")
        M.moe_w4a16_layer(X, ids, w, *w1, *w2, plain, 128, ws)
        ws = torch.empty(M.moe_w4a16_routed_layer_workspace_bytes(*sizes) + sums, dtype=torch.uint8, device="cuda")
        M.moe_w4a16_routed_layer(X, logits, None, *w1, *w2, routed, topk, 128, ws)
        torch.cuda.synchronize()
        assert M.moe_last_gemm_plan()["mt"] == (16 if block == 256 else 4)
    finally:
        M.moe_set_block_m_override(0)
        M.moe_set_reduction_splits(0)
    assert bool(plain.isfinite().all()) and torch.equal(plain, routed)


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
    M.fp8_set_layer_block_m(64)
    try:
        M.fp8_moe_layer(X, ids, w, w1, s1, w2, s2, out, ws)
        torch.cuda.synchronize()
    finally:
        M.fp8_set_layer_block_m(0)
    # align, quantise, product, SiLU and quantise, product, combine
    i32 = lambda *s: torch.zeros(*s, device="cuda", dtype=torch.int32)
    cap = M.moe_align_capacity(T, topk, E, 64)
    counts, offsets, slots, blocks, padded = i32(E), i32(E + 1), i32(cap), i32(cap // 64 + 1), i32(1)
    M.moe_align_by_expert(ids, E, 64, counts, offsets, slots, blocks, padded)
    codes, scales = torch.zeros(T, K, dtype=torch.uint8, device="cuda"), torch.zeros(T, K // 128, device="cuda")
    M.fp8_quantize_rows(X, codes, scales)
    H = torch.zeros(T * topk, 2 * N, dtype=DT[dtype], device="cuda")
    M.fp8_moe_grouped_gemm(codes, scales, topk, w1, s1, slots, blocks, padded, T * topk, 64, H)
    act, sa = torch.zeros(T * topk, N, dtype=torch.uint8, device="cuda"), torch.zeros(T * topk, N // 128, device="cuda")
    M.fp8_silu_mul_quantize(H, act, sa)
    Y = torch.zeros(T * topk, K, device="cuda")
    M.fp8_moe_grouped_gemm(act, sa, 1, w2, s2, slots, blocks, padded, T * topk, 64, Y)
    torch.cuda.synchronize()
    Y = Y.view(T, topk, K)
    want = w[:, :1] * Y[:, 0]
    for j in range(1, topk):      # (a fused multiply-add: the product of two float32 is exact in float64)
        want = (w[:, j:j + 1].double() * Y[:, j].double() + want.double()).float()
    assert bool(out.isfinite().all()) and torch.equal(out, want.to(DT[dtype]))

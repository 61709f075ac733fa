"""FP8 GEMM of up to 64 rows on the kernel whose workgroups split the reduction among their waves: one row, full and ragged
row tiles, the fewest blocks its groups take, counts that no group count divides, every output type.  Where the
plan has planes the workspace shows the route: this kernel leaves it untouched."""
import numpy as np
import pytest
import torch

from moe_workloads.fp8 import Fp8GemmConfig, make_fp8_inputs
from oracle import fp8_oracle as F
from test_gpu_widen_fp8_gemm import error_bound, say

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2504_16214_amd as M_

SHAPES = [  # rows, features, reduction: 16 features and 4 groups, 16 and 8, 32 and 4, 64 and 2, by row tile
    (1, 64, 512), (15, 320, 640), (16, 192, 1920), (9, 2048, 7168), (16, 6656, 512),
    (17, 64, 512), (31, 640, 1152), (32, 1472, 2688), (32, 6656, 640), (21, 14400, 1152), (15, 13952, 512),
    (33, 64, 896), (63, 192, 1152), (64, 1472, 1152), (33, 6656, 1152), (64, 12800, 1024),
    (16, 7744, 1024), (21, 4160, 1024), (32, 8256, 1024), (33, 4160, 1024)]


@pytest.mark.parametrize("rows,n,k", SHAPES)
def test_groups_match_the_oracle(rows, n, k):
    say(f"fp8 gemm groups M={rows} N={n} K={k}")
    inp = make_fp8_inputs(Fp8GemmConfig("g", M=rows, N=n, K=k, seed=rows + n + k))
    A, sa, B, sb = (torch.from_numpy(x).cuda() for x in (inp.a_codes, inp.a_scale, inp.b_codes, inp.b_scale))
    need = M_.fp8_blockwise_gemm_workspace_bytes(rows, n, k)
    ws = torch.full((need,), 255, dtype=torch.uint8, device="cuda") if need else None
    out = {}
    for dtype in (torch.bfloat16, torch.float16, torch.float32):
        # (guard rows behind the output: rows past the last are not stored)
        whole = torch.full((rows + 64, n), 7.0, dtype=dtype, device="cuda")
        M_.fp8_blockwise_gemm(A, sa, B, sb, whole[:rows], ws)
        torch.cuda.synchronize()
        assert bool((whole[rows:] == 7.0).all())
        out[dtype] = whole[:rows].clone()
    if need:
        assert bool((ws == 255).all()), "the planes were written"
    for dtype in (torch.bfloat16, torch.float16):
        assert torch.equal(out[torch.float32].to(dtype), out[dtype])
    want = F.blockwise_gemm(inp.a_codes, inp.a_scale, inp.b_codes, inp.b_scale, "bf16")
    bound = error_bound(want, inp.a_codes, inp.a_scale, inp.b_codes, inp.b_scale)
    assert float((np.abs(out[torch.bfloat16].double().cpu().numpy() - want) / bound).max()) <= 1.0
    # the tiles with planes, in their order of summation: float32 sums of K / 128 terms
    M_.fp8_set_plan_override(1 if rows <= 16 else 2 if rows <= 32 else 4, 1, 1, 0)
    try:
        tiles = torch.empty_like(out[torch.float32])
        M_.fp8_blockwise_gemm(A, sa, B, sb, tiles, None)
    finally:
        M_.fp8_set_plan_override(0, 0, 0, 0)
    assert float((tiles - out[torch.float32]).norm() / tiles.norm()) <= 2.0 ** -24 * (k // 128 + 8)


@pytest.mark.parametrize("rows,n,k", [(15, 2432, 13952), (24, 192, 4608), (33, 1024, 4096)])
def test_calls_left_to_the_planes(rows, n, k):
    """Splits that lie too close to call, or are faster: the planes are written."""
    say(f"fp8 gemm planes M={rows} N={n} K={k}")
    inp = make_fp8_inputs(Fp8GemmConfig("p", M=rows, N=n, K=k, seed=rows + n + k))
    A, sa, B, sb = (torch.from_numpy(x).cuda() for x in (inp.a_codes, inp.a_scale, inp.b_codes, inp.b_scale))
    ws = torch.full((M_.fp8_blockwise_gemm_workspace_bytes(rows, n, k),), 255, dtype=torch.uint8, device="cuda")
    out = torch.empty(rows, n, dtype=torch.bfloat16, device="cuda")
    M_.fp8_blockwise_gemm(A, sa, B, sb, out, ws)
    torch.cuda.synchronize()
    assert bool((ws[:rows * n * 4] != 255).any()), "another kernel ran"
    want = F.blockwise_gemm(inp.a_codes, inp.a_scale, inp.b_codes, inp.b_scale, "bf16")
    bound = error_bound(want, inp.a_codes, inp.a_scale, inp.b_codes, inp.b_scale)
    assert float((np.abs(out.double().cpu().numpy() - want) / bound).max()) <= 1.0

"""GPU tests of the vector products' forms: gate/up with 64 columns a workgroup or 32 and the reduction in halves (odd
numbers of groups, halves of unequal length, either side of the line between the forms), pairs of groups whose
second half lies past a row's end, the last row of the last expert included, and a workspace that has no room for act as digits.
Whole output against the CPU oracle, with the tolerance of the random-shape module."""
from __future__ import annotations

import pytest
import torch

from moe_workloads import MoEConfig, make_inputs
from test_gpu_random_shapes import check_case, say

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2504_16214_amd as M
    import gpu_util as U


# Workgroups of 64 columns (N / 64 * T * topk): 252 | 256; K 384 (never halved), 512 and 640 (2 + 2, 2 + 3 groups), 896 (4 + 3);
# K 4224, 8320 and 8448: more activations than the first loads bring (1, 2 rounds); 256 | 378 | 384, 528 | 640 workgroups, K 1024 and more
@pytest.mark.parametrize("K,N,E,topk,T", [(512, 8064, 4, 1, 2), (512, 8192, 4, 1, 2), (384, 128, 4, 2, 3), (640, 384, 8, 3, 2), (896, 896, 8, 1, 5),
                                          (4224, 256, 4, 2, 1), (8320, 128, 4, 1, 1), (8448, 1024, 16, 4, 1),
                                          (1024, 8192, 2, 1, 2), (1152, 8064, 2, 1, 3), (1024, 8192, 2, 1, 3), (1024, 2816, 4, 1, 12), (1024, 2560, 4, 1, 16)])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_forms_of_the_gate_up_product(K, N, E, topk, T, dtype):
    cfg = MoEConfig("few_forms", T=T, K=K, N=N, E=E, topk=topk, group=128, dtype=dtype, seed=K + N + T)
    inp = make_inputs(cfg)
    ids = inp.topk_ids.copy()
    ids[-1, -1] = E - 1                       # the end of the weights
    if topk == 1 or (ids[-1, :-1] != E - 1).all():
        inp.topk_ids = ids
    say(f"forms {cfg}")
    check_case(inp, str(cfg))
    assert M.moe_last_gemm_plan()["mt"] == 0


# act vectors of more than 80 KB beside more than 256 workgroups: two rounds of 4 slots, 2 + 1, 5 + 4, three rounds of one, and either side of both lines
@pytest.mark.parametrize("K,N,E,topk,T", [(4224, 2432, 8, 8, 1), (4224, 6528, 4, 3, 1), (2176, 2304, 16, 9, 2), (4224, 7680, 4, 3, 1),
                                          (4096, 2432, 8, 8, 1), (4224, 2304, 8, 8, 1)])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_act_in_rounds(K, N, E, topk, T, dtype):
    cfg = MoEConfig("few_rounds", T=T, K=K, N=N, E=E, topk=topk, group=128, dtype=dtype, seed=K + N + T)
    inp = make_inputs(cfg)
    inp.topk_ids[-1, -2] = -1                 # a slot without an expert, in the last round
    say(f"rounds {cfg}")
    check_case(inp, str(cfg))
    assert M.moe_last_gemm_plan()["mt"] == 0


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_act_in_rounds_has_the_same_bits_in_operand_order(dtype):
    """4 + 3 slots."""
    cfg = MoEConfig("few_rounds", T=1, K=5120, N=3072, E=8, topk=7, group=128, dtype=dtype, seed=12)
    say(f"rounds, operand order {cfg}")
    d = U.DevInputs(make_inputs(cfg))
    plain = U.run_layer(d)
    assert M.moe_last_gemm_plan()["mt"] == 0
    p1, p2 = torch.empty_like(d.qw1), torch.empty_like(d.qw2)
    M.moe_repack_qweight(d.qw1, False, p1)
    M.moe_repack_qweight(d.qw2, True, p2)
    out = torch.full_like(plain, float("nan"))
    ws = torch.full((M.moe_w4a16_layer_workspace_bytes(1, 5120, 3072, 8, 7, M.MOE_F16 if dtype == "f16" else M.MOE_BF16),), 255, dtype=torch.uint8, device="cuda")
    M.moe_w4a16_layer_prepacked(d.X, d.ids, d.w, p1, d.s1, d.z1, p2, d.s2, d.z2, out, 128, ws)
    torch.cuda.synchronize()
    assert M.moe_last_gemm_plan()["mt"] == 0 and bool(plain.isfinite().all()) and torch.equal(out.view(torch.int16), plain.view(torch.int16))


def test_a_workspace_without_room_for_the_digits_runs_on_a_tile():
    """A long act beside a short output: the bytes that the tiles need do not hold act as digits, and one block
    less than the size query names is between the two.  Accepted
    all the same, with the oracle's results, and nothing behind them is written."""
    cfg = MoEConfig("few_small_ws", T=2, K=256, N=4096, E=4, topk=2, group=128, dtype="f16", seed=8)
    inp = make_inputs(cfg)
    d = U.DevInputs(inp)
    need = M.moe_w4a16_layer_workspace_bytes(cfg.T, cfg.K, cfg.N, cfg.E, cfg.topk, M.MOE_F16)
    less = need - 256
    say(f"small workspace {cfg}: {less} of {need}")
    buf = torch.full((need,), 255, dtype=torch.uint8, device="cuda")
    outs = []
    for n, vector in ((need, True), (less, False)):
        buf.fill_(255)
        out = torch.full((cfg.T, cfg.K), float("nan"), dtype=torch.float16, device="cuda")
        M.moe_w4a16_layer(d.X, d.ids, d.w, d.qw1, d.s1, d.z1, d.qw2, d.s2, d.z2, out, cfg.group, buf[:n])
        torch.cuda.synchronize()
        assert (M.moe_last_gemm_plan()["mt"] == 0) == vector and bool((buf[n:] == 255).all())
        outs.append(U.dev_to_f64(out))
    # two roundings of act and one of the output, as far as the random-shape module lets two kernels differ
    U.assert_close(outs[1], outs[0], str(cfg))

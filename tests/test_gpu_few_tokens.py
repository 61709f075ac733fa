"""GPU tests of the vector-product kernels that moe_w4a16_layer runs for a few tokens (Section II-C's FP16 x
INT4 semantics at the smallest batches): reductions of a half step, of ragged panels and of several
panels, one and several parts of the down projection, both weight layouts, ids out of range, subnormal
and infinite activations; whole output against the CPU oracle with the tolerance of the random-shape
module (fp16 0.02 + 0.01 |oracle|; bf16 plus what one differently rounded activation moves)."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from moe_workloads import MoEConfig, make_inputs
from oracle import moe_oracle as O
from test_gpu_random_shapes import check_case, say

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2504_16214_amd as M
    import gpu_util as U


def ran_without_a_tile():
    return M.moe_last_gemm_plan()["mt"] == 0


# K, N, E, topk, T: one group; half step and ragged panels; a panel and a group; four down parts;
# more slots than waves; more than 4 x 256 x 8 staged values (the staging loop's tail)
SHAPES = [
    (128, 128, 4, 1, 1),
    (128, 256, 8, 2, 16),
    (384, 640, 4, 3, 2),
    (1152, 1152, 8, 2, 3),
    (1024, 4224, 4, 1, 2),
    (256, 512, 40, 10, 3),
    (8320, 1024, 16, 8, 1),
]


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("K,N,E,topk,T", SHAPES)
def test_few_tokens_against_the_oracle(K, N, E, topk, T, dtype):
    cfg = MoEConfig("few", T=T, K=K, N=N, E=E, topk=topk, group=128, dtype=dtype, seed=K + N)
    inp = make_inputs(cfg)
    if topk > 1:                       # a slot that contributes nothing, below and above the range
        ids = inp.topk_ids.copy()
        ids[0, 0], ids[-1, -1] = -1, E
        inp.topk_ids = ids
    say(f"few tokens {cfg}")
    check_case(inp, str(cfg))
    assert ran_without_a_tile()


def test_the_rule_ends_where_slots_share_experts():
    for T, few in ((16, True), (17, False)):
        cfg = MoEConfig("few_edge", T=T, K=256, N=512, E=8, topk=2, group=128, dtype="f16", seed=T)
        say(f"edge of the rule {cfg}")
        check_case(make_inputs(cfg), str(cfg))
        assert ran_without_a_tile() == few


@pytest.mark.parametrize("T,few", [(8, True), (24, False)])
def test_the_rule_ends_where_many_tokens_have_few_slots(T, few):
    """One expert a token: the down launch has a workgroup for every token, most of whose waves idle."""
    cfg = MoEConfig("few_top1", T=T, K=1024, N=1024, E=24, topk=1, group=128, dtype="f16", seed=T)
    say(f"edge of the rule {cfg}")
    check_case(make_inputs(cfg), str(cfg))
    assert ran_without_a_tile() == few


@pytest.mark.parametrize("K,N,E,topk,T,dtype,few", [
    (2048, 1408, 64, 6, 5, "f16", True),       # 38 us where the tiles take 46: what the launches save outweighs weights read twice
    (2048, 2048, 64, 4, 5, "bf16", True),
    (7168, 2048, 64, 1, 8, "f16", True),       # 39 and 53; one expert a token
    (4096, 2048, 8, 2, 7, "f16", False),       # fourteen slots on eight experts
    (1024, 1024, 24, 1, 20, "bf16", True),     # five rounds of down workgroups
])
def test_where_the_vector_products_are_chosen(K, N, E, topk, T, dtype, few):
    cfg = MoEConfig("few_rule", T=T, K=K, N=N, E=E, topk=topk, group=128, dtype=dtype, seed=T)
    say(f"rule for a few tokens {cfg}")
    check_case(make_inputs(cfg), str(cfg))
    assert ran_without_a_tile() == few


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_few_tokens_in_operand_order_are_the_same_bits(dtype):
    cfg = MoEConfig("few_pre", T=2, K=2048, N=1024, E=6, topk=3, group=128, dtype=dtype, seed=5)
    d = U.DevInputs(make_inputs(cfg))
    say(f"operand order {cfg}")
    plain = U.run_layer(d).clone()
    assert ran_without_a_tile()
    p1, p2 = torch.empty_like(d.qw1), torch.empty_like(d.qw2)
    M.moe_repack_qweight(d.qw1, False, p1)
    M.moe_repack_qweight(d.qw2, True, p2)
    ws = torch.empty(M.moe_w4a16_layer_workspace_bytes(cfg.T, cfg.K, cfg.N, cfg.E, cfg.topk,
                                                       M.MOE_F16 if dtype == "f16" else M.MOE_BF16),
                     dtype=torch.uint8, device="cuda")
    out = torch.full_like(plain, float("nan"))
    M.moe_w4a16_layer_prepacked(d.X, d.ids, d.w, p1, d.s1, d.z1, p2, d.s2, d.z2, out, cfg.group, ws)
    torch.cuda.synchronize()
    assert ran_without_a_tile() and torch.equal(out, plain)


def test_subnormal_activations_keep_their_digits():
    """Activations of about 2^-16 (half of them subnormal in fp16) with gate/up scales 2^15 times
    larger: the results are of the usual size, so a flushed activation would show at once."""
    cfg = MoEConfig("few_subnormal", T=2, K=512, N=512, E=8, topk=2, group=128, dtype="f16", seed=9)
    inp = make_inputs(cfg)
    x = inp.x_bits.view(np.float16).astype(np.float64) * 2.0 ** -15
    s1 = inp.s1_bits.view(np.float16).astype(np.float64) * 2.0 ** 15
    assert np.abs(x).min() < 2.0 ** -14 and s1.max() < 65504
    inp.x_bits = x.astype(np.float16).view(inp.x_bits.dtype)
    inp.s1_bits = s1.astype(np.float16).view(inp.s1_bits.dtype)
    say(f"subnormal activations {cfg}")
    check_case(inp, str(cfg))
    assert ran_without_a_tile()


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_an_infinite_activation_stays_in_its_token(dtype):
    cfg = MoEConfig("few_inf", T=3, K=512, N=512, E=8, topk=2, group=128, dtype=dtype, seed=3)
    inp = make_inputs(cfg)
    say(f"infinite activation {cfg}")
    clean = U.dev_to_f64(U.run_layer(U.DevInputs(inp)))
    bits = inp.x_bits.copy()
    bits[1, 77] = {"f16": 0x7C00, "bf16": 0x7F80}[dtype]
    inp.x_bits = bits
    got = U.dev_to_f64(U.run_layer(U.DevInputs(inp)))
    assert ran_without_a_tile()
    M.moe_set_block_m_override(16)
    try:
        tiled = U.dev_to_f64(U.run_layer(U.DevInputs(inp)))
    finally:
        M.moe_set_block_m_override(0)
    assert np.array_equal(got[[0, 2]], clean[[0, 2]])
    assert np.array_equal(np.isfinite(got), np.isfinite(tiled)) and not np.isfinite(got[1]).any()


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("with_bias", [False, True])
def test_routed_layer_of_a_few_tokens(dtype, with_bias):
    """Router and vector products behind one call: the oracle chain, and the bits of the plain entry."""
    cfg = MoEConfig("few_routed", T=16, K=256, N=512, E=8, topk=2, group=128, dtype=dtype, seed=21)
    say(f"routed, few tokens {cfg} bias={with_bias}")
    inp = make_inputs(cfg)
    bias = np.linspace(1.0, -1.0, cfg.E).astype(np.float32) if with_bias else None
    inp.topk_ids, w = O.route_topk(inp.logits, cfg.topk, bias=bias)
    inp.topk_weights = w.astype(np.float32)
    d = U.DevInputs(inp)
    logits, bd = torch.from_numpy(inp.logits).cuda(), None if bias is None else torch.from_numpy(bias).cuda()
    ws = torch.full((M.moe_w4a16_routed_layer_workspace_bytes(cfg.T, cfg.K, cfg.N, cfg.E, cfg.topk,
                                                              M.MOE_F16 if dtype == "f16" else M.MOE_BF16),),
                    255, dtype=torch.uint8, device="cuda")
    out = torch.full((cfg.T, cfg.K), float("nan"), dtype=U.TORCH_DT[dtype], device="cuda")
    M.moe_w4a16_routed_layer(d.X, logits, bd, d.qw1, d.s1, d.z1, d.qw2, d.s2, d.z2, out, cfg.topk, cfg.group, ws)
    torch.cuda.synchronize()
    assert ran_without_a_tile()
    check_case(inp, str(cfg))
    assert ran_without_a_tile()
    M.moe_route_topk(logits, bd, d.ids, d.w)
    assert torch.equal(out, U.run_layer(d))


@pytest.mark.parametrize("E,topk,T", [(64, 6, 4), (65, 6, 4), (17, 16, 1), (17, 17, 1), (5, 5, 6)])
def test_routing_inside_the_gate_up_launch(E, topk, T):
    """Either side of the limits (64 experts, 16 a token), with ties and signed zeros among the logits: the bits of
    the plain entry on the ids and weights of the stand-alone router."""
    cfg = MoEConfig("few_route_in", T=T, K=256, N=512, E=E, topk=topk, group=128, dtype="f16", seed=E + topk)
    say(f"routing inside {cfg}")
    inp = make_inputs(cfg)
    inp.logits[:] = np.round(inp.logits)              # many ties
    inp.logits[0, :3] = [0.0, -0.0, 0.0]
    d = U.DevInputs(inp)
    logits = torch.from_numpy(inp.logits).cuda()
    M.moe_route_topk(logits, None, d.ids, d.w)
    want = U.run_layer(d)
    assert ran_without_a_tile()
    ws = torch.full((M.moe_w4a16_routed_layer_workspace_bytes(T, cfg.K, cfg.N, E, topk, M.MOE_F16),), 255, dtype=torch.uint8, device="cuda")
    out = torch.full((T, cfg.K), float("nan"), dtype=torch.float16, device="cuda")
    M.moe_w4a16_routed_layer(d.X, logits, None, d.qw1, d.s1, d.z1, d.qw2, d.s2, d.z2, out, topk, cfg.group, ws)
    torch.cuda.synchronize()
    assert ran_without_a_tile() and torch.equal(out, want)


@pytest.mark.parametrize("K,N,E,topk,T", [(128, 30592, 4, 1, 1), (128, 30592, 4, 1, 2), (128, 15104, 4, 2, 1), (256, 30592, 4, 1, 2)])
def test_the_chunk_floats_stay_within_the_workspace(K, N, E, topk, T):
    """The longest rows against the shortest outputs: act's digits and its chunks' words, from where act lies on the other
    paths on, need more than those do.  Nothing behind the workspace of the size query is written."""
    cfg = MoEConfig("few_room", T=T, K=K, N=N, E=E, topk=topk, group=128, dtype="f16", seed=K + T)
    say(f"room for the chunk floats {cfg}")
    inp = make_inputs(cfg)
    d = U.DevInputs(inp)
    need = M.moe_w4a16_layer_workspace_bytes(T, K, N, E, topk, M.MOE_F16)
    assert cfg.S * (N * 4 + N // 32 * 8) <= need
    buf = torch.full((need + 4096,), 255, dtype=torch.uint8, device="cuda")
    out = torch.full((T, K), float("nan"), dtype=torch.float16, device="cuda")
    M.moe_w4a16_layer(d.X, d.ids, d.w, d.qw1, d.s1, d.z1, d.qw2, d.s2, d.z2, out, 128, buf[:need])
    torch.cuda.synchronize()
    assert ran_without_a_tile() and bool((buf[need:] == 255).all())
    check_case(inp, str(cfg))

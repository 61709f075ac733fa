"""GPU parity of the layer on its 64-slot tile (9 to 60 rows per expert, group 128): every number of live
16-slot parts of a block, experts of more than one block, both weight layouts, reductions from one panel of
1024 to an odd number of them, split and unsplit, several tiles per workgroup, zero scales and ignored ids."""
import copy
import dataclasses

import numpy as np
import pytest
import torch

from moe_workloads import MoEConfig, make_inputs
from test_gpu_twogroup_layer import _check, _inputs

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import gpu_util as U
    import paper_2504_16214_amd as M


def _on_mid():
    plan = M.moe_last_gemm_plan()
    return (plan["mt"], plan["ks"], plan["waves"]) == (4, 256, 4)


def _layer(inp, prepacked=False, tiles=0, splits=0):
    d, c = U.DevInputs(inp), inp.cfg
    out = torch.full((c.T, c.K), float("nan"), dtype=U.TORCH_DT[c.dtype], device="cuda")
    mdt = M.MOE_F16 if c.dtype == "f16" else M.MOE_BF16
    M.moe_set_block_m_override(64)
    M.moe_set_tiles_per_workgroup(tiles)
    M.moe_set_reduction_splits(splits)
    try:
        # (room for the bf16 row sums, which the size query adds only where the tile is the automatic choice)
        need = M.moe_w4a16_layer_workspace_bytes(c.T, c.K, c.N, c.E, c.topk, mdt) + c.S * (c.N // 128) * 4 + 256
        ws = torch.full((need,), 255, dtype=torch.uint8, device="cuda")
        if prepacked:
            p1, p2 = torch.empty_like(d.qw1), torch.empty_like(d.qw2)
            M.moe_repack_qweight(d.qw1, False, p1)
            M.moe_repack_qweight(d.qw2, True, p2)
            M.moe_w4a16_layer_prepacked(d.X, d.ids, d.w, p1, d.s1, d.z1, p2, d.s2, d.z2, out, c.group, ws)
        else:
            M.moe_w4a16_layer(d.X, d.ids, d.w, d.qw1, d.s1, d.z1, d.qw2, d.s2, d.z2, out, c.group, ws)
        torch.cuda.synchronize()
        assert _on_mid(), M.moe_last_gemm_plan()
        if splits:
            assert M.moe_last_gemm_plan()["reduction_splits"] == min(splits, c.N // 1024)
    finally:
        M.moe_set_block_m_override(0)
        M.moe_set_tiles_per_workgroup(0)
        M.moe_set_reduction_splits(0)
    return out


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("K,N,zero_scales", [(1024, 1024, True), (3072, 1024, False), (1024, 2048, False)])
def test_every_live_part_count(dtype, K, N, zero_scales):
    counts = [1, 15, 16, 17, 0, 32, 33, 48, 49, 63, 64, 65, 100, 130]
    print(f"64-slot layer {dtype} K={K} N={N}", flush=True)
    inp = _inputs(dtype, K, N, counts, seed=900 + K + N, zero_scales=zero_scales, bad_ids=5)
    got = _layer(inp)
    _check(inp, got, f"64-slot layer {dtype} K={K} N={N}")
    bad = (inp.topk_ids[:, 0] < 0) | (inp.topk_ids[:, 0] >= inp.cfg.E)
    assert np.all(U.dev_to_f64(got)[bad] == 0)
    same = _layer(inp, prepacked=True)
    assert torch.equal(got.view(torch.int16), same.view(torch.int16)), "operand-order weights: same words, same order"


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("tiles", [3, 8])
def test_tiles_per_workgroup(dtype, tiles):
    """Walking several feature tiles with one load pipeline gives the same bits as one tile each."""
    inp = _inputs(dtype, 2048, 1024, [7, 20, 40, 60, 90], seed=901)
    print(f"64-slot layer {dtype} tiles per workgroup {tiles}", flush=True)
    got = _layer(inp, tiles=tiles)
    _check(inp, got, f"tiles {tiles}")
    assert torch.equal(got.view(torch.int16), _layer(inp, tiles=1).view(torch.int16))


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("splits", [2, 3])
def test_split_down_product(dtype, splits):
    inp = _inputs(dtype, 1024, 3072, [5, 16, 30, 50, 20], seed=902)
    print(f"64-slot layer {dtype} splits {splits}", flush=True)
    _check(inp, _layer(inp, splits=splits), f"splits {splits}")


def test_small_workspace_falls_back():
    """bf16 without room for the row sums: the layer runs on the other tiles, within the same bound."""
    inp = _inputs("bf16", 1024, 1024, [10, 26, 40], seed=903)
    d, c = U.DevInputs(inp), inp.cfg
    out = torch.empty((c.T, c.K), dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(M.moe_w4a16_layer_workspace_bytes(c.T, c.K, c.N, c.E, c.topk, M.MOE_BF16), dtype=torch.uint8, device="cuda")
    M.moe_set_block_m_override(64)
    try:
        M.moe_w4a16_layer(d.X, d.ids, d.w, d.qw1, d.s1, d.z1, d.qw2, d.s2, d.z2, out, c.group, ws)
        torch.cuda.synchronize()
        assert not _on_mid()
    finally:
        M.moe_set_block_m_override(0)
    _check(inp, out, "fallback")


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_automatic_choice_through_the_three_entries(dtype):
    """Several slots a token, the workspace of the size query (with the planes of a split down product) and no
    override: the plain layer against the oracle, the prepacked and the routed one with the same bits."""
    cfg = MoEConfig("mid_auto", T=44, K=2048, N=20480, E=8, topk=2, group=128, dtype=dtype, seed=904)
    print(f"64-slot layer, automatic choice {cfg}", flush=True)
    inp = make_inputs(cfg)
    d = U.DevInputs(inp)
    logits = torch.from_numpy(inp.logits).cuda()
    M.moe_route_topk(logits, None, d.ids, d.w)
    inp.topk_ids, inp.topk_weights = d.ids.cpu().numpy(), d.w.cpu().numpy()
    got = U.run_layer(d)
    assert _on_mid() and M.moe_last_gemm_plan()["reduction_splits"] > 1
    _check(inp, got, "plain entry")
    sizes = (cfg.T, cfg.K, cfg.N, cfg.E, cfg.topk, M.MOE_F16 if dtype == "f16" else M.MOE_BF16)
    p1, p2 = torch.empty_like(d.qw1), torch.empty_like(d.qw2)
    M.moe_repack_qweight(d.qw1, False, p1)
    M.moe_repack_qweight(d.qw2, True, p2)
    out = torch.full_like(got, float("nan"))
    ws = torch.full((M.moe_w4a16_layer_workspace_bytes(*sizes),), 255, dtype=torch.uint8, device="cuda")
    M.moe_w4a16_layer_prepacked(d.X, d.ids, d.w, p1, d.s1, d.z1, p2, d.s2, d.z2, out, cfg.group, ws)
    torch.cuda.synchronize()
    assert _on_mid() and torch.equal(out.view(torch.int16), got.view(torch.int16))
    out = torch.full_like(got, float("nan"))
    ws = torch.full((M.moe_w4a16_routed_layer_workspace_bytes(*sizes),), 255, dtype=torch.uint8, device="cuda")
    M.moe_w4a16_routed_layer(d.X, logits, None, d.qw1, d.s1, d.z1, d.qw2, d.s2, d.z2, out, cfg.topk, cfg.group, ws)
    torch.cuda.synchronize()
    assert _on_mid() and torch.equal(out.view(torch.int16), got.view(torch.int16))


def _drawn_layer(K, N, E, T, topk, dtype, seed):
    """Arguments of a large layer, drawn on the device."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    tdt = U.TORCH_DT[dtype]

    def weight(rows, red):
        q = torch.randint(-2 ** 31, 2 ** 31, (E, rows, red // 8), generator=g, device="cuda", dtype=torch.int32)
        s = (torch.rand(E, rows, red // 128, generator=g, device="cuda") * 0.018 + 0.002).to(tdt)
        z = torch.randint(0, 16, (E, rows, red // 128), generator=g, device="cuda", dtype=torch.uint8)
        return q, s, z

    X = (0.5 * torch.randn(T, K, generator=g, device="cuda")).to(tdt)
    top, ids = torch.topk(torch.randn(T, E, generator=g, device="cuda"), topk, dim=1)
    return [X, ids.int().contiguous(), torch.softmax(top, dim=1), *weight(2 * N, K), *weight(K, N)]


@pytest.mark.parametrize("N,T,topk,dtype,splits", [(14336, 504, 2, "bf16", 2),     # two planes and the row sums: within the array of 64 MiB
                                                  (13312, 447, 2, "f16", 2),      # within it as well
                                                  (17408, 504, 2, "bf16", 1)])    # two planes would not be
def test_the_call_without_a_workspace_has_the_same_bits(N, T, topk, dtype, splits):
    """16 experts of K 4096, whose down product wants two splits: the entry without a workspace runs in as
    many as the one with the workspace of the size query."""
    K, E = 4096, 16
    print(f"64-slot layer without a workspace N={N} T={T} {dtype}", flush=True)
    args = _drawn_layer(K, N, E, T, topk, dtype, 905)
    need = M.moe_w4a16_layer_workspace_bytes(T, K, N, E, topk, M.MOE_F16 if dtype == "f16" else M.MOE_BF16)
    assert need <= 64 << 20
    got, want = (torch.full((T, K), float("nan"), dtype=U.TORCH_DT[dtype], device="cuda") for _ in range(2))
    M.moe_w4a16_layer(*args, want, 128, torch.full((need,), 255, dtype=torch.uint8, device="cuda"))
    assert _on_mid() and M.moe_last_gemm_plan()["reduction_splits"] == splits
    M.moe_w4a16_layer_noalloc(*args, got, 128)
    torch.cuda.synchronize()
    assert _on_mid() and M.moe_last_gemm_plan()["reduction_splits"] == splits
    assert torch.isfinite(want).all() and torch.equal(got.view(torch.int16), want.view(torch.int16))


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_workspace_without_room_for_all_planes(dtype):
    """A workspace from what the layer cannot do without (with the row sums) up to the size query: as many splits as
    it has planes for, within the bound, and nothing written behind it."""
    cfg = MoEConfig("mid_planes", T=120, K=2048, N=20480, E=8, topk=2, group=128, dtype=dtype, seed=906)
    print(f"64-slot layer, planes {cfg}", flush=True)
    inp = make_inputs(cfg)
    d = U.DevInputs(inp)
    need = M.moe_w4a16_layer_workspace_bytes(cfg.T, cfg.K, cfg.N, cfg.E, cfg.topk, M.MOE_F16 if dtype == "f16" else M.MOE_BF16)
    seen = set()
    for planes in range(7):
        size = need - planes * cfg.S * cfg.K * 4
        buf = torch.full((need,), 255, dtype=torch.uint8, device="cuda")
        out = torch.full((cfg.T, cfg.K), float("nan"), dtype=U.TORCH_DT[dtype], device="cuda")
        try:
            M.moe_w4a16_layer(d.X, d.ids, d.w, d.qw1, d.s1, d.z1, d.qw2, d.s2, d.z2, out, cfg.group, buf[:size])
        except M.MoEError as e:
            assert e.status == 3 and planes > 0
            break
        torch.cuda.synchronize()
        assert bool((buf[size:] == 255).all()), "written behind the workspace"
        if _on_mid():
            seen.add(M.moe_last_gemm_plan()["reduction_splits"])
        _check(inp, out, f"{planes} planes less")
    assert len(seen) > 1


@pytest.mark.parametrize("avg", [40, 64])
def test_operand_order_weights_split_with_the_queried_workspace(avg):
    """fp16 operand-order weights take this tile up to 71 rows per expert, stated ones up to 55: the splits of the down
    product do not drop in between, and the bits are those of the stated layout on the same tile."""
    K, N, E, T = 3072, 12288, 8, 4 * avg
    print(f"64-slot layer, operand order, {avg} rows per expert", flush=True)
    X, ids, w, q1, s1, z1, q2, s2, z2 = _drawn_layer(K, N, E, T, 2, "f16", 907)
    p1, p2 = torch.empty_like(q1), torch.empty_like(q2)
    M.moe_repack_qweight(q1, False, p1)
    M.moe_repack_qweight(q2, True, p2)
    ws = torch.full((M.moe_w4a16_layer_workspace_bytes(T, K, N, E, 2, M.MOE_F16),), 255, dtype=torch.uint8, device="cuda")
    got, want = (torch.full((T, K), float("nan"), dtype=torch.float16, device="cuda") for _ in range(2))
    M.moe_w4a16_layer_prepacked(X, ids, w, p1, s1, z1, p2, s2, z2, got, 128, ws)
    assert _on_mid() and M.moe_last_gemm_plan()["reduction_splits"] == 4
    M.moe_set_block_m_override(64)
    try:
        M.moe_w4a16_layer(X, ids, w, q1, s1, z1, q2, s2, z2, want, 128, ws)
        assert _on_mid() and M.moe_last_gemm_plan()["reduction_splits"] == 4
    finally:
        M.moe_set_block_m_override(0)
    torch.cuda.synchronize()
    assert torch.isfinite(got).all() and torch.equal(got, want)


@pytest.mark.parametrize("dtype,pre,K,N,E,avg,on", [
    ("f16", False, 2048, 4096, 32, 20, False), ("f16", False, 2048, 4096, 32, 28, True),      # small layers
    ("f16", True, 2048, 4096, 32, 20, True), ("f16", True, 1024, 4096, 64, 20, False),
    ("f16", False, 4096, 4096, 32, 20, True), ("f16", False, 4096, 4096, 32, 56, False),
    ("f16", True, 4096, 4096, 32, 71, True),
    ("bf16", False, 4096, 4096, 32, 63, True), ("bf16", False, 4096, 4096, 32, 64, False),    # half the experts need a second block
    ("bf16", True, 4096, 4096, 32, 72, True), ("bf16", False, 4096, 12288, 8, 72, True),
])
def test_where_the_tile_is_chosen(dtype, pre, K, N, E, avg, on):
    """Either side of the rule's lines: where even routing on this tile takes longer than before it, the layer runs on another."""
    print(f"64-slot layer, choice {dtype} K={K} N={N} E={E} avg={avg} pre={pre}", flush=True)
    T = avg * E
    args = _drawn_layer(K, N, E, T, 1, dtype, 908)        # (any words stand for repacked ones: only the choice is looked at)
    ws = torch.empty(M.moe_w4a16_layer_workspace_bytes(T, K, N, E, 1, M.MOE_F16 if dtype == "f16" else M.MOE_BF16), dtype=torch.uint8, device="cuda")
    out = torch.empty(T, K, dtype=U.TORCH_DT[dtype], device="cuda")
    (M.moe_w4a16_layer_prepacked if pre else M.moe_w4a16_layer)(*args, out, 128, ws)
    torch.cuda.synchronize()
    assert _on_mid() == on, M.moe_last_gemm_plan()


def _other_tile(inp):
    """The layer on 16-slot blocks."""
    M.moe_set_block_m_override(16)
    try:
        return U.run_layer(U.DevInputs(inp))
    finally:
        M.moe_set_block_m_override(0)


def _block_64(inp):
    """The layer in blocks of 64: this tile where the shapes admit it, else the 64 x 128 tile with its scales in LDS."""
    if inp.cfg.group == 128 and inp.cfg.K % 1024 == 0 and inp.cfg.N % 1024 == 0:
        return _layer(inp)
    M.moe_set_block_m_override(64)
    try:
        out = U.run_layer(U.DevInputs(inp))
        plan = M.moe_last_gemm_plan()
        assert (plan["mt"], plan["nt"], plan["ks"], plan["register_scales"]) == (4, 2, 128, 0), plan
        return out
    finally:
        M.moe_set_block_m_override(0)


# this tile; the 64 x 128 tile with its scales in LDS: row sums in bf16 at any size and in large launches only, former zero points
BLOCKS_OF_64 = [(128, 1024, 75), (256, 1024, 75), (64, 512, 5200), (32, 1024, 75)]


@pytest.mark.parametrize("group,N,T", BLOCKS_OF_64)
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("what", ["infinity", "NaN"])
def test_an_infinite_activation_stays_in_its_token(group, N, T, dtype, what):
    """Also where the zero points leave by sums over rows that share an instruction: every other token has the bits it
    had, and that token is as on the 16-slot tile."""
    cfg = MoEConfig("mid_inf", T=T, K=1024, N=N, E=3, topk=1, group=group, dtype=dtype, seed=909)
    print(f"blocks of 64, {what} {cfg}", flush=True)
    inp = make_inputs(cfg)
    clean = U.dev_to_f64(_block_64(inp))
    bits = inp.x_bits.copy()
    for t, k in ((0, 0), (20, 77), (T - 1, 1023)):
        bits[t, k] = {("f16", "infinity"): 0x7C00, ("bf16", "infinity"): 0xFF80, ("f16", "NaN"): 0x7E01, ("bf16", "NaN"): 0x7FC1}[dtype, what]
    inp.x_bits = bits
    got, tiled = U.dev_to_f64(_block_64(inp)), U.dev_to_f64(_other_tile(inp))
    others = np.setdiff1d(np.arange(T), [0, 20, T - 1])
    assert np.isfinite(clean).all() and np.array_equal(got[others], clean[others])
    assert np.array_equal(np.isfinite(got), np.isfinite(tiled)) and not np.isfinite(got[[0, 20, T - 1]]).any()


@pytest.mark.parametrize("group,N,T", BLOCKS_OF_64[:3])
def test_the_largest_bf16_scales(group, N, T):
    """Zero points by row sums: scales up to the type's largest value on activations that are small in proportion: no product of a scale and a zero point
    leaves the float32 range by itself.  Tolerance: two bf16 roundings (act, output) of sums that agree to 2^-9 of
    their magnitude."""
    cfg = MoEConfig("mid_big", T=T, K=1024, N=N, E=3, topk=1, group=group, dtype="bf16", seed=910)
    print(f"blocks of 64, largest scales {cfg}", flush=True)
    inp = make_inputs(cfg)
    s1 = inp.s1_bits.copy()
    s1 -= 20 << 7                                   # 2^-20: act of about 2^-40
    inp.s1_bits = s1
    inp.s2_bits = inp.s2_bits.copy()
    inp.s2_bits[:, ::3, 1::2] = 0x7F7F              # 3.39e38
    inp.s2_bits[:, 1::3, ::2] = 0x7E80              # 8.5e37
    inp.z2 = inp.z2.copy()
    inp.z2[:, ::5] = 15
    got, tiled = U.dev_to_f64(_block_64(inp)), U.dev_to_f64(_other_tile(inp))
    assert np.isfinite(tiled).all() and np.isfinite(got).all()
    rms = np.sqrt((tiled ** 2).mean(axis=0))        # by column: its scales
    assert (np.abs(got - tiled) <= 2.0 ** -6 * (np.abs(tiled) + rms)).all()


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("group,K,N", [(32, 544, 544), (64, 576, 1088), (96, 672, 576), (128, 1152, 640), (256, 768, 512)])
def test_scale_table_in_a_large_launch(group, K, N, dtype):
    """More workgroups than two and a half for every CU: one activation buffer, odd and even numbers of stages and a last one
    that is short.  The first rows have the bits of a launch of their own, with two buffers, except where the larger launch takes the
    zero points by row sums as well (bf16, chunk-steps of 64)."""
    cfg = MoEConfig(name="t64_large", T=9000, K=K, N=N, E=4, topk=1, group=group, dtype=dtype, seed=22)
    print(f"blocks of 64, large launch {cfg}", flush=True)
    inp = make_inputs(cfg)
    few = copy.copy(inp)
    few.cfg = dataclasses.replace(cfg, T=150)
    few.x_bits, few.topk_ids, few.topk_weights = inp.x_bits[:150], inp.topk_ids[:150], inp.topk_weights[:150]
    large, small = _block_64(inp)[:150], _block_64(few)
    _check(few, large, "large launch")
    assert torch.equal(large, small) == (dtype == "f16" or group != 64)


@pytest.mark.parametrize("group,K,N", [(32, 160, 544), (64, 64, 1088), (96, 192, 672), (64, 640, 320)])
def test_few_groups_in_a_large_launch_of_32_slot_blocks(group, K, N):
    """fp16, up to five groups and (groups of 64) more than three workgroups for every CU: the tile that does not read its words
    ahead.  The first rows have the bits of a launch of their own, with groups of 64 on the tile that does."""
    cfg = MoEConfig(name="t32_large", T=6000, K=K, N=N, E=4, topk=1, group=group, dtype="f16", seed=23)
    print(f"blocks of 32, large launch {cfg}", flush=True)
    inp = make_inputs(cfg)
    few = copy.copy(inp)
    few.cfg = dataclasses.replace(cfg, T=150)
    few.x_bits, few.topk_ids, few.topk_weights = inp.x_bits[:150], inp.topk_ids[:150], inp.topk_weights[:150]
    M.moe_set_block_m_override(32)
    try:
        large, small = U.run_layer(U.DevInputs(inp))[:150], U.run_layer(U.DevInputs(few))
        torch.cuda.synchronize()
        assert M.moe_last_gemm_plan()["mt"] == 2
    finally:
        M.moe_set_block_m_override(0)
    _check(few, large, "large launch")
    assert torch.equal(large, small)

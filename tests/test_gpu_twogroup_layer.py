"""GPU parity of the layer on its two-group 256-slot tile (large batches, group 128): every number of
live 32-slot parts of a block, both weight layouts, reductions from the shortest the tile takes to
ones with an odd number of panels, several tiles per workgroup, zero scales and ignored ids."""
import numpy as np
import pytest
import torch

from moe_workloads import MoEConfig, make_inputs
from oracle import moe_oracle as O
from test_gpu_random_shapes import bf16_flip_allowance

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import gpu_util as U
    import paper_2504_16214_amd as M


def _inputs(dtype, K, N, counts, seed, zero_scales=False, bad_ids=0):
    """One slot per token, counts[e] of them on expert e, bad_ids of them on no expert."""
    E, T = len(counts), sum(counts) + bad_ids
    cfg = MoEConfig("tg", T=T, K=K, N=N, E=E, topk=1, group=128, dtype=dtype, seed=seed)
    inp = make_inputs(cfg)
    rng = np.random.default_rng(seed)
    ids = np.concatenate([np.repeat(np.arange(E), counts), rng.choice([-1, E, E + 7], size=bad_ids)]).astype(np.int32)
    rng.shuffle(ids)
    inp.topk_ids = ids.reshape(T, 1)
    inp.topk_weights = np.full((T, 1), 0.75, np.float32)
    if zero_scales:                    # single groups, a whole row, the first and the last group of rows
        inp.s1_bits[:, 3, 1] = 0
        inp.s1_bits[:, N + 5, :] = 0
        inp.s1_bits[1:, 40:44, 0] = 0
        inp.s2_bits[:, 17, -1] = 0
        inp.s2_bits[:, 64:66, 2] = 0
    return inp


def _layer(inp, prepacked=False, tiles=0):
    d, c = U.DevInputs(inp), inp.cfg
    mdt = M.MOE_F16 if c.dtype == "f16" else M.MOE_BF16
    out = torch.full((c.T, c.K), float("nan"), dtype=U.TORCH_DT[c.dtype], device="cuda")
    M.moe_set_block_m_override(256)
    M.moe_set_tiles_per_workgroup(tiles)
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
        plan = M.moe_last_gemm_plan()
        assert plan["mt"] == 16 and plan["waves"] == 8, plan
    finally:
        M.moe_set_block_m_override(0)
        M.moe_set_tiles_per_workgroup(0)
    return out


def _check(inp, out, what):
    """The plain bound; bf16 plus what one differently rounded activation may move (bf16_flip_allowance)."""
    c = inp.cfg
    want, mid = O.layer(O.decode_bits(inp.x_bits, c.dtype), inp.topk_ids, inp.topk_weights, inp.qw1,
                        O.decode_bits(inp.s1_bits, c.dtype), inp.z1, inp.qw2, O.decode_bits(inp.s2_bits, c.dtype),
                        inp.z2, c.group, c.dtype, return_intermediates=True)
    got = U.dev_to_f64(out)
    if c.dtype == "f16":
        U.assert_close(got, want, what)
        return
    assert np.all(np.isfinite(got)), what
    err, plain = np.abs(got - want), U.ATOL + U.RTOL * np.abs(want)
    assert np.all(err <= plain + bf16_flip_allowance(inp, mid)), what
    assert np.mean(err > plain) <= 1e-4, f"{what}: {np.mean(err > plain):.2e} of the outputs beyond the plain bound"


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("K,N,zero_scales", [(1024, 1024, True), (3072, 1024, False), (1024, 2048, False)])
def test_every_live_part_count(dtype, K, N, zero_scales):
    counts = [1, 32, 33, 64, 0, 96, 97, 128, 150, 192, 200, 224, 256, 257, 300]
    print(f"two-group layer {dtype} K={K} N={N}", flush=True)
    inp = _inputs(dtype, K, N, counts, seed=700 + K + N, zero_scales=zero_scales, bad_ids=5)
    got = _layer(inp)
    _check(inp, got, f"two-group layer {dtype} K={K} N={N}")
    bad = (inp.topk_ids[:, 0] < 0) | (inp.topk_ids[:, 0] >= inp.cfg.E)
    assert np.all(U.dev_to_f64(got)[bad] == 0)
    same = _layer(inp, prepacked=True)
    assert torch.equal(got.view(torch.int16), same.view(torch.int16)), "operand-order weights: same words, same order"


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_a_zero_scale_contributes_exactly_nothing(dtype):
    """Every live-part count.  A down row whose scales are all zero gives exact zeros; one whose only scale
    is its last group's 2^-20 gives the product of that group alone, which anything left behind by the seven
    groups before it would drown (their products are expressed in units of 1: one float32 rounding of
    them is as large as the whole result).  Bound in the 2-norm: two 16-bit roundings (activation, output)."""
    inp = _inputs(dtype, 1024, 1024, [1, 33, 70, 100, 150, 170, 200, 256], seed=803)
    c = inp.cfg
    inp.s2_bits[:, 16, :] = 0
    inp.s2_bits[:, 32, :] = 0
    inp.s2_bits[:, 32, -1] = O.encode_bits(np.array([2.0 ** -20]), dtype)[0]
    print(f"two-group layer {dtype}, rows of zero scales", flush=True)
    got = U.dev_to_f64(_layer(inp))
    assert np.all(got[:, 16] == 0)
    want = O.layer(O.decode_bits(inp.x_bits, dtype), inp.topk_ids, inp.topk_weights, inp.qw1,
                   O.decode_bits(inp.s1_bits, dtype), inp.z1, inp.qw2, O.decode_bits(inp.s2_bits, dtype),
                   inp.z2, c.group, dtype)
    # (fp16: an output of 2^-15 is subnormal and rounds to a multiple of 2^-24)
    abs_step = 2.0 ** -25 if dtype == "f16" else 0.0
    rms = np.sqrt(np.mean((got[:, 32] - want[:, 32]) ** 2))
    assert rms <= 2.0 ** -7 * np.sqrt(np.mean(want[:, 32] ** 2)) + 2 * abs_step


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("tiles", [1, 3, 8])
def test_tiles_per_workgroup(dtype, tiles):
    """Walking several feature tiles with one load pipeline gives the same bits as one tile each."""
    inp = _inputs(dtype, 2048, 1024, [20, 50, 250, 130], seed=801)
    print(f"two-group layer {dtype} tiles per workgroup {tiles}", flush=True)
    got = _layer(inp, tiles=tiles)
    _check(inp, got, f"tiles {tiles}")
    assert torch.equal(got.view(torch.int16), _layer(inp, tiles=1).view(torch.int16))


def test_small_workspace_falls_back():
    """bf16 without room for the row sums: the layer runs on the other tiles, within the same bound."""
    inp = _inputs("bf16", 1024, 1024, [100, 260], seed=802)
    d, c = U.DevInputs(inp), inp.cfg
    out = torch.empty((c.T, c.K), dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(M.moe_w4a16_layer_workspace_bytes(c.T, c.K, c.N, c.E, c.topk, M.MOE_BF16), dtype=torch.uint8, device="cuda")
    M.moe_set_block_m_override(256)
    try:
        M.moe_w4a16_layer(d.X, d.ids, d.w, d.qw1, d.s1, d.z1, d.qw2, d.s2, d.z2, out, c.group, ws)
        torch.cuda.synchronize()
        assert M.moe_last_gemm_plan()["mt"] == 8
    finally:
        M.moe_set_block_m_override(0)
    _check(inp, out, "fallback")


def test_scales_of_less_alignment_take_the_tiles_that_read_them():
    """8-byte aligned scale rows: the layer runs on a tile with a scale table, and asking for scales in
    registers is refused, as at every other token number."""
    inp = _inputs("f16", 1024, 1024, [100, 260], seed=804)
    print("two-group layer, 8-byte aligned scales", flush=True)
    d, c = U.DevInputs(inp), inp.cfg
    for name in ("s1", "s2"):
        t = getattr(d, name)
        room = torch.empty(t.numel() + 4, dtype=t.dtype, device="cuda")
        moved = room[4:].view(t.shape)
        moved.copy_(t)
        setattr(d, name, moved)
    assert d.s1.data_ptr() % 16 == 8
    M.moe_set_block_m_override(256)
    try:
        out = U.run_layer(d)
        assert M.moe_last_gemm_plan()["mt"] == 8 and M.moe_last_gemm_plan()["register_scales"] == 0
        M.moe_set_scale_path(2)
        with pytest.raises(M.MoEError) as e:
            U.run_layer(d)
        assert e.value.status == 2
    finally:
        M.moe_set_scale_path(0)
        M.moe_set_block_m_override(0)
    _check(inp, out, "8-byte aligned scales")


def test_automatic_choice_through_the_three_entries():
    """bf16, several slots a token (the row sums of X are gathered by token, not by slot), the workspace of
    the size query and no override: the plain layer against the oracle, the prepacked and the routed one
    with the same bits."""
    cfg = MoEConfig("tg_auto", T=3200, K=1024, N=1024, E=64, topk=4, group=128, dtype="bf16", seed=805)
    print(f"two-group layer, automatic choice {cfg}", flush=True)
    inp = make_inputs(cfg)
    d = U.DevInputs(inp)
    logits = torch.from_numpy(inp.logits).cuda()
    M.moe_route_topk(logits, None, d.ids, d.w)
    inp.topk_ids, inp.topk_weights = d.ids.cpu().numpy(), d.w.cpu().numpy()

    def on_two_group():
        plan = M.moe_last_gemm_plan()
        return plan["mt"] == 16 and plan["waves"] == 8

    got = U.run_layer(d)
    assert on_two_group()
    _check(inp, got, "plain entry")
    sizes = (cfg.T, cfg.K, cfg.N, cfg.E, cfg.topk, M.MOE_BF16)
    p1, p2 = torch.empty_like(d.qw1), torch.empty_like(d.qw2)
    M.moe_repack_qweight(d.qw1, False, p1)
    M.moe_repack_qweight(d.qw2, True, p2)
    out = torch.full_like(got, float("nan"))
    ws = torch.full((M.moe_w4a16_layer_workspace_bytes(*sizes),), 255, dtype=torch.uint8, device="cuda")
    M.moe_w4a16_layer_prepacked(d.X, d.ids, d.w, p1, d.s1, d.z1, p2, d.s2, d.z2, out, cfg.group, ws)
    torch.cuda.synchronize()
    assert on_two_group() and torch.equal(out.view(torch.int16), got.view(torch.int16))
    out = torch.full_like(got, float("nan"))
    ws = torch.full((M.moe_w4a16_routed_layer_workspace_bytes(*sizes),), 255, dtype=torch.uint8, device="cuda")
    M.moe_w4a16_routed_layer(d.X, logits, None, d.qw1, d.s1, d.z1, d.qw2, d.s2, d.z2, out, cfg.topk, cfg.group, ws)
    torch.cuda.synchronize()
    assert on_two_group() and torch.equal(out.view(torch.int16), got.view(torch.int16))

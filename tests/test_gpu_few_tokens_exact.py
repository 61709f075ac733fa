"""GPU tests of the few-token layer's integer sums at their limits: activations that a chunk of 32 cannot all hold in 30 bits
(fp16; bf16 has them rounded to 2^-30 of the largest), and large ones whose weights are their zero points, which must leave nothing.  Both types and weight layouts, whole output
against the float64 oracle.

Bound: gate, up, act and output are rounded to 16 bits; if the sums' last bits moved every one of these roundings, the
difference would be four units of 2^-10 (fp16) or 2^-7 (bf16) of the result, in the 2-norm.  An outlier that left 2^-24 of
15 times itself, or digits that were cut off, are far beyond it at the ratios used."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from moe_workloads import MoEConfig, make_inputs
from oracle import moe_oracle as O
from test_gpu_random_shapes import say

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2504_16214_amd as M
    import gpu_util as U

BOUND = {"f16": 4 * 2.0 ** -10, "bf16": 4 * 2.0 ** -7}
K = N = 1024


def near_zero_points(rng, z, red, where):
    """Nibbles within one of their zero point, equal to it at the reduction indices `where`."""
    zz = np.repeat(z.astype(np.int64), 128, axis=-1)
    d = rng.integers(-1, 2, size=zz.shape)
    d[..., where] = 0
    return O.pack_int4(np.clip(zz + d, 0, 15))


def layer(inp, order):
    c = inp.cfg
    d = U.DevInputs(inp)
    if order == "operand":
        p1, p2 = torch.empty_like(d.qw1), torch.empty_like(d.qw2)
        M.moe_repack_qweight(d.qw1, False, p1)
        M.moe_repack_qweight(d.qw2, True, p2)
        d.qw1, d.qw2 = p1, p2
    ws = torch.empty(M.moe_w4a16_layer_workspace_bytes(c.T, K, N, c.E, c.topk, M.MOE_F16 if c.dtype == "f16" else M.MOE_BF16), dtype=torch.uint8, device="cuda")
    out = torch.full((c.T, K), float("nan"), dtype=U.TORCH_DT[c.dtype], device="cuda")
    (M.moe_w4a16_layer_prepacked if order == "operand" else M.moe_w4a16_layer)(d.X, d.ids, d.w, d.qw1, d.s1, d.z1, d.qw2, d.s2, d.z2, out, 128, ws)
    torch.cuda.synchronize()
    assert M.moe_last_gemm_plan()["mt"] == 0
    return U.dev_to_f64(out)


def check(inp, x, s1, s2, order, what):
    c = inp.cfg
    inp.x_bits = O.encode_bits(x, c.dtype)
    inp.s1_bits, inp.s2_bits = O.encode_bits(s1, c.dtype), O.encode_bits(s2, c.dtype)
    say(f"exact sums {what} {order} {c}")
    got = layer(inp, order)
    want = O.layer(O.decode_bits(inp.x_bits, c.dtype), inp.topk_ids, inp.topk_weights, inp.qw1, O.decode_bits(inp.s1_bits, c.dtype), inp.z1,
                   inp.qw2, O.decode_bits(inp.s2_bits, c.dtype), inp.z2, 128, c.dtype)
    assert np.isfinite(want).all() and np.isfinite(got).all() and np.linalg.norm(want) > 0
    err = np.linalg.norm(got - want) / np.linalg.norm(want)
    say(f"  error {err:.2e}")
    assert err <= BOUND[c.dtype]


def inputs(dtype, seed):
    return make_inputs(MoEConfig("few_exact", T=2, K=K, N=N, E=8, topk=1, group=128, dtype=dtype, seed=seed)), np.random.default_rng(seed)


@pytest.mark.parametrize("order", ["plain", "operand"])
@pytest.mark.parametrize("dtype,ratio", [("f16", 12), ("f16", 20), ("f16", 28), ("bf16", 12), ("bf16", 20)])
def test_a_large_activation_whose_weights_are_zero(dtype, ratio, order):
    """One activation of every chunk 2^ratio times the rest, which then fit 30 bits beside it, or do not (fp16, 28)."""
    inp, rng = inputs(dtype, ratio)
    where = np.arange(0, K, 32) + rng.integers(0, 32, K // 32)
    small = 2.0 ** (15.5 - ratio if dtype == "f16" else 0)
    x = rng.normal(size=(2, K)).clip(-3, 3) * small / 4
    x[:, where] = np.where(rng.random((2, K // 32)) < 0.5, -1, 1) * small * 2.0 ** ratio
    inp.qw1 = near_zero_points(rng, inp.z1, K, where)
    s1 = np.full(inp.s1_bits.shape, 0.1 / small) * rng.uniform(0.7, 1.3, inp.s1_bits.shape)
    inp.qw2 = near_zero_points(rng, inp.z2, N, np.array([], dtype=int))
    check(inp, x, s1, rng.uniform(0.05, 0.1, inp.s2_bits.shape), order, f"x 2^{ratio}")


@pytest.mark.parametrize("order", ["plain", "operand"])
def test_three_large_activations_whose_weights_are_zero(order):
    """The most large values of a chunk beside which small ones are kept, 2^-24 of them: nothing else is left of the chunk."""
    inp, rng = inputs("f16", 24)
    where = np.concatenate([32 * c + rng.permutation(32)[:3] for c in range(K // 32)])
    small = 2.0 ** (15 - 24)
    x = rng.normal(size=(2, K)).clip(-3, 3) * small / 4
    x[:, where] = np.where(rng.random((2, where.size)) < 0.5, -1, 1) * small * 2.0 ** 24
    inp.qw1 = near_zero_points(rng, inp.z1, K, where)
    s1 = np.full(inp.s1_bits.shape, 0.1 / small) * rng.uniform(0.7, 1.3, inp.s1_bits.shape)
    inp.qw2 = near_zero_points(rng, inp.z2, N, np.array([], dtype=int))
    check(inp, x, s1, rng.uniform(0.05, 0.1, inp.s2_bits.shape), order, "three")


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_wide_activations(dtype):
    """Values over eight decades and act in the hundreds, any weights: chunks of every kind."""
    inp, rng = inputs(dtype, 10)
    x = rng.normal(size=(2, K)) * np.exp(1.5 * rng.normal(size=(2, K)))
    check(inp, x, rng.uniform(0.02, 0.06, inp.s1_bits.shape) / 4, rng.uniform(0.002, 0.004, inp.s2_bits.shape), "plain", "wide")


@pytest.mark.parametrize("order", ["plain", "operand"])
@pytest.mark.parametrize("dtype,ratio", [("f16", 14), ("f16", 24), ("bf16", 14), ("bf16", 20)])
def test_a_large_act_whose_weights_are_zero(dtype, ratio, order):
    """The same for the down product: one column of act in every chunk has up scales 2^ratio times the others'."""
    inp, rng = inputs(dtype, 100 + ratio)
    where = np.arange(0, N, 32) + rng.integers(0, 32, N // 32)
    x = rng.normal(size=(2, K)).clip(-3, 3)
    none = np.array([], dtype=int)
    inp.qw1, inp.qw2 = near_zero_points(rng, inp.z1, K, none), near_zero_points(rng, inp.z2, N, where)
    s1 = rng.uniform(0.02, 0.06, inp.s1_bits.shape)
    low = 2.0 ** -(ratio - 10)
    s1[:, N:] *= low
    s1[:, N + where] *= 2.0 ** ratio
    check(inp, x, s1, rng.uniform(0.05, 0.1, inp.s2_bits.shape) / low, order, f"act 2^{ratio}")


@pytest.mark.parametrize("order", ["plain", "operand"])
def test_bf16_activations_near_the_smallest_normal_number(order):
    inp, rng = inputs("bf16", 7)
    none = np.array([], dtype=int)
    inp.qw1, inp.qw2 = near_zero_points(rng, inp.z1, K, none), near_zero_points(rng, inp.z2, N, none)
    x = rng.normal(size=(2, K)).clip(-3, 3) * 2.0 ** -121
    check(inp, x, rng.uniform(0.02, 0.06, inp.s1_bits.shape) * 2.0 ** 121, rng.uniform(0.05, 0.1, inp.s2_bits.shape), order, "tiny")


@pytest.mark.parametrize("order", ["plain", "operand"])
def test_a_bf16_chunk_whose_sum_is_beyond_float32(order):
    """32 times 1.5 * 2^127, weights at their zero points."""
    inp, rng = inputs("bf16", 8)
    inp.qw1, inp.qw2 = near_zero_points(rng, inp.z1, K, np.arange(64, 96)), near_zero_points(rng, inp.z2, N, np.array([], dtype=int))
    x = rng.normal(size=(2, K)).clip(-3, 3)
    x[:, 64:96] = 1.5 * 2.0 ** 127
    check(inp, x, rng.uniform(0.02, 0.06, inp.s1_bits.shape), rng.uniform(0.05, 0.1, inp.s2_bits.shape), order, "huge")


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_values_beside_digits_in_one_group(dtype):
    """Chunks that are kept as they are beside chunks of digits, every weight random: the sums of both kinds meet."""
    inp, rng = inputs(dtype, 9)
    x = rng.normal(size=(2, K)).clip(-3, 3)
    for c in (0, 5, 6, 17, 31):
        x[:, 32 * c:32 * c + 32] = rng.normal(size=(2, 32)) * np.where(np.arange(32) % 11 == 0, 100.0, 3e-6 if dtype == "f16" else 1e-9)
    check(inp, x, rng.uniform(0.002, 0.004, inp.s1_bits.shape), rng.uniform(0.002, 0.02, inp.s2_bits.shape), "plain", "mixed")

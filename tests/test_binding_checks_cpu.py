"""The layer's one-expression check accepts nothing that the checks which name a fault would refuse, and accepts a right call."""
import pytest
import torch

from paper_2504_16214_amd import binding as B

T, K, N, E, TOPK, G = 3, 256, 128, 2, 2, 64


def right(dt=torch.float16, routed=False):
    i32, u8 = torch.int32, torch.uint8
    a = dict(X=torch.zeros(T, K, dtype=dt), topk_ids=torch.zeros(T, TOPK, dtype=i32), topk_weights=torch.zeros(T, TOPK),
             qw1=torch.zeros(E, 2 * N, K // 8, dtype=i32), s1=torch.zeros(E, 2 * N, K // G, dtype=dt), z1=torch.zeros(E, 2 * N, K // G, dtype=u8),
             qw2=torch.zeros(E, K, N // 8, dtype=i32), s2=torch.zeros(E, K, N // G, dtype=dt), z2=torch.zeros(E, K, N // G, dtype=u8),
             out=torch.zeros(T, K, dtype=dt), group_size=G)
    if routed:
        a["topk_ids"] = a["topk_weights"] = None
    return a


def named(args):
    """The verdict of the checks that name a fault."""
    keep = B._layer_is_right
    B._layer_is_right = lambda *a: False
    try:
        B._expect_layer(**args)
        return True
    except (ValueError, AttributeError, TypeError):
        return False
    finally:
        B._layer_is_right = keep


@pytest.mark.parametrize("dt", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("routed", [False, True])
def test_a_right_call_is_accepted(dt, routed):
    args = right(dt, routed)
    assert B._layer_is_right(**args) and named(args)


@pytest.mark.parametrize("name", [n for n in right() if n != "group_size"])
@pytest.mark.parametrize("change", ["none", "dtype", "transposed", "longer", "shorter", "flat", "extra dimension"])
def test_a_wrong_argument_is_not_accepted(name, change):
    args = right()
    t = args[name]
    args[name] = {"none": lambda: None, "dtype": lambda: t.to(torch.float64), "transposed": lambda: t.transpose(0, -1),
                  "longer": lambda: torch.cat([t, t], dim=-1), "shorter": lambda: t[..., :-1], "flat": lambda: t.reshape(-1),
                  "extra dimension": lambda: t[None]}[change]()
    assert not B._layer_is_right(**args) or named(args)
    if change in ("dtype", "longer", "flat", "extra dimension") and not (name in ("topk_ids", "topk_weights") and change == "longer"):
        assert not B._layer_is_right(**args)


@pytest.mark.parametrize("group", [0, -64, 32, 96, 128, 512])
def test_another_group_size_gets_the_named_verdict(group):
    args = right()
    args["group_size"] = group
    assert not B._layer_is_right(**args) or named(args)

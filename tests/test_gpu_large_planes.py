"""Outputs past the reach of 32-bit row offsets (about 4 GB): the tiles of 64 rows and more and the two-group tile store
them by another form.  Sampled rows, first, last and at block borders, against float64."""
import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import gpu_util as U
    import paper_2504_16214_amd as M

LIMIT = 0xF0000000        # bytes of a plane that offsets serve


def _int4(gen, *shape_rows_red, group, dtype):
    *lead, rows, red = shape_rows_red
    q = torch.randint(-2 ** 31, 2 ** 31, (*lead, rows, red // 8), generator=gen, device="cuda", dtype=torch.int32)
    s = (torch.rand(*lead, rows, red // group, generator=gen, device="cuda") * 0.018 + 0.002).to(dtype)
    z = torch.randint(0, 16, (*lead, rows, red // group), generator=gen, device="cuda", dtype=torch.uint8)
    return q, s, z


def _dequant(q, s, z, group):
    shifts = torch.arange(0, 32, 4, device="cuda", dtype=torch.int32)
    nib = ((q[..., None] >> shifts) & 15).flatten(-2).double()
    return (nib - z.double().repeat_interleave(group, -1)) * s.double().repeat_interleave(group, -1)


@pytest.mark.parametrize("m,n", [(32784, 61440), (32752, 61440)])      # just past the limit, just below it
def test_dense_output_of_four_gigabytes(m, n):
    k, group = 64, 32
    assert (2 * m * n > LIMIT) == (m == 32784)
    gen = torch.Generator(device="cuda").manual_seed(5)
    x = (0.5 * torch.randn(m, k, generator=gen, device="cuda")).half()
    q, s, z = _int4(gen, n, k, group=group, dtype=torch.float16)
    out = torch.full((m, n), float("nan"), dtype=torch.float16, device="cuda")
    M.moe_w4a16_dense_gemm(x, q, s, z, group, out)
    rows = torch.tensor([0, 1, 63, 64, m // 2 + 3, m - 17, m - 16, m - 1], device="cuda")
    U.assert_close(U.dev_to_f64(out[rows]), (x[rows].double() @ _dequant(q, s, z, group).t()).cpu().numpy(), f"dense {m}x{n}")
    assert not torch.isnan(out.sum(dim=1, dtype=torch.float32)).any()


@pytest.mark.parametrize("t", [131071, 122800])      # float32 planes past the limit, just below it
def test_two_group_layer_of_four_gigabytes(t):
    k = n = 1024
    e = topk = 8
    assert (4 * t * topk * k > LIMIT) == (t == 131071)
    gen = torch.Generator(device="cuda").manual_seed(6)
    x = (0.5 * torch.randn(t, k, generator=gen, device="cuda")).half()
    w1, w2 = _int4(gen, e, 2 * n, k, group=128, dtype=torch.float16), _int4(gen, e, k, n, group=128, dtype=torch.float16)
    ids = torch.rand(t, e, generator=gen, device="cuda").argsort(dim=1).int().contiguous()
    w = torch.softmax(torch.randn(t, topk, generator=gen, device="cuda"), dim=1).contiguous()
    out = torch.full((t, k), float("nan"), dtype=torch.float16, device="cuda")
    ws = torch.empty(M.moe_w4a16_layer_workspace_bytes(t, k, n, e, topk, M.MOE_F16), dtype=torch.uint8, device="cuda")
    M.moe_w4a16_layer(x, ids, w, *w1, *w2, out, 128, ws)
    assert M.moe_last_gemm_plan()["mt"] == 16
    rows = torch.tensor([0, 1, 255, 256, t // 2 + 5, t - 2, t - 1], device="cuda")
    want = torch.zeros(len(rows), k, dtype=torch.float64, device="cuda")
    for i in range(e):
        h = (x[rows].double() @ _dequant(*(v[i] for v in w1), 128).t()).half().double()
        act = (h[:, :n] * torch.sigmoid(h[:, :n]) * h[:, n:]).half().double()
        share = (w[rows].double() * (ids[rows] == i)).sum(dim=1)
        want += share[:, None] * (act @ _dequant(*(v[i] for v in w2), 128).t())
    U.assert_close(U.dev_to_f64(out[rows]), want.cpu().numpy(), f"two-group layer, {t} tokens")
    assert not torch.isnan(out.sum(dim=1, dtype=torch.float32)).any()
